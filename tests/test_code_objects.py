"""The instructions of the built kernels, where nothing but a look at them
shows a fault (not gpu)."""
import re

import code_objects


def test_lds_loads_do_not_directly_follow_their_m0(tmp_path):
    """A load into LDS takes its LDS address from M0 and needs one wait state
    after a scalar write of M0 (an s_nop or any other instruction between); the
    compiler inserts it for its own loads, not inside inline asm."""
    loads, early = 0, []
    for obj in code_objects.disassembly(str(tmp_path)):
        for before, ins in zip(obj, obj[1:]):
            if re.match(r"(global|scratch)_load_lds_|buffer_load_\w+ .*\blds\b", ins):
                loads += 1
                if re.match(r"s_\w+ m0,", before):
                    early.append((before, ins))
    assert loads > 0
    assert not early, f"{len(early)} of {loads}: {early[:3]}"
