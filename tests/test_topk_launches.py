"""GPU: the fused score and top-k where its launches hand the scores on."""
import numpy as np
import pytest
import torch

import paper_2603_19610_amd as pv
from gpu_util import note, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layer", [0, -1])
@pytest.mark.parametrize("m_cap", [12544, 16385, 131072])
def test_scores_written_over_a_criterion(m_cap, layer):
    """The scores may take the place of either criterion they come from: the
    launches after the first must not read the criteria again."""
    B = 3
    rng = np.random.default_rng(m_cap)
    stack = rng.standard_normal((3, B, m_cap)).astype(np.float32)
    stack[:, :, ::7] = stack[:, :, :1]
    m = np.array([m_cap, m_cap - 17, m_cap // 3], np.int32)
    k = np.array([m_cap // 10, m_cap // 3, 0], np.int32)
    note(f"topk in place m_cap={m_cap} layer={layer}")
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    d_stack, d_m, d_k = to_dev(stack), to_dev(m), to_dev(k)
    score, idx = pv.uvprune_topk_mass(d_stack, d_m, d_k, int(k.max()), status=status)
    over, idx2 = pv.uvprune_topk_mass(d_stack, d_m, d_k, int(k.max()), score=d_stack[layer], status=status)
    torch.cuda.synchronize()
    assert int(status.item()) == 0
    assert over.data_ptr() == d_stack[layer].data_ptr()
    assert torch.equal(over.view(torch.int32), score.view(torch.int32))
    assert torch.equal(idx2, idx)
