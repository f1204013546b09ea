"""GPU: speculative accept at the edges of its launches (statistics chunks of
12288 entries, draw chunks of 1024 and 4096, one entry, many batch rows),
eager against the oracle and captured against eager."""
import numpy as np
import pytest
import torch

import oracle
import paper_2603_19610_amd as pv
from gpu_util import note, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,gamma,V,tau", [
    (1, 1, 1, 1.0), (1, 1, 5, 0.7), (2, 3, 1023, 1.0), (2, 3, 1025, 1.0), (1, 2, 12288, 0.5), (1, 2, 12289, 1.0),
    (3, 32, 4097, 1.0), (256, 1, 1024, 1.0), (256, 1, 1025, 1.0), (5, 4, 65537, 1.3), (2, 2, 30001, 0.0)])
def test_launch_edges(B, gamma, V, tau):
    note(f"accept edge B={B} gamma={gamma} V={V} tau={tau}")
    rng = np.random.default_rng(B + gamma + V)
    z = rng.standard_normal((B, gamma + 1, V)).astype(np.float32) * 2
    target = z + rng.standard_normal(z.shape).astype(np.float32) * np.float32(0.4)
    draft = np.ascontiguousarray(z[:, :gamma])
    tok = draft.argmax(axis=-1).astype(np.int32)
    ua, us = rng.random((B, gamma)), rng.random(B)
    args = [to_dev(x) for x in (draft, target, tok, ua, us)]
    ws = pv.Workspace(torch.device("cuda", 0))
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    got = [t.clone() for t in pv.spec_accept(*args, tau, ws=ws, status=status)]
    torch.cuda.synchronize()
    rn, ry, rt = oracle.spec_accept(draft, target, tok, ua, us, tau)
    n, y, tie = (t.cpu().numpy() for t in got)
    ok = (rt == 0) & (tie == 0)
    assert int(status.item()) == 0 and ok.mean() > 0.9
    assert np.array_equal(n[ok], rn[ok]) and np.array_equal(y[ok], ry[ok])
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        outs = pv.spec_accept(*args, tau, ws=ws, status=status)
    for _ in range(3):
        for t in outs:
            t.fill_(-9)
        g.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(outs, got))
        again = pv.spec_accept(*args, tau, ws=ws, status=status)
        assert all(torch.equal(a, b) for a, b in zip(again, got))
