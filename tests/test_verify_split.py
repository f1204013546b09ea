"""GPU: verify attention at the edges of its plan -- stage and chunk
boundaries, every number of row tiles, the resident and the two-pass form of
the mass (eager against captured, bit for bit), fp32, unaligned views --
against the float64 oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2603_19610_amd as pv
import workloads as W
from gpu_util import assert_lse, assert_mass, assert_out, f64, note, to_dev, to_host_f64

pytestmark = pytest.mark.gpu


def _eager_and_graph(inp, ws):
    """(eager, captured) results of one call; the graph is replayed three times
    with eager work between, every replay equal."""
    args = [to_dev(x) for x in (inp.q, inp.k, inp.v, inp.ctx_len)]
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    kw = dict(scale=inp.scale, max_ctx=int(inp.ctx_len.max()), ws=ws, status=status)
    eager = [t.clone() for t in pv.verify_attn(*args, **kw)]
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        outs = pv.verify_attn(*args, **kw)
    for _ in range(3):
        for t in outs:
            t.fill_(7.0)
        g.replay()
        torch.cuda.synchronize()
        assert int(status.item()) == 0
        assert all(torch.equal(a, b) for a, b in zip(outs, eager))
        again = pv.verify_attn(*args, **kw)
        assert all(torch.equal(a, b) for a, b in zip(again, eager))
    return eager


def _check(inp, got, hq, T):
    ro, rl, rm = oracle.verify_attn(f64(inp.q, inp.dtype), f64(inp.k, inp.dtype), f64(inp.v, inp.dtype),
                                    inp.ctx_len, inp.scale)
    out, mass, lse = (to_host_f64(t) for t in got)
    if inp.dtype == "f32":  # 32-bit sums and exponentials over a few thousand terms
        assert np.abs(out - ro).max() <= 2e-5 * max(1.0, np.abs(ro).max())
    else:
        assert_out(out, ro)
    assert_lse(lse, rl)
    assert_mass(mass, rm, hq, T)


@pytest.mark.parametrize("shape", [
    # B, T, Hq, Hkv, D, ctx, dtype
    (1, 1, 1, 1, 128, [0], "bf16"),                # one row, one token
    (1, 1, 4, 4, 128, [62], "bf16"),               # one stage short of a row, full, one over
    (1, 1, 4, 4, 128, [63], "bf16"),
    (1, 1, 4, 4, 128, [64], "bf16"),
    (1, 1, 4, 4, 128, [127], "bf16"),              # one chunk of two stages, then a second of one row
    (1, 1, 4, 4, 128, [128], "bf16"),
    (2, 2, 32, 2, 64, [191, 3], "bf16"),           # two row tiles, D = 64, a second sequence of one block
    (1, 3, 16, 1, 128, [2047], "bf16"),            # three tiles
    (1, 4, 32, 2, 128, [515], "bf16"),             # four
    (1, 9, 64, 8, 128, [14300], "bf16"),           # five, seven resident stages
    (1, 9, 64, 8, 128, [14400], "bf16"),           # ... and one too many: two passes
    (1, 6, 16, 1, 128, [1000], "bf16"),            # six
    (1, 7, 16, 1, 128, [1000], "bf16"),            # seven tiles as two workgroups' four and three
    (1, 15, 32, 4, 64, [30000], "bf16"),           # eight in one workgroup
    (1, 9, 16, 1, 64, [70000], "bf16"),            # nine
    (1, 32, 20, 1, 128, [333], "bf16"),            # 640 rows: 40 tiles
    (3, 5, 7, 1, 128, [5000, 0, 257], "bf16"),     # padding rows, empty chunks
    (1, 1, 8, 8, 128, [20000], "bf16"),            # one tile, ten stages resident
    (1, 2, 32, 8, 64, [4096], "bf16"),             # D = 64: one workgroup a compute unit, resident
    (1, 4, 32, 8, 64, [8192], "bf16"),
    (1, 4, 32, 8, 64, [2100], "f32"),
    (40, 2, 32, 8, 64, [300] * 40, "bf16"),        # 320 workgroups: more than fit, so two passes
    (1, 5, 4, 1, 64, [31], "f32"),                 # fp32 stages of 32 rows
    (1, 5, 4, 1, 64, [1024], "f32"),
    (2, 7, 14, 2, 128, [95, 31], "f32"),           # four fp32 tiles
    (1, 16, 9, 1, 64, [2900], "f32"),              # nine fp32 tiles
], ids=lambda s: f"B{s[0]}T{s[1]}H{s[2]}/{s[3]}D{s[4]}c{s[5][0]}{s[6]}")
def test_plan_edges(shape):
    B, T, Hq, Hkv, D, ctx, dt = shape
    inp = W.random_verify_inputs(B, T, Hq, Hkv, D, ctx, dt, seed=sum(ctx) + Hq + T, n_cap=max(ctx) + T + 37)
    note(f"verify plan edge q{inp.q.shape} k{inp.k.shape} ctx={ctx} {dt}")
    _check(inp, _eager_and_graph(inp, pv.Workspace(torch.device("cuda", 0))), Hq, T)


def test_captured_forms_share_a_workspace():
    """Resident launches leave their statistics records cleared: two shapes
    captured over one workspace, replayed in turn, keep their results."""
    ws = pv.Workspace(torch.device("cuda", 0))
    note("verify: two captured shapes over one workspace")
    for ctx, T in ([1500], 9), ([4000], 4), ([1500], 9):
        inp = W.random_verify_inputs(1, T, 32, 4, 128, ctx, "bf16", seed=T)
        _check(inp, _eager_and_graph(inp, ws), 32, T)


@pytest.mark.parametrize("dt", ["bf16", "f32"])
def test_unaligned_views(dt):
    """Contiguous views that start one element into their storage."""
    inp = W.random_verify_inputs(1, 4, 8, 2, 128, [300], dt, seed=5)
    note(f"verify unaligned views {dt}")

    def shift(x):
        t = to_dev(x)
        return torch.cat([t.new_zeros(1), t.flatten()])[1:].view(t.shape)

    got = pv.verify_attn(shift(inp.q), shift(inp.k), shift(inp.v), to_dev(inp.ctx_len), scale=inp.scale)
    torch.cuda.synchronize()
    _check(inp, got, 8, 4)


def test_mass_of_a_long_page_table():
    """More logical cache rows than the finish kernel has workgroups times
    rows: its workgroups take several pieces each, and the rows past the
    sequence are 0."""
    inp = W.random_verify_inputs(1, 3, 4, 1, 64, [100], "bf16", seed=8, n_cap=128)
    pages = (1 << 24) // 32 + 1000
    note(f"verify: page table of {pages} pages")
    q, ctx = to_dev(inp.q), to_dev(inp.ctx_len)
    k, v = (to_dev(x).view(1, 1, 4, 32, 64).transpose(1, 2).reshape(4, 1, 32, 64).contiguous()
            for x in (inp.k, inp.v))
    table = torch.full((1, pages), -1, dtype=torch.int32, device="cuda")
    table[0, :4] = torch.arange(4, dtype=torch.int32, device="cuda")
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    got = pv.verify_attn_paged(q, k, v, table, ctx, scale=inp.scale, max_ctx=100, status=status,
                               mass=torch.full((1, 32 * pages), 5.0, device="cuda"))
    ref = pv.verify_attn(q, to_dev(inp.k), to_dev(inp.v), ctx, scale=inp.scale, max_ctx=100, status=status)
    torch.cuda.synchronize()
    assert int(status.item()) == 0
    assert torch.equal(got[0], ref[0]) and torch.equal(got[2], ref[2])
    assert torch.equal(got[1][:, :103], ref[1][:, :103]) and not got[1][:, 103:].any()


def test_workspace_of_the_queried_size_on_a_budgeted_stream():
    """Seven and more tiles, and chunks that only the budget makes long: the
    size asked for without a stream is enough."""
    inp = W.random_verify_inputs(8, 32, 4, 1, 64, [4096] + [700] * 7, "bf16", seed=12)
    note("verify: queried workspace on a stream of 128 compute units")
    s = torch.cuda.Stream()
    pv.set_stream_cu_budget(s, 128)
    try:
        args = [to_dev(x) for x in (inp.q, inp.k, inp.v, inp.ctx_len)]
        ws = pv.Workspace(torch.device("cuda", 0))
        torch.cuda.synchronize()
        with torch.cuda.stream(s):
            got = pv.verify_attn(*args, scale=inp.scale, max_ctx=4096, ws=ws)
        torch.cuda.synchronize()
    finally:
        pv.set_stream_cu_budget(s, 0)
    _check(inp, got, 4, 32)
