"""GPU: the co-residency contract of the calls whose workgroups wait on each
other (verify attention with mass, captured into a graph while its chunks'
scores stay in registers), and calls on several streams at once.

The waits rely on every workgroup becoming resident.  Another stream's bounded
kernels (here GEMMs) can hold compute units for a while; the waits then last
until those kernels retire.  A replay must then give exactly the eager result,
or flag PVLM_DEV_TIMEOUT when a wait gave up: never a silently wrong result.
Two waiting graphs may run together on streams whose budgets fit the device.
Default workspaces are per stream, so calls on two streams never share
records."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import paper_2603_19610_amd as pv
import workloads as W
from gpu_util import assert_mass, assert_out, f64, note, to_dev, to_host_f64

pytestmark = pytest.mark.gpu


def _kernels(graph):
    """Kernel nodes of a captured graph (CUDAGraph(keep_graph=True))."""
    hip = ctypes.CDLL("libamdhip64.so")
    raw, n = ctypes.c_void_p(graph.raw_cuda_graph()), ctypes.c_size_t(0)
    assert hip.hipGraphGetNodes(raw, None, ctypes.byref(n)) == 0
    return n.value


WAITING = 2  # launches of the waiting form: the partial kernel, the finish; three where it is two passes


def test_captured_verify_beside_busy_stream():
    w = W.WORKLOADS["llava72b"]
    inp = W.make_verify_inputs(w, layer=1)
    q, k, v, ctx = to_dev(inp.q), to_dev(inp.k), to_dev(inp.v), to_dev(inp.ctx_len)
    dev = q.device
    note("concurrency: eager reference")
    ref = pv.verify_attn(q, k, v, ctx, ws=pv.Workspace(dev))
    torch.cuda.synchronize()
    out = torch.empty_like(ref[0])
    mass = torch.empty_like(ref[1])
    lse = torch.empty_like(ref[2])
    ws = pv.Workspace(dev)
    status = torch.zeros(1, dtype=torch.int32, device=dev)
    pv.verify_attn(q, k, v, ctx, out=out, mass=mass, lse=lse, ws=ws, status=status)  # sizes ws
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(g):
        pv.verify_attn(q, k, v, ctx, out=out, mass=mass, lse=lse, ws=ws, status=status)
    assert _kernels(g) == WAITING
    g.instantiate()
    torch.cuda.synchronize()
    other = torch.cuda.Stream()
    a = torch.randn((4096, 4096), device=dev, dtype=torch.bfloat16)
    b = torch.randn((4096, 4096), device=dev, dtype=torch.bfloat16)
    equal = timeouts = 0
    for rep in range(4):
        note(f"concurrency: replay {rep} beside GEMMs on another stream")
        status.zero_()
        out.zero_()
        torch.cuda.synchronize()
        with torch.cuda.stream(other):
            for _ in range(6):
                c = a @ b
        g.replay()                     # no dependency on the other stream
        torch.cuda.synchronize()
        st = int(status.item())
        if st & pv.PVLM_DEV_TIMEOUT:
            timeouts += 1
            ws.buf.zero_()             # records undefined after a timeout
            torch.cuda.synchronize()
            continue
        assert st == 0, f"device status {st}"
        assert torch.equal(out, ref[0]) and torch.equal(mass, ref[1]) and torch.equal(lse, ref[2])
        equal += 1
    del c
    print(f"[concurrency] {equal} replays equal to eager, {timeouts} flagged a timeout", flush=True)
    assert equal + timeouts == 4


def test_default_workspaces_are_per_stream():
    w = W.WORKLOADS["llava7b"]
    inp = W.make_verify_inputs(w, layer=1)
    q, k, v, ctx = to_dev(inp.q), to_dev(inp.k), to_dev(inp.v), to_dev(inp.ctx_len)
    note("concurrency: default workspaces on two streams")
    ref = pv.verify_attn(q, k, v, ctx, ws=pv.Workspace(q.device))
    torch.cuda.synchronize()
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    outs = []
    for s in (s1, s2):
        s.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(s):
            outs.append(pv.verify_attn(q, k, v, ctx))
        torch.cuda.current_stream().wait_stream(s)   # the calls do not overlap
    assert pv.synchronize() == 0
    key = lambda s: ("verify", torch.cuda.current_device(), s.cuda_stream)
    assert pv._ws_cache[key(s1)].buf.data_ptr() != pv._ws_cache[key(s2)].buf.data_ptr()
    for o in outs:
        assert torch.equal(o[0], ref[0]) and torch.equal(o[1], ref[1]) and torch.equal(o[2], ref[2])


@pytest.mark.parametrize("budgets,first", [((224, 32), "72b"), ((128, 128), "72b"), ((224, 32), "nine-tiles")])
def test_two_budgeted_streams_run_eager_calls_together(budgets, first):
    """Verify (72B layer, or 136 rows per KV head over a 20K-token cache: nine
    row tiles in one workgroup) on one budgeted stream and verify + accept (7B
    layer) on another, called eagerly, enqueued together and repeated: every
    result equals the same call's result on a lone stream with the same
    budget (none of these launches waits; see the next test)."""
    dev = torch.device("cuda", 0)
    w72, w7 = W.WORKLOADS["llava72b"], W.WORKLOADS["llava7b"]
    if first == "nine-tiles":
        a_in = W.random_verify_inputs(1, 17, 64, 8, 128, [20000], "bf16", seed=5)
    else:
        a_in = W.make_verify_inputs(w72, layer=1)
    b_in = W.make_verify_inputs(w7, layer=1)
    A = [to_dev(x) for x in (a_in.q, a_in.k, a_in.v, a_in.ctx_len)]
    Bt = [to_dev(x) for x in (b_in.q, b_in.k, b_in.v, b_in.ctx_len)]
    rng = np.random.default_rng(3)
    Vv, g = 152064, 5
    dl = torch.from_numpy(rng.standard_normal((1, g, Vv)).astype(np.float32)).to(dev)
    tl = torch.from_numpy(rng.standard_normal((1, g + 1, Vv)).astype(np.float32)).to(dev)
    tok = torch.from_numpy(rng.integers(0, Vv, (1, g)).astype(np.int32)).to(dev)
    ua = torch.from_numpy(rng.random((1, g))).to(dev)
    us = torch.from_numpy(rng.random(1)).to(dev)
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    pv.set_stream_cu_budget(s1, budgets[0])
    pv.set_stream_cu_budget(s2, budgets[1])
    ws1, ws2 = pv.Workspace(dev), pv.Workspace(dev)
    st1 = torch.zeros(1, dtype=torch.int32, device=dev)
    st2 = torch.zeros(1, dtype=torch.int32, device=dev)

    def run1():
        return pv.verify_attn(*A, ws=ws1, status=st1)

    def run2():
        o = pv.verify_attn(*Bt, ws=ws2, status=st2)
        n, y, _ = pv.spec_accept(dl, tl, tok, ua, us, 1.0, ws=ws2, status=st2)
        return o + (n, y)

    note(f"budgets {budgets}: each stream alone")
    with torch.cuda.stream(s1):
        r1 = [t.clone() for t in run1()]
    torch.cuda.synchronize()
    with torch.cuda.stream(s2):
        r2 = [t.clone() for t in run2()]
    torch.cuda.synchronize()
    assert int(st1.item()) == 0 and int(st2.item()) == 0
    if first == "nine-tiles":
        ro, rl, rm = oracle.verify_attn(f64(a_in.q, "bf16"), f64(a_in.k, "bf16"), f64(a_in.v, "bf16"),
                                        a_in.ctx_len, a_in.scale)
        assert_out(to_host_f64(r1[0]), ro)
        assert_mass(to_host_f64(r1[1]), rm, 64, 17)
    for rep in range(5):
        note(f"budgets {budgets}: both streams together, round {rep}")
        with torch.cuda.stream(s1):
            x1 = run1()
        with torch.cuda.stream(s2):
            x2 = run2()
        torch.cuda.synchronize()
        assert int(st1.item()) == 0 and int(st2.item()) == 0
        assert all(torch.equal(a, b) for a, b in zip(x1, r1))
        assert all(torch.equal(a, b) for a, b in zip(x2, r2))
    pv.set_stream_cu_budget(s1, 0)
    pv.set_stream_cu_budget(s2, 0)


@pytest.mark.parametrize("budgets,ctx", [((224, 32), (12000, 3500)), ((128, 128), (7000, 6432))])
def test_two_budgeted_streams_replay_waiting_graphs_together(budgets, ctx):
    """A 72B layer's verify with mass captured on one budgeted stream and a 7B
    layer's on another, both in the waiting form, replayed together: every
    replay equals the eager call, no wait gives up, and the statistics records
    are 0 again afterwards."""
    dev = torch.device("cuda", 0)
    runs = []
    for (T, hq, hkv), budget, n in zip(((9, 64, 8), (6, 28, 4)), budgets, ctx):
        inp = W.random_verify_inputs(1, T, hq, hkv, 128, [n], "bf16", seed=n)
        args = [to_dev(x) for x in (inp.q, inp.k, inp.v, inp.ctx_len)]
        s, ws = torch.cuda.Stream(), pv.Workspace(dev)
        status = torch.zeros(1, dtype=torch.int32, device=dev)
        pv.set_stream_cu_budget(s, budget)
        torch.cuda.synchronize()
        note(f"waiting graph: budget {budget}, {hq}/{hkv} heads, ctx {n}")
        with torch.cuda.stream(s):
            ref = [t.clone() for t in pv.verify_attn(*args, scale=inp.scale, max_ctx=n, ws=ws, status=status)]
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph(keep_graph=True)
        with torch.cuda.graph(g, stream=s):
            outs = pv.verify_attn(*args, scale=inp.scale, max_ctx=n, ws=ws, status=status)
        assert _kernels(g) == WAITING
        g.instantiate()
        with torch.cuda.stream(s):
            g.replay()
        torch.cuda.synchronize()
        assert int(status.item()) == 0
        assert all(torch.equal(a, b) for a, b in zip(outs, ref))
        runs.append((s, g, outs, ref, status, ws, args))
    for rep in range(20):
        note(f"waiting graphs on budgets {budgets} together, round {rep}")
        for s, g, *_ in runs * 3:
            with torch.cuda.stream(s):
                g.replay()
        torch.cuda.synchronize()
        for _, _, outs, ref, status, ws, _ in runs:
            assert int(status.item()) == 0
            assert all(torch.equal(a, b) for a, b in zip(outs, ref))
            assert not ws.buf[256 * 1024:768 * 1024].any()
    for s, *_ in runs:
        pv.set_stream_cu_budget(s, 0)
