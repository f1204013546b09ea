"""The calls whose speed this library is about, as a serving program makes them.

Five kinds of case, each one step of ParallelVLM's verify + prune path:

* ``decode``   rotary embedding and append of the new rows, then verify
               attention with its attention mass, layer after layer: the
               target's verify forward (T = gamma + 1 rows) or the draft's
               decode step (T = 1).  Several layers are one HIP graph, which a
               serving loop captures once and replays for every step; a single
               layer is called eagerly.
* ``prune``    UV-Prune's MASS score with its top-k, then the gather of the
               kept rows of every layer into the draft's compact cache.
* ``accept``   speculative accept/reject with the residual or bonus draw.
* ``cossim``   UV-Prune's score from the hidden states of two layers.
* ``epilogue`` a prefill layer's residual add with the criterion fused in.

Shapes are those of ``workloads`` (LLaVA-OV 7B and 72B, Qwen2.5-VL-32B, the
131K-token video and the small fp32 configuration); ``draw`` spreads over the
ranges around them.  ``prepare`` makes seeded inputs with the workloads'
structure (normal draws, a share of salient keys, draft logits plus noise).
"""
import math
import random

import torch

import paper_2603_19610_amd as pv

BF16, F32 = "bf16", "f32"


# ------------------------------------------------------------------ cases --
def _decode(name, dtype, layers, B, T, hq, hkv, D, ctx_lo, ctx_hi, page=0, spare=0, mass=True,
            mrope=False):
    c = dict(kind="decode", dtype=dtype, layers=layers, B=B, T=T, hq=hq, hkv=hkv, D=D,
             ctx_lo=ctx_lo, ctx_hi=ctx_hi, page=page, spare=spare, mass=mass, mrope=mrope)
    return dict(c, name=name) if name else c


def _prune(name, layers, B, hkv, D, m_lo, m_hi, n, keep_num, keep_den, crit=21):
    c = dict(kind="prune", layers=layers, B=B, hkv=hkv, D=D, m_lo=m_lo, m_hi=m_hi, n=n,
             keep_num=keep_num, keep_den=keep_den, crit=crit)
    return dict(c, name=name) if name else c


def _accept(name, B, gamma, V, temperature):
    c = dict(kind="accept", B=B, gamma=gamma, V=V, temperature=temperature)
    return dict(c, name=name) if name else c


def _hidden(name, kind, dtype, B, m, n, dh):
    c = dict(kind=kind, dtype=dtype, B=B, m=m, n=n, dh=dh)
    return dict(c, name=name) if name else c


def listed():
    return [
        # The small fp32 configuration, one layer, called eagerly: the smallest
        # call, where launches and latency are everything.
        _decode("decode-tiny-f32", F32, 1, 1, 5, 4, 1, 64, 1024, 1024),
        # The 7B draft's decode step over its compact cache (a tenth of the
        # visual rows and the text): short caches, one new row, no mass.
        _decode("decode-draft-7b", BF16, 28, 1, 1, 28, 4, 128, 787, 787, mass=False),
        # The 7B target's verify forward, 32 frames, gamma = 5.
        _decode("decode-7b", BF16, 28, 1, 6, 28, 4, 128, 6432, 6432),
        # The headline: the 72B target's verify forward, 64 frames, gamma = 8.
        _decode("decode-72b", BF16, 80, 1, 9, 64, 8, 128, 12800, 12800),
        # A ragged batch over a paged cache with M-RoPE, one Qwen-32B layer.
        _decode("decode-32b-paged", BF16, 1, 4, 9, 40, 8, 128, 16384, 33280, page=32, mrope=True),
        # One layer over a 131K-token video, gamma = 16: the longest context.
        _decode("decode-long", BF16, 1, 1, 17, 64, 8, 128, 132096, 132096, spare=37),
        # The hand-over to the draft at the 72B shape: score, top-k, and the
        # gather of all 80 layers.
        _prune("prune-72b", 80, 1, 8, 128, 12544, 12544, 256, 1, 10),
        # Selection over a 131K-row video with one layer's gather.
        _prune("prune-long", 1, 1, 8, 128, 131072, 131072, 1024, 3, 100),
        # Accept/reject of eight drafts over the full vocabulary, one sequence.
        _accept("accept-72b", 1, 8, 152064, 1.0),
        # The same for a batch of four.
        _accept("accept-batch4", 4, 8, 152064, 0.7),
        # UV-Prune's own criterion at the 72B hidden size (layers 0 and L).
        _hidden("cossim-72b", "cossim", BF16, 1, 12544, 256, 8192),
        # A 7B prefill layer's epilogue.
        _hidden("epilogue-7b", "epilogue", BF16, 1, 6272, 160, 3584),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["decode"] * 5 + ["prune", "prune", "accept", "accept", "cossim",
                                        "epilogue"])
    if kind == "decode":
        f32 = rng.random() < 0.2
        B = rng.choice([1, 1, 2, 3, 4])
        hkv = rng.choice([1, 2, 4, 8])
        group = rng.choice([1, 4, 5, 7, 8])
        D = rng.choice([64, 128, 128])
        T = rng.choice([1, 1, rng.randint(2, 9), rng.randint(2, 17)])
        hi = _log(rng, 300, 8000 if f32 else 120000 // B)
        lo = hi if B == 1 else max(64, int(hi * rng.uniform(0.4, 1.0)))
        layers = 1
        if rng.random() < 0.5:
            # keep the whole stack within 2 GB of cache
            layers = max(1, min(rng.randint(2, 32), 2 ** 31 // (4 * B * hi * hkv * D)))
            layers = min(layers, 8) if f32 else layers
        page = 0 if f32 or rng.random() < 0.6 else rng.choice([32, 64, 256])
        return _decode(None, F32 if f32 else BF16, layers, B, T, group * hkv, hkv, D, lo, hi,
                       page=page, spare=rng.choice([0, rng.randint(1, 200)]),
                       mass=rng.random() < 0.8, mrope=D == 128 and rng.random() < 0.3)
    if kind == "prune":
        B = rng.choice([1, 1, 2, 4])
        hi = _log(rng, 700, 131072)
        lo = hi if B == 1 else max(64, int(hi * rng.uniform(0.4, 1.0)))
        hkv = rng.choice([2, 4, 8])
        layers = max(1, min(rng.choice([1, 28, 64, 80]), 2 ** 31 // (4 * B * hi * hkv * 128)))
        return _prune(None, layers, B, hkv, 128, lo, hi, rng.randint(16, 1024),
                      rng.randint(1, 50), 100)
    if kind == "accept":
        return _accept(None, rng.randint(1, 8), rng.randint(1, 16), _log(rng, 1024, 152064),
                       rng.choice([0.0, 0.5, 0.7, 1.0, 1.0]))
    B = rng.choice([1, 1, 2])
    dh = 8 * rng.randint(64, 1024)
    return _hidden(None, kind, rng.choice([BF16, BF16, F32]), B, _log(rng, 500, 14000 // B),
                   rng.randint(8, 512), dh)


# ----------------------------------------------------------------- inputs --
def _torch_dtype(case):
    return torch.bfloat16 if case["dtype"] == BF16 else torch.float32


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(1000003 * int(seed) + 17)
    return g


def _lengths(lo, hi, B):
    """Lengths of a ragged batch: the longest is hi, the others between."""
    r = random.Random(7919 * lo + 31 * hi + B)
    return [hi] + [r.randint(lo, hi) for _ in range(B - 1)]


def _i32(values):
    return torch.tensor(values, dtype=torch.int32, device="cuda")


def _rotate(x, pos, base, sections):
    """Rotate-half RoPE in float64; x [B][T][H][D], pos [B][T] or [3][B][T]."""
    D = x.shape[-1]
    h = D // 2
    theta = base ** (-2.0 * torch.arange(h, dtype=torch.float64, device=x.device) / D)
    if sections is None:
        p = pos.double()[..., None].expand(*pos.shape, h)
    else:
        axis = torch.repeat_interleave(torch.arange(3, device=x.device),
                                       torch.tensor(sections, device=x.device))
        p = pos.double()[axis].permute(1, 2, 0)
    ang = (p * theta)[:, :, None, :]
    c, s = torch.cos(ang), torch.sin(ang)
    a, b = x.double()[..., :h], x.double()[..., h:]
    return torch.cat([a * c - b * s, a * s + b * c], dim=-1)


_BASE = 1.0e6


def _decode_inputs(case, seed):
    g, dt = _gen(seed), _torch_dtype(case)
    L, B, T, hq, hkv, D = (case[k] for k in ("layers", "B", "T", "hq", "hkv", "D"))
    lens = _lengths(case["ctx_lo"], case["ctx_hi"], B)
    ctx = _i32(lens)
    n_cap = max(lens) + T + case["spare"]

    def randn(*shape):
        return torch.randn(shape, dtype=dt, device="cuda", generator=g)

    q, k_new, v_new = randn(L, B, T, hq, D), randn(L, B, T, hkv, D), randn(L, B, T, hkv, D)
    pos = ctx[:, None] + torch.arange(T, dtype=torch.int32, device="cuda")[None]
    sections = (D // 8, D // 4 - D // 16, D // 4 - D // 16) if case["mrope"] else None
    if sections is not None:
        pos = torch.stack([pos, pos, pos]).contiguous()
    k, v = randn(L, B, hkv, n_cap, D), randn(L, B, hkv, n_cap, D)
    # one key in fifty is salient: it gains 3 along its group's mean query
    for layer in range(L):
        mean_q = _rotate(q[layer], pos, _BASE, sections).view(B, T, hkv, hq // hkv, D)
        mean_q = mean_q.mean(dim=(1, 3))
        mean_q = (3.0 * mean_q / mean_q.norm(dim=-1, keepdim=True)).to(dt)
        rows = torch.randint(0, min(lens), (max(1, min(lens) // 50),), device="cuda",
                             generator=g).unique()
        k[layer][:, :, rows] += mean_q[:, :, None, :]
    s = dict(q=q, k_new=k_new, v_new=v_new, pos=pos, ctx=ctx, sections=sections, lens=lens,
             max_ctx=max(lens))
    if case["page"]:
        P = case["page"]
        mp = -(-n_cap // P)
        need = [-(-(n + T) // P) for n in lens]
        n_pages = sum(need) + 3
        perm = torch.randperm(n_pages, device="cuda", generator=g)
        table = torch.full((B, mp), -1, dtype=torch.int32, device="cuda")
        pools = []
        for cache in (k, v):
            pad = torch.zeros((L, B, hkv, mp * P, D), dtype=dt, device="cuda")
            pad[..., :n_cap, :] = cache
            blocks = pad.view(L, B, hkv, mp, P, D).transpose(2, 3).contiguous()
            pool = torch.zeros((L, n_pages, hkv, P, D), dtype=dt, device="cuda")
            o = 0
            for b in range(B):
                pages = perm[o:o + need[b]]
                table[b, :need[b]] = pages.to(torch.int32)
                pool[:, pages] = blocks[:, b, :need[b]]
                o += need[b]
            pools.append(pool)
        k, v = pools
        s["table"] = table
        s["n_cap"] = mp * P
    else:
        s["n_cap"] = n_cap
    s["k"], s["v"] = k, v
    return s


def _decode_layers(s):
    for layer in range(s["q"].shape[0]):
        mass = None if s["mass"] is None else s["mass"][layer]
        kw = dict(out=s["out"][layer], lse=s["lse"][layer], mass=mass)
        q_rot, k, v = s["q_rot"][layer], s["k"][layer], s["v"][layer]
        rows = (s["q"][layer], s["k_new"][layer], s["v_new"][layer], s["pos"], s["ctx"], k, v)
        if "table" in s:
            pv.rope_append_paged(*rows, s["table"], base=_BASE, sections=s["sections"],
                                 q_out=q_rot)
            pv.verify_attn_paged(q_rot, k, v, s["table"], s["ctx"], max_ctx=s["max_ctx"],
                                 want_mass=mass is not None, ws=s["ws"], **kw)
        else:
            pv.rope_append(*rows, base=_BASE, sections=s["sections"], q_out=q_rot)
            pv.verify_attn(q_rot, k, v, s["ctx"], max_ctx=s["max_ctx"],
                           want_mass=mass is not None, ws=s["ws"], **kw)


def _prepare_decode(case, seed):
    s = _decode_inputs(case, seed)
    L, B, T, hq = (case[k] for k in ("layers", "B", "T", "hq"))
    s["q_rot"], s["out"] = torch.empty_like(s["q"]), torch.empty_like(s["q"])
    s["lse"] = torch.empty((L, B, hq, T), dtype=torch.float32, device="cuda")
    s["mass"] = (torch.empty((L, B, s["n_cap"]), dtype=torch.float32, device="cuda")
                 if case["mass"] else None)
    s["ws"] = pv.Workspace()
    s["ws"].get(pv.verify_attn_workspace_size(
        pv.PVLM_BF16 if case["dtype"] == BF16 else pv.PVLM_F32, B, T, hq, case["hkv"], case["D"],
        s["n_cap"], s["max_ctx"]))
    pv.default_status()
    if L > 1:
        torch.cuda.synchronize()
        s["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(s["graph"]):
            _decode_layers(s)
    return s


def _prepare_prune(case, seed):
    g = _gen(seed)
    L, B, hkv, D, n = (case[k] for k in ("layers", "B", "hkv", "D", "n"))
    m = _lengths(case["m_lo"], case["m_hi"], B)
    m_cap = max(m)
    # masses: softmax-like positive values, a share of them raised with depth
    crit = torch.rand((case["crit"], B, m_cap), device="cuda", generator=g).pow(-0.5).mul_(0.02)
    rows = torch.randint(0, m_cap, (max(1, m_cap // 50),), device="cuda", generator=g)
    crit[-1][:, rows] *= 8.0
    keep = [x * case["keep_num"] // case["keep_den"] for x in m]
    shape = (L, B, hkv, m_cap + n, D)
    return dict(crit=crit, m=_i32(m), k=_i32(keep), k_cap=max(keep), tail=_i32([n] * B),
                keys=torch.randn(shape, dtype=torch.bfloat16, device="cuda", generator=g),
                values=torch.randn(shape, dtype=torch.bfloat16, device="cuda", generator=g),
                score=torch.empty((B, m_cap), dtype=torch.float32, device="cuda"),
                idx=torch.empty((B, max(keep)), dtype=torch.int32, device="cuda"),
                k_dst=torch.zeros((L, B, hkv, max(keep) + n, D), dtype=torch.bfloat16,
                                  device="cuda"),
                v_dst=torch.zeros((L, B, hkv, max(keep) + n, D), dtype=torch.bfloat16,
                                  device="cuda"))


def _prepare_accept(case, seed):
    g = _gen(seed)
    B, gamma, V, tau = (case[k] for k in ("B", "gamma", "V", "temperature"))
    z = torch.randn((B, gamma + 1, V), device="cuda", generator=g) * 2.0
    target = z + torch.randn((B, gamma + 1, V), device="cuda", generator=g) * 0.5
    draft = z[:, :gamma].contiguous()
    if tau == 0.0:
        tokens = draft.argmax(dim=-1)
    else:
        u = torch.rand(draft.shape, device="cuda", generator=g).clamp_min(1e-30)
        tokens = (draft / tau - torch.log(-torch.log(u))).argmax(dim=-1)
    return dict(draft=draft, target=target, tokens=tokens.to(torch.int32), tau=tau,
                u_accept=torch.rand((B, gamma), dtype=torch.float64, device="cuda", generator=g),
                u_sample=torch.rand((B,), dtype=torch.float64, device="cuda", generator=g))


def _prepare_cossim(case, seed):
    g, dt = _gen(seed), _torch_dtype(case)
    B, m, n, dh = (case[k] for k in ("B", "m", "n", "dh"))
    hv = torch.randn((2, B, m, dh), dtype=dt, device="cuda", generator=g)
    ht = torch.randn((2, B, n, dh), dtype=dt, device="cuda", generator=g)
    u = ht[1].float().mean(dim=1, keepdim=True)
    rows = torch.randint(0, m, (max(1, m // 50),), device="cuda", generator=g).unique()
    hv[1][:, rows] += (3.0 * u / u.norm(dim=-1, keepdim=True)).to(dt)
    return dict(hv=hv, ht=ht, m=_i32([m] * B), n=_i32([n] * B))


def _prepare_epilogue(case, seed):
    g, dt = _gen(seed), _torch_dtype(case)
    B, m, n, dh = (case[k] for k in ("B", "m", "n", "dh"))

    def randn(rows, scale):
        return torch.randn((B, rows, dh), dtype=dt, device="cuda", generator=g) * scale

    s = dict(vis=randn(m, 1.0), vis_delta=randn(m, 0.25), txt=randn(n, 1.0),
             txt_delta=randn(n, 0.25), m=_i32([m] * B), n=_i32([n] * B))
    s["vis_out"], s["txt_out"] = torch.empty_like(s["vis"]), torch.empty_like(s["txt"])
    return s


def prepare(case, seed):
    s = {"decode": _prepare_decode, "prune": _prepare_prune, "accept": _prepare_accept,
         "cossim": _prepare_cossim, "epilogue": _prepare_epilogue}[case["kind"]](case, seed)
    s["kind"] = case["kind"]
    return s


def run(s):
    kind = s["kind"]
    if kind == "decode":
        if "graph" in s:
            s["graph"].replay()
        else:
            _decode_layers(s)
        r = dict(out=s["out"], lse=s["lse"], q_rot=s["q_rot"], k=s["k"], v=s["v"])
        if s["mass"] is not None:
            r["mass"] = s["mass"]
        return r
    if kind == "prune":
        score, idx = pv.uvprune_topk_mass(s["crit"], s["m"], s["k"], s["k_cap"],
                                          score=s["score"], idx=s["idx"])
        k, v = pv.gather_kv(s["keys"], s["values"], idx, s["k"], s["m"], s["tail"],
                            s["k_dst"].shape[-2], k_dst=s["k_dst"], v_dst=s["v_dst"])
        return dict(score=score, idx=idx, k=k, v=v)
    if kind == "accept":
        n, token, tie = pv.spec_accept(s["draft"], s["target"], s["tokens"], s["u_accept"],
                                       s["u_sample"], s["tau"])
        return dict(n_accepted=n, next_token=token, near_tie=tie)
    if kind == "cossim":
        return dict(score=pv.uvprune_score_cossim(s["hv"], s["ht"], s["m"], s["n"]))
    vis, txt, crit = pv.prefill_epilogue_cossim(s["vis"], s["vis_delta"], s["txt"],
                                                s["txt_delta"], s["m"], s["n"],
                                                vis_out=s["vis_out"], txt_out=s["txt_out"])
    return dict(vis=vis, txt=txt, crit=crit)


# ------------------------------------------------------- work and accuracy --
def work(case):
    kind = case["kind"]
    if kind == "decode":
        L, B, T, hq, hkv, D = (case[k] for k in ("layers", "B", "T", "hq", "hkv", "D"))
        e = 2 if case["dtype"] == BF16 else 4
        rows = sum(n + T for n in _lengths(case["ctx_lo"], case["ctx_hi"], B))
        # K and V of every visible row; q and the new rows in; out, lse, mass out
        size = 2 * rows * hkv * D * e + B * T * (2 * hq + 2 * hkv) * D * e + 4 * B * hq * T
        size += 4 * rows if case["mass"] else 0
        return dict(bytes=L * size, flops=L * 4 * rows * hq * T * D)
    if kind == "prune":
        m = _lengths(case["m_lo"], case["m_hi"], case["B"])
        kept = sum(x * case["keep_num"] // case["keep_den"] for x in m)
        moved = kept + case["B"] * case["n"]
        return dict(bytes=12 * sum(m) + 4 * kept
                    + 8 * case["layers"] * case["hkv"] * case["D"] * moved, flops=sum(m))
    if kind == "accept":
        entries = case["B"] * (2 * case["gamma"] + 1) * case["V"]
        return dict(bytes=4 * entries, flops=3 * entries)
    e = 2 if case["dtype"] == BF16 else 4
    values = case["B"] * (case["m"] + case["n"]) * case["dh"]
    if kind == "cossim":
        return dict(bytes=2 * values * e + 4 * case["B"] * case["m"], flops=2 * 4 * values)
    return dict(bytes=3 * values * e + 4 * case["B"] * case["m"], flops=5 * values)


def tolerance(case):
    kind, bf16 = case["kind"], case.get("dtype") == BF16
    if kind == "decode":
        # bf16 probabilities and partial sums; fp32 sums over the context
        return dict(rel=1e-2, max=0.1) if bf16 else dict(rel=1e-5, max=4e-4)
    if kind in ("prune", "accept"):
        return "exact"  # one fp32 subtraction, indices, copies, float64 decisions
    if kind == "epilogue" and bf16:
        return dict(rel=1e-3, max=2e-2)  # one rounding of each sum
    return dict(rel=1e-5, max=4e-4)  # float64 sums, fp32 results


def _exact_decode(case, seed):
    s = _decode_inputs(case, seed)
    L, B, T, hq, hkv, D = (case[k] for k in ("layers", "B", "T", "hq", "hkv", "D"))
    G = hq // hkv
    dt = s["q"].dtype
    f64 = dict(dtype=torch.float64, device="cuda")
    out, lse = torch.zeros((L, B, T, hq, D), **f64), torch.zeros((L, B, hq, T), **f64)
    q_all = torch.zeros((L, B, T, hq, D), **f64)
    mass = torch.zeros((L, B, s["n_cap"]), **f64)
    for layer in range(L):
        # the call stores rotated rows in the storage type, and attends over those
        q_all[layer] = _rotate(s["q"][layer], s["pos"], _BASE, s["sections"])
        q = q_all[layer].to(dt).double()
        k_new = _rotate(s["k_new"][layer], s["pos"], _BASE, s["sections"]).to(dt).double()
        for b in range(B):
            n = s["lens"][b]
            for h in range(hkv):
                if "table" in s:
                    P = case["page"]
                    pages = s["table"][b, :-(-(n + T) // P)].long()
                    K = s["k"][layer][pages, h].reshape(-1, D)[:n]
                    V = s["v"][layer][pages, h].reshape(-1, D)[:n]
                else:
                    K, V = s["k"][layer, b, h, :n], s["v"][layer, b, h, :n]
                K = torch.cat([K.double(), k_new[b, :, h]])
                V = torch.cat([V.double(), s["v_new"][layer, b, :, h].double()])
                x = q[b, :, h * G:(h + 1) * G].reshape(T * G, D) @ K.t() * D ** -0.5
                hidden = (torch.arange(n + T, device="cuda")[None]
                          > n + torch.arange(T, device="cuda").repeat_interleave(G)[:, None])
                x.masked_fill_(hidden, -math.inf)
                z = torch.logsumexp(x, dim=-1, keepdim=True)
                p = torch.exp(x - z)
                out[layer, b, :, h * G:(h + 1) * G] = (p @ V).view(T, G, D)
                lse[layer, b, h * G:(h + 1) * G] = z.view(T, G).t()
                mass[layer, b, :n + T] += p.sum(dim=0)
    r = dict(out=out, lse=lse, q_rot=q_all, k=None, v=None)
    if case["mass"]:
        r["mass"] = mass
    return r


def exact(case, seed):
    kind = case["kind"]
    if kind == "decode":
        return _exact_decode(case, seed)
    if kind == "prune":  # the score only: the rest are indices and copied rows
        s = _prepare_prune(case, seed)
        d = s["crit"][-1].double() - s["crit"][0].double()
        live = torch.arange(d.shape[1], device="cuda")[None] < s["m"][:, None]
        return dict(score=torch.where(live, d, 0.0), idx=None, k=None, v=None)
    if kind == "accept":  # whole numbers only
        return None

    def criterion(hv, ht):
        u = (ht / ht.norm(dim=-1, keepdim=True)).sum(dim=1)
        return (hv @ u[:, :, None])[..., 0] / hv.norm(dim=-1)

    if kind == "cossim":
        s = _prepare_cossim(case, seed)
        c0, c1 = (criterion(s["hv"][i].double(), s["ht"][i].double()) for i in (0, 1))
        return dict(score=c1 - c0)
    s = _prepare_epilogue(case, seed)
    vis, txt = s["vis"].double() + s["vis_delta"].double(), s["txt"].double() + s["txt_delta"].double()
    # the criterion is that of the stored rows
    crit = criterion(vis.to(s["vis"].dtype).double(), txt.to(s["vis"].dtype).double())
    return dict(vis=vis, txt=txt, crit=crit)
