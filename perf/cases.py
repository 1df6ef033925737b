"""The work that programs have this framework do, as cases that can be timed and compared.

A case is one call of a public entry point of ``paper_2602_07265_amd.xshare`` on the shapes of
the layers that this repository's benchmark and tests use (Mixtral-, Qwen-MoE- and
DeepSeek-R1-shaped, and sizes of no particular model), over the batch sizes that the library
takes: one token, ordinary decode batches, speculative batches, and prefill chunks up to the
limit of 8192 (token, expert) pairs; in each weight format; flat, per-request and GPU-group
selection.  Inputs follow the repository's workload recipe: logits of a few domain centroids
N(0, 1.5) plus token noise N(0, 0.5) (speculative batches: per-request offsets N(0, 1) and
token noise N(0, 0.3)), x ~ N(0, 1), weights ~ N(0, 0.02), quantized per row (FP8) or per
block of 32 (MXFP4) where the case says so.
"""
import math

import numpy as np
import torch

from paper_2602_07265_amd import xshare as X

SHAPES = {
    "mixtral": dict(N=8, k=2, d=4096, f=14336, Q=4),
    "qwen": dict(N=128, k=8, d=2048, f=768, Q=8),
    "ds": dict(N=256, k=8, d=7168, f=2048, Q=8),
}


def _case(shape, T, M, op="forward", fmt="bf16", **more):
    c = dict(op=op, fmt=fmt, T=T, M=M, k0=1, score="topk", reqs=0, m_r=0, groups=0, local=-1,
             shared=0, **SHAPES[shape])
    c.update(more)
    return c


def listed():
    return [
        # selection alone, for a program with expert kernels of its own: the smallest call
        dict(_case("ds", 16, 48, op="route"), name="route_t16"),
        # one user's decode step through a small layer: launches and latency
        dict(_case("qwen", 1, 8), name="qwen_t1_bf16"),
        # a large decode batch over small experts in the narrowest weights
        dict(_case("qwen", 256, 64, fmt="mxfp4"), name="qwen_t256_mxfp4"),
        # the benchmark's own workload: an ordinary decode batch
        dict(_case("ds", 32, 48), name="ds_t32_bf16"),
        # a small decode batch in FP8 weights
        dict(_case("ds", 8, 24, fmt="fp8"), name="ds_t8_fp8"),
        # a speculative verify batch, 16 requests of 4 tokens, per-request selection
        dict(_case("ds", 64, 64, reqs=16, m_r=4, Q=4), name="ds_spec_16x4_bf16"),
        # a decode batch over few, large experts
        dict(_case("mixtral", 16, 5), name="mixtral_t16_bf16"),
        # the whole layer from hidden states, with its router and shared expert
        dict(_case("ds", 32, 48, op="layer", shared=1), name="ds_layer_t32_bf16"),
        # one GPU's share of an expert-parallel layer, eight groups of at most eight experts
        dict(_case("ds", 128, 8, fmt="fp8", groups=8, local=3), name="ds_ep_t128_fp8"),
        # sizes that divide by nothing but 32, an odd batch
        dict(_case("qwen", 37, 30, N=60, k=6, d=2720, f=1376, Q=5), name="ragged_t37_bf16"),
        # a prefill chunk over few, large experts: hundreds of rows an expert
        dict(_case("mixtral", 1024, 8), name="mixtral_t1024_bf16"),
        # a prefill chunk of the large layer: the largest call
        dict(_case("ds", 512, 96), name="ds_t512_bf16"),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _cost(c):
    w = work(c)
    return max(w["bytes"], w["flops"] / 200)


def draw(rng):
    """One more case: a shape, weight format, selection and batch size of the same ranges."""
    most = _cost(listed()[-1])
    while True:
        op = rng.choice(["forward"] * 7 + ["layer"] * 2 + ["route"])
        shape = rng.choice(["mixtral", "qwen", "ds", "other", "other"])
        fmt = rng.choice(["bf16", "bf16", "fp8", "mxfp4"])
        kind = rng.choice(["flat"] * 4 + ["spec", "ep"])
        more = {}
        if shape == "other":
            N = rng.randint(8, 160)
            more = dict(N=N, k=rng.randint(1, min(8, N)), d=32 * rng.randint(8, 128),
                        f=32 * rng.randint(4, 96), Q=rng.randint(2, 8))
        s = dict(SHAPES.get(shape, {}), **more)
        N, k = s["N"], s["k"]
        T = _log_uniform(rng, 1, min(1024, 8192 // k))
        M = max(k, _log_uniform(rng, k, min(N, 96)))
        if op == "layer":
            fmt = "bf16"
            more["shared"] = rng.randint(0, 2)
        if rng.random() < 0.1:
            more["score"] = "dense"
        if kind == "spec" and op != "route":
            L = rng.randint(2, 5)
            R = max(1, min(T, 160) // L)
            T = R * L
            more.update(reqs=R, m_r=rng.randint(1, 4))
        if kind == "ep" and op == "forward" and N % 8 == 0 and N >= 32:
            M = rng.randint(2, max(2, N // 16))
            more.update(groups=8, local=rng.randint(0, 7))
        c = _case("qwen" if shape == "other" else shape, T, M, op=op, fmt=fmt, **more)
        if c not in [dict((a, b) for a, b in x.items() if a != "name") for x in listed()] \
                and _cost(c) <= most:
            return c


# ---------------------------------------------------------------------------- inputs

def _gen(seed, what, dev="cuda"):
    g = torch.Generator(device=dev)
    g.manual_seed(int(seed) * 1000003 + what)
    return g


def _logits(c, seed, dev="cuda"):
    g = _gen(seed, 1, dev)
    n = lambda *s: torch.randn(*s, generator=g, device=dev, dtype=torch.float32)  # noqa: E731
    T, N, Q = c["T"], c["N"], c["Q"]
    cent = 1.5 * n(Q, N)
    if c["reqs"]:
        R = c["reqs"]
        dom = torch.arange(R, device=dev) % Q
        h = cent[dom][:, None, :] + n(R, 1, N) + 0.3 * n(R, T // R, N)
        return h.reshape(T, N).contiguous()
    dom = torch.randint(0, Q, (T,), generator=g, device=dev)
    return cent[dom] + 0.5 * n(T, N)


def _x(c, seed):
    g = _gen(seed, 2)
    n = lambda *s: torch.randn(*s, generator=g, device="cuda", dtype=torch.float32)  # noqa: E731
    T, d, Q = c["T"], c["d"], c["Q"]
    if c["op"] == "layer":     # hidden states carry the domains: the router sees them
        dom = torch.randint(0, Q, (T,), generator=g, device="cuda")
        return (n(Q, d)[dom] + 0.5 * n(T, d)).to(torch.bfloat16)
    return n(T, d).to(torch.bfloat16)


def _router(c, seed):
    w = torch.empty((c["N"], c["d"]), dtype=torch.bfloat16, device="cuda")
    return w.normal_(0.0, 1.5 / math.sqrt(c["d"]), generator=_gen(seed, 3))


def _quant_fp8(w):
    """[n, rows, cols] -> E4M3FN codes and one fp32 scale a row."""
    v = w.float()
    s = v.abs().amax(dim=2) / 448.0
    return (v / s[:, :, None]).clamp(-448, 448).to(torch.float8_e4m3fn).view(torch.uint8), s


def _quant_mx(w):
    """[n, rows, cols] -> packed E2M1 codes and E8M0 scales (row-major), blocks of 32."""
    v = w.float()
    n, r, cols = v.shape
    b = v.view(n, r, cols // 32, 32)
    ex = torch.frexp(b.abs().amax(dim=3)).exponent - 3
    a = torch.ldexp(b.abs(), -ex[..., None]).clamp(max=6.0)
    step = torch.where(a < 2.0, 0.5, torch.where(a < 4.0, 1.0, 2.0))
    q = torch.round(a / step) * step
    code = torch.where(q < 2.0, q * 2.0, torch.where(q < 4.0, q + 2.0, q / 2.0 + 4.0))
    code = code.to(torch.uint8) | ((b < 0).to(torch.uint8) << 3)
    code = code.view(n, r, cols)
    return (code[..., 0::2] | (code[..., 1::2] << 4)).contiguous(), (ex + 127).to(torch.uint8)


def _weights(c, seed, count, what, fmt):
    """The three weight arrays of `count` experts and their scales (None for bf16), w2 last."""
    d, f = c["d"], c["f"]
    ws, ss = [], []
    for m, (rows, cols) in enumerate(((f, d), (f, d), (d, f))):
        g = _gen(seed, what + m)
        if fmt == "bf16":
            w = torch.empty((count, rows, cols), dtype=torch.bfloat16, device="cuda")
            for e in range(0, count, 16):
                w[e:e + 16].normal_(0.0, 0.02, generator=g)
            ws.append(w)
            ss.append(None)
            continue
        div, quant = (1, _quant_fp8) if fmt == "fp8" else (2, _quant_mx)
        w = torch.empty((count, rows, cols // div), dtype=torch.uint8, device="cuda")
        s = (torch.empty((count, rows), dtype=torch.float32, device="cuda") if fmt == "fp8" else
             torch.empty((count, rows, cols // 32), dtype=torch.uint8, device="cuda"))
        part = max(1, (1 << 26) // (rows * cols))
        for e in range(0, count, part):
            n = min(part, count - e)
            v = torch.empty((n, rows, cols), dtype=torch.bfloat16, device="cuda")
            w[e:e + n], s[e:e + n] = quant(v.normal_(0.0, 0.02, generator=g))
        ws.append(w)
        ss.append(s)
    return ws, ss


def prepare(case, seed):
    c = case
    s = {"case": c, "opts": {}, "ws": None}
    if c["op"] == "layer":
        s["gate"] = _router(c, seed)
    else:
        s["logits"] = _logits(c, seed)
    offsets = None
    if c["reqs"]:
        step = c["T"] // c["reqs"]
        offsets = torch.arange(0, c["T"] + 1, step, dtype=torch.int32, device="cuda")
        s["opts"] = dict(req_offsets=offsets, per_request_budget=c["m_r"])
    p = X.params(c["N"], c["k"], c["k0"], c["M"], "per_group" if c["groups"] else "total",
                 c["score"], c["m_r"])
    if c["op"] == "route":
        nbytes = X.route_workspace_bytes(c["T"], p)
    else:
        s["x"] = _x(c, seed)
        ws, ss = _weights(c, seed, c["N"], 10, c["fmt"])
        s["w"] = ws
        if c["fmt"] == "fp8":
            s["w"] = ws + ss
        elif c["fmt"] == "mxfp4":     # the GEMMs' scale layout, made once with the weights
            s["w"] = ws + [X.tile_mx_scales(v) for v in ss]
        ep = sh = None
        if c["groups"]:
            s["opts"]["groups"] = X.GroupMap(c["groups"], None, c["local"])
            ep = s["opts"]["groups"].layout
        if c["shared"]:
            s["opts"]["shared"] = tuple(_weights(c, seed, c["shared"], 20, "bf16")[0])
            sh = X.SharedExperts(c["shared"], *[w.data_ptr() for w in s["opts"]["shared"]])
        size = X.layer_workspace_bytes if c["op"] == "layer" else X.moe_workspace_bytes
        nbytes = size(c["T"], c["d"], c["f"], p, ep, sh)
    s["ws"] = torch.empty(max(nbytes, 256), dtype=torch.uint8, device="cuda")
    return s


def run(state):
    s, c = state, state["case"]
    if c["op"] == "route":
        return X.route(s["logits"], c["k"], c["k0"], c["M"], "total", c["score"],
                       workspace=s["ws"])
    if c["op"] == "layer":
        return X.moe_layer(s["x"], s["gate"], *s["w"], c["k"], c["k0"], c["M"], "total",
                           c["score"], workspace=s["ws"], **s["opts"])
    call = {"bf16": X.moe_forward, "fp8": X.moe_forward_fp8,
            "mxfp4": X.moe_forward_mxfp4}[c["fmt"]]
    return call(s["x"], s["logits"], *s["w"], c["k"], c["k0"], c["M"], "total", c["score"],
                workspace=s["ws"], **s["opts"])


# ---------------------------------------------------------------------------- work, tolerance

def _active(c):
    """Experts whose weights a pass reads, on a batch of the case's distribution."""
    top = _logits(c, 0, "cpu").topk(c["k"], dim=1).indices
    used = torch.unique(top)
    if c["groups"]:
        size = c["N"] // c["groups"]
        return max(1, min(c["M"], int(((used // size) == c["local"]).sum())))
    return min(c["M"], int(used.numel()))


def work(case):
    c = case
    T, N, k, d, f = (c[a] for a in ("T", "N", "k", "d", "f"))
    out = N + T * k * 8 + 32                       # mask, ids, gates, counts
    if c["op"] == "route":
        return {"bytes": T * N * 4 + out, "flops": T * N * 4.0}
    per = {"bf16": 6 * d * f, "fp8": 3 * d * f + 4 * (2 * f + d),
           "mxfp4": 3 * d * f // 2 + 3 * d * f // 32}[c["fmt"]]
    rows = T * k if not c["groups"] else T * k / c["groups"]
    flops = 6.0 * d * f * (rows + T * c["shared"])
    nbytes = _active(c) * per + c["shared"] * 6 * d * f + T * d * 4 + T * N * 4 + out
    if c["op"] == "layer":
        nbytes += N * d * 2
        flops += 2.0 * T * N * d
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # selection is defined bit for bit on its fp32 logits.  y is rounded to bf16 once: against
    # 64 bits that alone is a relative error of 1.7e-3 and half a bf16 step (2^-8) at most.
    if case["op"] == "route":
        return "exact"
    return {"rel": 7e-3, "max": 1.6e-2, "differ": 0.002 if case["op"] == "layer" else 0.0}


# ---------------------------------------------------------------------------- in 64 bits

def _decode(w, s, fmt):
    if fmt == "bf16":
        return w.double()
    if fmt == "fp8":
        return w.view(torch.float8_e4m3fn).double() * s.double()[:, None]
    table = torch.tensor([0, 0.5, 1, 1.5, 2, 3, 4, 6], dtype=torch.float64, device=w.device)
    table = torch.cat([table, -table])
    v = torch.stack([table[(w & 15).long()], table[(w >> 4).long()]], dim=-1).flatten(-2)
    return v * torch.exp2(s.double() - 127.0).repeat_interleave(32, dim=-1)


def _rank(score):
    """Indices by score descending, index ascending on ties."""
    return sorted(range(len(score)), key=lambda j: (-score[j], j))


def _topk(h, k, allowed=None):
    """Each row's k best (logit descending, index ascending) among `allowed`."""
    v = h if allowed is None else np.where(allowed[None, :], h, -np.inf)
    return np.argsort(-v, axis=1, kind="stable")[:, :k]


def _gates(h, ids):
    z = np.take_along_axis(h, ids, 1)
    e = np.exp(z - z[:, :1])
    return e / e.sum(1, keepdims=True)


def _select(c, h):
    """(set mask, ids, gates) in 64 bits."""
    T, N = h.shape
    k, k0, M = c["k"], c["k0"], c["M"]
    ids = _topk(h, k)
    g = _gates(h, ids)
    G = np.zeros((T, N))
    np.put_along_axis(G, ids, g, 1)
    cand = np.zeros(N, bool)
    cand[ids.ravel()] = True
    chosen = np.zeros((T, N), bool)
    np.put_along_axis(chosen, ids, True, 1)
    if c["score"] == "dense":
        G = np.exp(h - h.max(1, keepdims=True))
        G /= G.sum(1, keepdims=True)
        cand[:] = True
        chosen[:] = True
    warm = np.zeros(N, bool)
    warm[ids[:, :k0].ravel()] = True
    score = G.sum(0)
    if c["groups"]:
        size = N // c["groups"]
        sel = warm.copy()
        while sel.sum() < M * c["groups"]:
            grew = False
            for grp in range(c["groups"]):
                mine = np.arange(N) // size == grp
                left = np.flatnonzero(mine & cand & ~sel)
                if (sel & mine).sum() >= M or not len(left):
                    continue
                sel[left[np.argmax(score[left])]] = True
                grew = True
            if not grew:
                break
        more = [j for j in _rank(score) if cand[j] and not sel[j]]
        sel[more[:max(0, min(k, int(cand.sum())) - int(sel.sum()))]] = True
    else:
        tier = np.where(warm, 0, np.where(cand, 2, 3))
        if c["reqs"] and c["m_r"]:
            step = T // c["reqs"]
            for r in range(c["reqs"]):
                at = slice(r * step, (r + 1) * step)
                first = np.zeros(N, bool)
                first[ids[at, :k0].ravel()] = True
                own = chosen[at].any(0) & ~first
                picks = [j for j in _rank(G[at].sum(0)) if own[j]][:c["m_r"]]
                tier[picks] = np.minimum(tier[picks], 1)
        order = sorted(np.flatnonzero(tier < 3), key=lambda j: (tier[j], -score[j], j))
        sel = np.zeros(N, bool)
        sel[order[:max(M, k)]] = True
    ids = _topk(h, k, sel)
    return sel, ids, _gates(h, ids)


def _swiglu(x, w1, w3, w2):
    a, b = x @ w1.t(), x @ w3.t()
    return (a * torch.sigmoid(a) * b) @ w2.t()


def exact(case, seed):
    c = case
    out = {}
    if c["op"] == "layer":
        x = _x(c, seed).double()
        h = x @ _router(c, seed).double().t()
        out["logits"] = h
        h = h.cpu().numpy()
    else:
        h = _logits(c, seed).double().cpu().numpy()
    sel, ids, w = _select(c, h)
    out.update(sel_mask=torch.from_numpy(sel.astype(np.uint8)),
               ids=torch.from_numpy(ids.astype(np.int32)), w=torch.from_numpy(w), stats=None)
    if c["op"] == "route":
        return out
    x = _x(c, seed).double()
    y = torch.zeros_like(x)
    ws, ss = _weights(c, seed, c["N"], 10, c["fmt"])
    tid, tw = torch.from_numpy(ids).cuda(), torch.from_numpy(w).cuda()
    for e in np.unique(ids):
        if c["groups"] and e // (c["N"] // c["groups"]) != c["local"]:
            continue
        t, r = torch.nonzero(tid == int(e), as_tuple=True)
        m = [_decode(a[e], b if b is None else b[e], c["fmt"]) for a, b in zip(ws, ss)]
        y.index_add_(0, t, tw[t, r, None] * _swiglu(x[t], *m))
    if c["shared"]:
        for m in zip(*_weights(c, seed, c["shared"], 20, "bf16")[0]):
            y += _swiglu(x, *[v.double() for v in m])
    out["y"] = y
    return out
