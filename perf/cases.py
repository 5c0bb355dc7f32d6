"""The work that a serving engine has this library do, as cases that can be timed and checked.

A decode step calls the whole MoE layer (lynx_moe_layer and its FP8 / MXFP4 variants) once per layer; an engine that has
its own router calls lynx_moe_ffn* with its own picks; one that keeps the remap apart from the expert FFN calls
lynx_route*, lynx_affinity_bin* and lynx_permute.  Batch sizes run from one sequence to the library's limit of 1024
tokens.  Shapes are those of the repository's configurations (Mixtral-8x7B, Qwen1.5-MoE, DeepSeek-V2-Lite, Qwen3-30B-A3B,
the routing side of a DeepSeek-V3-shaped layer) and, among the drawn cases, generic ones.

Inputs: hidden states N(0,1) in bf16, expert weights N(0, 0.02^2) in bf16 (quantised from there), router N(0, 1/H) with a
Zipf-shaped popularity bias, which gives the activation skew that the remap works on.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2411_08982_amd as L

#           H     F      N    k  shared F_shared zipf
SHAPES = {
    "tiny":      (512, 1024, 8, 2, 0, 0, 1.1),
    "mixtral":   (4096, 14336, 8, 2, 0, 0, 1.1),
    "qwen15moe": (2048, 1408, 60, 4, 1, 5632, 1.0),
    "dsv2lite":  (2048, 1408, 64, 6, 2, 1408, 0.9),
    "qwen3":     (2048, 768, 128, 8, 0, 0, 1.0),
    "dsv3":      (7168, 2048, 256, 8, 1, 2048, 1.0),
}
REMAP = {"off": (4.0, 1, 0), "moderate": (2.0, 2, 1), "aggressive": (4.0, 1, 1)}   # alpha, beta, enable
MAX_T = 1024


def _case(kind, shape, T, fmt="bf16", remap="aggressive", gate="softmax", groups=(1, 1), name=None):
    H, F, N, k, S, Fs, z = SHAPES[shape] if isinstance(shape, str) else shape
    c = dict(kind=kind, T=T, H=H, F=F, N=N, k=k, n_shared=S, F_shared=Fs, zipf=z, fmt=fmt, remap=remap, gate=gate,
             n_group=groups[0], topk_group=groups[1])
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # The smallest call: a layer of a small model, 16 sequences.  Launches and latency only.
        _case("layer", "tiny", 16, name="tiny_T16"),
        # One sequence decoding alone on a model of few, huge experts.
        _case("layer", "mixtral", 1, name="mixtral_T1"),
        # A handful of sequences, many small experts beside a wide shared one.
        _case("layer", "qwen15moe", 8, name="qwen15moe_T8"),
        # The batch size at which the remap saves most on a model of many tiny experts.
        _case("layer", "qwen3", 32, name="qwen3_T32"),
        # A ragged batch (continuous batching never fills a round number), the milder remap, two shared experts.
        _case("layer", "dsv2lite", 61, remap="moderate", name="dsv2lite_T61"),
        # The layer of the benchmark's headline stack: 512 sequences, nearly every expert in use.
        _case("layer", "qwen3", 512, name="qwen3_T512"),
        # The expert FFN alone, as an engine with its own router calls it: every expert holds tens of tokens.
        _case("ffn", "mixtral", 128, remap="off", name="mixtral_ffn_T128"),
        # A full decode batch at the upper end, where the remap is switched off because the batch is no longer bound by
        # weight traffic (the call's enable flag); ragged.
        _case("layer", "mixtral", 1000, remap="off", name="mixtral_T1000_off"),
        # Weight-only quantised serving, small batch: FP8.
        _case("layer", "mixtral", 8, fmt="fp8", name="mixtral_fp8_T8"),
        # The same with MXFP4 and many small experts.
        _case("layer", "dsv2lite", 16, fmt="fp4", name="dsv2lite_fp4_T16"),
        # Quantised weights, a larger ragged batch, the FFN alone.
        _case("ffn", "mixtral", 100, fmt="fp4", remap="off", name="mixtral_fp4_ffn_T100"),
        # The routing side alone for 256 experts: group-limited sigmoid router, remap, token assignment.
        _case("route", "dsv3", 200, remap="moderate", gate="sigmoid", groups=(8, 4), name="dsv3_route_T200"),
    ]


def _cost(c):
    """Rough microseconds of a pass at the card's rates: keeps a drawn case below the largest listed one."""
    w = work(c)
    return w["bytes"] / 6e6 + w["flops"] / 6e8


def draw(rng):
    limit = max(_cost(c) for c in listed())
    while True:
        kind = rng.choice(["layer", "layer", "ffn", "ffn", "route"])
        T = int(round(2.0 ** rng.uniform(0.0, math.log2(MAX_T))))
        fmt = rng.choice(["bf16", "bf16", "fp8", "fp4"])
        gate = rng.choice(["softmax", "softmax", "sigmoid"])
        remap = rng.choice(["off", "moderate", "aggressive", "aggressive"])
        if rng.random() < 0.3:   # a shape of its own: any sizes the format accepts
            step = {"bf16": 32, "fp8": 64, "fp4": 128}[fmt]
            size = lambda lo, hi: max(1, int(round(2.0 ** rng.uniform(math.log2(lo), math.log2(hi))) // step)) * step
            N = int(round(2.0 ** rng.uniform(3.0, 8.0)))
            S = rng.choice([0, 0, 1, 2])
            shape = (size(512, 4096), size(256, 4096), N, rng.randint(1, min(8, N)), S, size(256, 4096) if S else 0, 1.0)
        else:
            shape = rng.choice(["tiny", "mixtral", "qwen15moe", "dsv2lite", "qwen3"] if kind != "route" else list(SHAPES))
        c = _case(kind, shape, T, fmt, remap, gate)
        if kind == "route":
            c["fmt"] = "bf16"
            if rng.random() < 0.4:
                opts = [(g, tg) for g in (2, 4, 8) for tg in (1, 2, 4) if tg < g and c["N"] % g == 0 and tg * c["N"] // g >= c["k"]]
                if opts:
                    c["n_group"], c["topk_group"] = rng.choice(opts)
        elif kind == "layer" and fmt != "bf16":
            c["gate"] = "softmax"
        stored = 6 * c["H"] * (c["F"] * c["N"] + c["F_shared"] * c["n_shared"])   # all experts, in bf16 before packing
        if _cost(c) <= limit and (kind == "route" or stored <= 4 << 30):
            return c


# ---- the method in plain numpy, 64-bit: for exact() and for the expert counts of work() --------------------------------

def _zipf_bias(N, s, rng):
    lw = -s * np.log(rng.permutation(N) + 1.0)
    return 0.5 * (lw - lw.mean())


def _top(values, allowed, k):
    v = np.where(allowed, values, -np.inf)
    return np.argsort(-v, axis=1, kind="stable")[:, :k]


def _select(z, c):
    """Logits [T,N] -> allowed mask, own picks [T,k], remapped picks [T,k]."""
    T, N = z.shape
    k, G, TG = c["k"], c["n_group"], c["topk_group"]
    alpha, beta, enable = REMAP[c["remap"]]
    allowed = np.ones((T, N), bool)
    if G > 1 and TG < G:
        best = z.reshape(T, G, N // G).max(axis=2)
        chosen = np.zeros((T, G), bool)
        np.put_along_axis(chosen, np.argsort(-best, axis=1, kind="stable")[:, :TG], True, axis=1)
        allowed = np.repeat(chosen, N // G, axis=1)
    own = _top(z, allowed, k)
    if not enable or T <= 1:
        return allowed, own, own
    za = np.where(allowed, z, -np.inf)
    q = np.minimum(np.floor(alpha * (za.max(axis=1, keepdims=True) - za)), beta).astype(np.int64)
    score = np.zeros(N, object)
    for j in range(beta):
        score = score * T + np.array([int(x) for x in ((q == j) & allowed).sum(axis=0)], object)
    order = np.array(sorted(range(N), key=lambda e: (-score[e], e)))
    in_use = np.zeros(N, bool)
    in_use[own.ravel()] = True
    active = np.zeros(N, bool)
    cand = order[in_use[order]]
    for t in range(T):
        free = allowed[t, cand].copy()
        qc = q[t, cand]
        for s in range(k):
            qs = q[t, own[t, s]]
            if qs >= beta:
                break
            hit = np.flatnonzero(free & (qc <= qs))
            if hit.size:
                active[cand[hit[0]]] = True
                free[hit[0]] = False
    for e in cand:
        if active.sum() >= k:
            break
        active[e] = True
    new = _top(z, allowed & active, k)
    for t in np.flatnonzero((allowed & active).sum(axis=1) < k):
        have = int((allowed[t] & active).sum())
        new[t, have:] = [e for e in own[t] if not active[e]][:k - have]
    return allowed, own, new


def _gates(z, idx, c):
    zs = np.take_along_axis(z, idx, axis=1)
    if c["gate"] == "sigmoid":
        s = 1.0 / (1.0 + np.exp(-zs))
        return s / s.sum(axis=1, keepdims=True), s.sum(axis=1)
    e = np.exp(zs - zs.max(axis=1, keepdims=True))
    full = np.exp(z - zs.max(axis=1, keepdims=True)).sum(axis=1)
    return e / e.sum(axis=1, keepdims=True), e.sum(axis=1) / full


def _experts_in_use(c):
    rng = np.random.default_rng(7)
    z = rng.standard_normal((c["T"], c["N"])) + _zipf_bias(c["N"], c["zipf"], rng)
    return len(np.unique(_select(z, c)[2]))


def work(case):
    c = case
    T, H, F, N, k = c["T"], c["H"], c["F"], c["N"], c["k"]
    nbytes = flops = 0
    if c["kind"] != "ffn":      # router: x, Wr and bias in; logits, picks, gates and the assignment out
        nbytes += T * H * 2 + N * H * 4 + N * 4 + T * N * 4 + T * k * 20 + T * 8
        flops += 2 * T * H * N
    if c["kind"] != "route":    # experts in use and shared experts once, tokens in, layer output out
        per_weight = {"bf16": 2.0, "fp8": 1.0, "fp4": 17.0 / 32.0}[c["fmt"]]
        weights = 3 * H * F * _experts_in_use(c) + 3 * H * c["F_shared"] * c["n_shared"]
        nbytes += weights * per_weight + T * H * 4 + (T * H * 2 + T * k * 12 if c["kind"] == "ffn" else 0)
        flops += 2 * 3 * H * (F * T * k + c["F_shared"] * c["n_shared"] * T)
    return {"bytes": int(nbytes), "flops": int(flops)}


def tolerance(case):
    # The routing side is fp32 sums over the hidden size.  The layer rounds the intermediate vector to bf16 between the
    # projections, which alone puts y 1.7e-3 from the 64-bit result (measured, the same for every weight format).  A pick
    # may differ where two logits are equal to within their last bits.
    if case["kind"] == "route":
        return {"rel": 1e-5, "differ": 2e-3}
    return {"rel": 7e-3, "max": 5e-2, "differ": 2e-3}


# ---- inputs -------------------------------------------------------------------------------------------------------------

def _generator(seed, part):
    g = torch.Generator(device="cuda")
    g.manual_seed((seed * 1000003 + part) & 0x7fffffffffff)
    return g


def _tokens_and_router(c, seed):
    g = _generator(seed, 1)
    x = torch.randn((c["T"], c["H"]), generator=g, device="cuda").to(torch.bfloat16)
    Wr = torch.randn((c["N"], c["H"]), generator=g, device="cuda") / math.sqrt(c["H"])
    bias = torch.from_numpy(_zipf_bias(c["N"], c["zipf"], np.random.default_rng(seed)).astype(np.float32)).cuda()
    return x, Wr, bias


def _logits64(x, Wr, bias):
    return (x.double() @ Wr.double().T + bias.double()).cpu().numpy()


def _picks(c, x, Wr, bias):
    """Picks and gates that an engine's own router hands to the FFN."""
    z = _logits64(x, Wr, bias)
    idx = _select(z, c)[2]
    return idx, _gates(z, idx, c)[0].astype(np.float32)


def _weights(E, H, F, seed, part):
    """Row-major gate, up [E,F,H] and down [E,H,F]."""
    g = _generator(seed, part)
    out = []
    for rows, cols in ((F, H), (F, H), (H, F)):
        w = torch.empty((E, rows, cols), dtype=torch.bfloat16, device="cuda")
        for e in range(E):
            w[e] = torch.randn((rows, cols), generator=g, device="cuda").mul_(0.02)
        out.append(w)
    return out


PACK = {"bf16": "lynx_pack_weights", "fp8": "lynx_quantize_weights_fp8", "fp4": "lynx_quantize_weights_fp4"}


def prepare(case, seed):
    c = dict(case)
    T, H, F, N, k, S, Fs = c["T"], c["H"], c["F"], c["N"], c["k"], c["n_shared"], c["F_shared"]
    alpha, beta, _ = REMAP[c["remap"]]
    x, Wr, bias = _tokens_and_router(c, seed)
    st = dict(c=c, x=x, Wr=Wr, bias=bias)
    if c["kind"] == "route":
        return st
    st["W"] = getattr(L, PACK[c["fmt"]])(*_weights(N, H, F, seed, 2))
    st["S"] = getattr(L, PACK[c["fmt"]])(*_weights(S, H, Fs, seed, 3)) if S else None
    if c["kind"] == "layer":
        st["buffers"] = L.LayerBuffers(T, H, F, N, k, beta, S, Fs)
    else:
        idx, gate = _picks(c, x, Wr, bias)
        st["idx"] = torch.from_numpy(idx.astype(np.int32)).cuda()
        st["gate"] = torch.from_numpy(gate).cuda()
        st["perm"] = L.lynx_permute(st["idx"], N)
        st["workspace"] = L.new_workspace(T, H, F, N, k, S, Fs)
        st["y"] = torch.empty((T, H), dtype=torch.float32, device="cuda")
    torch.cuda.empty_cache()   # the row-major weights are gone: a program keeps the packed ones only
    return st


def run(state):
    s, c = state, state["c"]
    alpha, beta, enable = REMAP[c["remap"]]
    k, N, F = c["k"], c["N"], c["F"]
    if c["kind"] == "route":
        if c["n_group"] > 1:
            fn = 1 if c["gate"] == "sigmoid" else 0
            r = L.lynx_route_grouped(s["x"], s["Wr"], s["bias"], k, c["n_group"], c["topk_group"], fn)
            a = L.lynx_affinity_bin_grouped(r["logits"], k, c["n_group"], c["topk_group"], alpha, beta, fn, enable)
        else:
            sig = "_sigmoid" if c["gate"] == "sigmoid" else ""
            r = getattr(L, "lynx_route" + sig)(s["x"], s["Wr"], s["bias"], k)
            a = getattr(L, "lynx_affinity_bin" + sig)(r["logits"], r["idx"], alpha, beta, enable)
        p = L.lynx_permute(a["new_idx"], N)
        return dict(logits=r["logits"], idx=r["idx"], gate=r["gate"], psum=r["psum"], new_idx=a["new_idx"],
                    new_gate=a["new_gate"], new_psum=a["new_psum"], cnt_before=a["cnt_before"], cnt_after=a["cnt_after"],
                    bin_hist=a["bin_hist"], num_active=a["num_active"], offsets=p["offsets"], perm=p["perm"],
                    active=p["active"])
    shared = dict(n_shared=c["n_shared"], F_shared=c["F_shared"])
    if c["fmt"] == "bf16":
        weights = s["W"]
        if s["S"] is not None:
            shared.update(Sgu=s["S"][0], Sdp=s["S"][1])
        suffix = ""
    else:
        weights = (s["W"],)
        shared["shared"] = s["S"]
        suffix = "_" + c["fmt"]
    if c["kind"] == "ffn":
        return getattr(L, "lynx_moe_ffn" + suffix)(s["x"], *weights, s["idx"], s["gate"], s["perm"], N, F,
                                                   workspace=s["workspace"], y=s["y"], **shared)
    if c["gate"] == "sigmoid":
        suffix = "_sigmoid"
    b = getattr(L, "lynx_moe_layer" + suffix)(s["x"], s["Wr"], s["bias"], *weights, F, k, alpha, beta, enable,
                                              buffers=s["buffers"], **shared)
    return dict(y=b.y, logits=b.logits, idx=b.topk_idx, gate=b.topk_gate, psum=b.topk_psum, new_idx=b.new_idx,
                new_gate=b.new_gate, new_psum=b.new_psum, cnt_before=b.cnt_before, cnt_after=b.cnt_after,
                bin_hist=b.bin_hist, num_active=b.num_active, offsets=b.offsets, perm=b.perm, active=b.active,
                status=b.status)


# ---- the same in 64 bits ------------------------------------------------------------------------------------------------

def _stored(w, fmt):
    """The value that the weight format stores for a bf16 matrix [rows, cols], in float64."""
    if fmt == "fp8":
        w = w.float()
        amax = w.abs().amax(dim=1, keepdim=True)
        scale = torch.where(amax == 0, torch.ones_like(amax), amax / torch.full_like(amax, 448.0))
        return (w / scale).to(torch.float8_e4m3fn).double() * scale.double()
    if fmt == "fp4":
        b = w.double().reshape(w.shape[0], -1, 32)
        amax = b.abs().amax(dim=2, keepdim=True)
        e = torch.where(amax == 0, torch.zeros_like(amax), torch.frexp(amax)[1].double() - 3.0)   # floor(log2) - 2
        scale = torch.exp2(e)
        m = (b / scale).abs()
        step = torch.where(m < 2, 0.5, torch.where(m < 4, 1.0, 2.0))
        m = (torch.round(m / step) * step).clamp(max=6.0)   # torch.round: ties to even, which is the even code
        return (torch.sign(b) * m * scale).reshape(w.shape)
    return w.double()


def _expert64(x, Wg, Wu, Wd, fmt):
    g = x @ _stored(Wg, fmt).T
    h = g * torch.sigmoid(g) * (x @ _stored(Wu, fmt).T)
    return h @ _stored(Wd, fmt).T


def _ffn64(c, seed, x, idx, gate):
    Wg, Wu, Wd = _weights(c["N"], c["H"], c["F"], seed, 2)
    xd = x.double()
    y = torch.zeros((c["T"], c["H"]), dtype=torch.float64, device="cuda")
    for e in np.unique(idx):
        t, j = np.nonzero(idx == e)
        ti = torch.from_numpy(t).cuda()
        o = _expert64(xd[ti], Wg[e], Wu[e], Wd[e], c["fmt"])
        y.index_add_(0, ti, o * torch.from_numpy(gate[t, j].astype(np.float64)).cuda()[:, None])
    if c["n_shared"]:
        Sg, Su, Sd = _weights(c["n_shared"], c["H"], c["F_shared"], seed, 3)
        for s in range(c["n_shared"]):
            y += _expert64(xd, Sg[s], Su[s], Sd[s], c["fmt"])
    return y


def exact(case, seed):
    c = case
    x, Wr, bias = _tokens_and_router(c, seed)
    if c["kind"] == "ffn":
        return _ffn64(c, seed, x, *_picks(c, x, Wr, bias))
    z = _logits64(x, Wr, bias)
    _, own, new = _select(z, c)
    gate, psum = _gates(z, own, c)
    new_gate, new_psum = _gates(z, new, c)
    out = dict(logits=z, idx=None, gate=gate, psum=psum, new_idx=None, new_gate=new_gate, new_psum=new_psum,
               cnt_before=None, cnt_after=None, bin_hist=None, num_active=None, offsets=None, perm=None, active=None)
    if c["kind"] == "layer":
        out = dict(y=_ffn64(c, seed, x, new, new_gate), **out, status=None)
    return out
