"""GPU parity: every C-ABI entry point of liblynx against the CPU oracle on the same seeded inputs.

Bars: integer outputs (indices, counts, offsets, permutation, histogram) bit-exact given identical
fp32 logits; router logits within 1e-5; gates within 1e-5; layer outputs within 1e-2 per token row
(max_h |y - y_ref| / max_h |y_ref|; bf16 operands, fp32 accumulation, bf16 intermediate vector).
"""
import numpy as np
import pytest
import torch

import oracle
import workloads as wl
from gpu_util import bf16_bits, dev, host, pack_reference, row_rel_err, to_bf16_dev

pytestmark = pytest.mark.gpu

Y_TOL = 1e-2
LOGIT_TOL = 1e-5
GATE_TOL = 1e-5


@pytest.fixture(scope="module")
def L():
    import paper_2411_08982_amd as lib
    lib.lib()   # fails loudly if liblynx.so is not built
    assert torch.cuda.is_available()
    return lib


def _say(msg):
    print(msg, flush=True)


# ------------------------------------------------------------------------------------------------ route

@pytest.mark.parametrize("T,H,N,k,bias", [(16, 512, 8, 2, True), (1, 4096, 8, 2, True), (33, 2048, 60, 4, True),
                                          (64, 2048, 64, 6, False), (128, 2048, 128, 8, True), (5, 32, 256, 16, True),
                                          (3, 64, 4, 4, True)])
def test_route(L, T, H, N, k, bias):
    _say(f"route T={T} H={H} N={N} k={k}")
    rng = np.random.default_rng(T * 7 + N)
    x = wl.f32_to_bf16_bits(rng.standard_normal((T, H)).astype(np.float32))
    Wr = (rng.standard_normal((N, H)) / np.sqrt(H)).astype(np.float32)
    b = wl.zipf_bias(N, 1.0, 0.5, rng) if bias else None
    ref = oracle.route(x, Wr, b, k)
    out = L.lynx_route(to_bf16_dev(x), dev(Wr), None if b is None else dev(b), k)
    torch.cuda.synchronize()
    z = host(out["logits"])
    assert np.all(np.abs(z - ref["logits"]) <= LOGIT_TOL * np.maximum(1.0, np.abs(ref["logits"])))
    # selection, gates and selected mass are judged on the GPU's own fp32 logits (identical logits on both sides)
    ref2 = oracle.topk(z, k)
    assert np.array_equal(host(out["idx"]), ref2["idx"])
    np.testing.assert_allclose(host(out["gate"]), ref2["gate"], rtol=GATE_TOL, atol=1e-7)
    np.testing.assert_allclose(host(out["psum"]), ref2["psum"], rtol=GATE_TOL, atol=1e-7)


def test_route_ties_go_to_lower_index(L):
    H = N = 32
    rng = np.random.default_rng(1)
    Wr = rng.integers(-2, 3, size=(N, H)).astype(np.float32)      # exact small-integer logits, many ties
    x = wl.f32_to_bf16_bits(np.eye(H, dtype=np.float32))
    out = L.lynx_route(to_bf16_dev(x), dev(Wr), None, 5)
    torch.cuda.synchronize()
    ref = oracle.route(x, Wr, None, 5)
    assert np.array_equal(host(out["logits"]), ref["logits"])
    assert np.array_equal(host(out["idx"]), ref["idx"])


# ------------------------------------------------------------------------------------------------ affinity_bin

BIN_CASES = [(16, 8, 2, 1.1, 0.0), (8, 8, 2, 1.1, 0.0), (32, 60, 4, 1.0, 0.0), (64, 64, 6, 0.9, 0.05),
             (128, 128, 8, 1.0, 0.0), (512, 128, 8, 1.0, 0.0), (256, 64, 6, 0.9, 0.05), (5, 6, 3, 1.0, 0.2),
             (2, 4, 2, 1.0, 0.0), (1, 8, 2, 1.0, 0.0), (33, 17, 5, 1.0, 0.1), (1024, 256, 16, 1.0, 0.0),
             (7, 200, 16, 1.0, 0.0), (40, 10, 10, 1.0, 0.0), (9, 12, 1, 1.0, 0.0), (70, 12, 1, 1.0, 0.0),
             # expert counts above 64 that leave the last group of 64 score ranks partly empty, no popularity prior, many
             # picks per token: experts of the last ranks get nominated (a lane past the last rank must still take part
             # in the lane exchanges that fetch a ranked expert's logit)
             (65, 200, 14, 0.0, 0.0), (16, 100, 12, 0.0, 0.0), (48, 130, 16, 0.0, 0.0), (300, 250, 10, 0.3, 0.1)]


def _check_bin(L, z, k, alpha, beta, enable):
    idx = oracle.topk(z, k)["idx"]
    ref = oracle.affinity_bin(z, idx, alpha, beta, enable)
    out = L.lynx_affinity_bin(dev(z), dev(idx), alpha, beta, enable)
    torch.cuda.synchronize()
    for key in ("new_idx", "cnt_before", "cnt_after", "bin_hist", "num_active"):
        assert np.array_equal(host(out[key]), ref[key]), key
    np.testing.assert_allclose(host(out["new_gate"]), ref["new_gate"], rtol=GATE_TOL, atol=1e-7)
    # the probability mass of the new selection (the remap's "top-k weight sum"), and against the router's own: the
    # GPU computes both the same way, so a token whose selection did not change shows the same bits
    np.testing.assert_allclose(host(out["new_psum"]), ref["new_psum"], rtol=GATE_TOL, atol=1e-7)
    top = L.lynx_affinity_bin(dev(z), dev(idx), alpha, beta, 0)
    torch.cuda.synchronize()
    same = np.all(np.sort(host(out["new_idx"]), axis=1) == np.sort(idx, axis=1), axis=1)
    assert np.array_equal(host(out["new_psum"])[same], host(top["new_psum"])[same])
    assert np.all(host(out["new_psum"]) <= host(top["new_psum"]) * (1 + 1e-6))
    return ref


@pytest.mark.parametrize("T,N,k,s,tail", BIN_CASES)
def test_affinity_bin(L, T, N, k, s, tail):
    for alpha, beta in [(2.0, 2), (4.0, 1), (1.0, 3), (0.5, 6), (0.0, 2), (1.0e6, 1)]:
        if T ** beta >= 2 ** 62:
            continue
        for seed, quantum in [(0, None), (1, 0.25)]:               # quantised logits: exact ties and bin-boundary hits
            _say(f"affinity_bin T={T} N={N} k={k} alpha={alpha} beta={beta} seed={seed} quantum={quantum}")
            z = wl.make_logits(T, N, seed=seed * 100 + T, zipf_s=s, tail_frac=tail, quantum=quantum)
            ref = _check_bin(L, z, k, alpha, beta, 1)
            if T > 1 and alpha > 0:
                assert ref["num_active"][1] <= ref["num_active"][0]
    z = wl.make_logits(T, N, seed=3, zipf_s=s, tail_frac=tail)
    _check_bin(L, z, k, 2.0, 2, 0)                                   # bypass


@pytest.mark.parametrize("T,N,beta", [(256, 255, 3), (256, 256, 3), (1024, 64, 2), (1024, 256, 2), (40, 100, 6), (16, 255, 3)])
def test_affinity_bin_score_order_at_the_key_width_boundary(L, T, N, beta):
    """The kernels order the experts by one 32-bit key, score * N + (N - 1 - index), whenever its largest possible value
    fits (a score reaches T^beta when every token puts an expert into bin 0), and by the 64-bit score otherwise.  Both
    sides of that switch, with every token agreeing on its top expert so that the largest score occurs, and with
    many equal scores so that the index decides."""
    k = 4
    _say(f"score order at the key boundary: T={T} N={N} beta={beta} (T^beta*N+N = {T ** beta * N + N}, 2^32 = {2 ** 32})")
    z = wl.make_logits(T, N, seed=T + N, quantum=0.5)
    z[:, 7] = z.max() + 1.0                       # everybody's top-1: the score T^beta occurs
    for alpha in (1.0, 0.25):
        _check_bin(L, z, k, alpha, beta, 1)


def test_affinity_bin_signed_zero_logits_stay_tied(L):
    """-0.0 and +0.0 are equal logits: the lower expert index wins, whichever sign it carries (the kernels pick on
    integer keys of the floats, which would tell the two zeros apart if -0 were not made +0 first)."""
    for T, N, k in [(3, 6, 2), (20, 70, 5)]:
        rng = np.random.default_rng(N)
        z = np.where(rng.random((T, N)) < 0.5, np.float32(-0.0), np.float32(0.0)).astype(np.float32)
        z[:, N - 2:] = -5.0
        assert np.signbit(z).any() and (~np.signbit(z)).any()
        idx = oracle.topk(z, k)["idx"]
        assert np.array_equal(idx, np.tile(np.arange(k, dtype=np.int32), (T, 1)))      # all zeros tie: indices 0..k-1
        _say(f"signed zeros T={T} N={N} k={k}")
        for alpha, beta in [(1.0, 1), (2.0, 3)]:
            _check_bin(L, z, k, alpha, beta, 1)


def test_affinity_bin_picks_in_any_order(L):
    """Picks that are k distinct experts but neither the top-k nor in rank order: same result as the oracle, which
    lets a slot without a candidate nominate nothing."""
    for seed in range(12):
        rng = np.random.default_rng(seed)
        T = int(rng.choice([3, 16, 17, 70, 300]))
        N = int(rng.choice([5, 60, 100, 130, 256]))
        k = int(rng.integers(1, min(N, 16) + 1))
        alpha, beta = float(rng.choice([0.5, 2.0, 4.0])), int(rng.integers(1, 5))
        _say(f"affinity_bin, arbitrary picks: T={T} N={N} k={k} alpha={alpha} beta={beta}")
        z = wl.make_logits(T, N, seed=seed, quantum=[None, 0.25][seed % 2])
        idx = np.stack([rng.permutation(N)[:k] for _ in range(T)]).astype(np.int32)
        ref = oracle.affinity_bin(z, idx, alpha, beta, 1)
        out = L.lynx_affinity_bin(dev(z), dev(idx), alpha, beta, 1)
        torch.cuda.synchronize()
        for key in ("new_idx", "cnt_before", "cnt_after", "bin_hist", "num_active"):
            assert np.array_equal(host(out[key]), ref[key]), key
        np.testing.assert_allclose(host(out["new_gate"]), ref["new_gate"], rtol=GATE_TOL, atol=1e-7)


def test_affinity_bin_worked_example(L, golden_w1):
    z = np.array(golden_w1["logits"], np.float32)
    idx = np.array(golden_w1["topk_idx"], np.int32)
    out = L.lynx_affinity_bin(dev(z), dev(idx), 1.0, 2, 1)
    torch.cuda.synchronize()
    assert host(out["new_idx"]).tolist() == [[int(v) for v in r] for r in golden_w1["new_idx"]]
    assert host(out["cnt_after"]).tolist() == [int(v) for v in golden_w1["cnt_after"][0]]
    assert host(out["num_active"]).tolist() == [4, 2]
    np.testing.assert_allclose(host(out["new_gate"]), np.array(golden_w1["gate_after"]), atol=6e-6)


def test_affinity_bin_is_deterministic(L):
    z = wl.make_logits(256, 128, seed=9, tail_frac=0.05)
    idx = dev(oracle.topk(z, 8)["idx"])
    zd = dev(z)
    first = {k_: host(v).copy() for k_, v in L.lynx_affinity_bin(zd, idx, 2.0, 2, 1).items()}
    for _ in range(5):
        again = L.lynx_affinity_bin(zd, idx, 2.0, 2, 1)
        torch.cuda.synchronize()
        for key, v in first.items():
            assert np.array_equal(host(again[key]), v), key


@pytest.mark.parametrize("T,N,k,s,tail", BIN_CASES)
def test_affinity_bin_biased(L, T, N, k, s, tail):
    """Score-biased selection variant: every integer output bit-exact, gates within tolerance."""
    for alpha, beta, gamma in [(2.0, 2, 1.0), (4.0, 1, 0.5), (1.0, 3, 4.0), (0.5, 6, 0.0), (2.0, 2, 1.0e6)]:
        if T ** beta >= 2 ** 62:
            continue
        for seed, quantum in [(0, None), (1, 0.25)]:               # quantised logits: exact ties in logit + bias
            _say(f"affinity_bin_biased T={T} N={N} k={k} alpha={alpha} beta={beta} gamma={gamma} seed={seed} q={quantum}")
            z = wl.make_logits(T, N, seed=seed * 100 + T, zipf_s=s, tail_frac=tail, quantum=quantum)
            idx = oracle.topk(z, k)["idx"]
            ref = oracle.affinity_bin_biased(z, idx, alpha, beta, gamma, 1)
            out = L.lynx_affinity_bin_biased(dev(z), dev(idx), alpha, beta, gamma, 1)
            torch.cuda.synchronize()
            for key in ("new_idx", "cnt_before", "cnt_after", "bin_hist", "num_active"):
                assert np.array_equal(host(out[key]), ref[key]), key
            np.testing.assert_allclose(host(out["new_gate"]), ref["new_gate"], rtol=GATE_TOL, atol=1e-7)
            np.testing.assert_allclose(host(out["new_psum"]), ref["new_psum"], rtol=GATE_TOL, atol=1e-7)
    z = wl.make_logits(T, N, seed=3, zipf_s=s, tail_frac=tail)
    idx = oracle.topk(z, k)["idx"]
    out = L.lynx_affinity_bin_biased(dev(z), dev(idx), 2.0, 2, 3.0, 0)   # bypass
    torch.cuda.synchronize()
    assert np.array_equal(host(out["new_idx"]), idx)


def test_biased_selection_through_the_ffn(L):
    """The variant composes with lynx_permute and lynx_moe_ffn: whole layer against the oracle."""
    cfg = wl.CONFIGS["tiny"]
    T = 40
    d = wl.make_layer(cfg, T)
    x, Wr, bias = to_bf16_dev(d["x"]), dev(d["Wr"]), dev(d["bias"])
    r = L.lynx_route(x, Wr, bias, cfg.k)
    a = L.lynx_affinity_bin_biased(r["logits"], r["idx"], 2.0, 2, 2.0, 1)
    p = L.lynx_permute(a["new_idx"], cfg.N)
    Wgu, Wdp = L.lynx_pack_weights(to_bf16_dev(d["Wg"]), to_bf16_dev(d["Wu"]), to_bf16_dev(d["Wd"]))
    y = L.lynx_moe_ffn(x, Wgu, Wdp, a["new_idx"], a["new_gate"], p, cfg.N, cfg.F)
    torch.cuda.synchronize()
    z = host(r["logits"])
    ra = oracle.affinity_bin_biased(z, oracle.topk(z, cfg.k)["idx"], 2.0, 2, 2.0, 1)
    assert np.array_equal(host(a["new_idx"]), ra["new_idx"])
    assert ra["num_active"][1] <= ra["num_active"][0]
    y_ref = oracle.moe_ffn(d["x"], d["Wg"], d["Wu"], d["Wd"], ra["new_idx"], ra["new_gate"])
    assert row_rel_err(host(y), y_ref).max() <= Y_TOL


# ------------------------------------------------------------------------------------------------ permute

# The logits on the matrix cores: hidden sizes that leave waves without a k-step, with an odd number of them and with the last one
# short; token and expert tiles that are partly filled; both sides of the line at T * N = 8192 and of 128 tokens.
@pytest.mark.parametrize("T,H,N", [(129, 32, 3), (130, 96, 17), (200, 288, 16), (129, 544, 60), (32, 256, 256), (31, 256, 256), (65, 2080, 127),
                                   (145, 800, 33), (1024, 64, 8), (128, 7168, 63)])
def test_logits_of_large_batches(L, T, H, N):
    _say(f"logits T={T} H={H} N={N}")
    rng = np.random.default_rng([T, H, N])
    x = wl.f32_to_bf16_bits(rng.standard_normal((T, H)).astype(np.float32))
    Wr = (rng.standard_normal((N, H)) / np.sqrt(H)).astype(np.float32)
    b = rng.standard_normal(N).astype(np.float32)
    out = L.lynx_route(to_bf16_dev(x), dev(Wr), dev(b), min(4, N))
    want = wl.bf16_bits_to_f32(x).astype(np.float64) @ Wr.astype(np.float64).T + b
    assert np.all(np.abs(host(out["logits"]) - want) <= 1e-5 * np.maximum(1.0, np.abs(want)))


@pytest.mark.parametrize("T,N,k", [(1, 1, 1), (1024, 1, 1), (33, 3, 3), (1023, 256, 7), (1024, 255, 16), (17, 129, 13), (700, 64, 11)])
def test_permute_with_skipped_pairs(L, T, N, k):
    """Every number of picks divides pair ids into tokens; pairs without an expert leave -1 at the end of the permutation."""
    _say(f"permute with skipped pairs T={T} N={N} k={k}")
    rng = np.random.default_rng([T, N, k])
    idx = np.stack([rng.permutation(N)[:k] for _ in range(T)]).astype(np.int32)
    idx[rng.random(idx.shape) < 0.2] = -1
    idx[rng.random(idx.shape) < 0.05] = N
    flat = idx.ravel()
    valid = np.flatnonzero((flat >= 0) & (flat < N))
    want = np.full(T * k, -1, np.int32)
    want[:valid.size] = valid[np.argsort(flat[valid], kind="stable")]
    counts = np.bincount(flat[valid], minlength=N)
    out = L.lynx_permute(dev(idx), N)
    torch.cuda.synchronize()
    assert np.array_equal(host(out["perm"]), want)
    assert np.array_equal(host(out["offsets"]), np.concatenate([[0], np.cumsum(counts)]))
    used = np.flatnonzero(counts)
    assert host(out["num_active"])[0] == used.size
    assert np.array_equal(host(out["active"]), np.concatenate([used, np.full(N - used.size, -1)]))


@pytest.mark.parametrize("T,N,k,seed", [(1, 4, 2, 0), (16, 8, 2, 1), (37, 60, 4, 2), (128, 128, 8, 3), (512, 128, 8, 4),
                                        (1024, 256, 16, 5), (100, 8, 8, 6), (65, 3, 1, 7)])
def test_permute(L, T, N, k, seed):
    _say(f"permute T={T} N={N} k={k}")
    rng = np.random.default_rng(seed)
    hot = max(k, N // 3)                                             # leave some experts empty
    idx = np.stack([rng.permutation(hot)[:k] for _ in range(T)]).astype(np.int32)
    ref = oracle.permute(idx, N)
    out = L.lynx_permute(dev(idx), N)
    torch.cuda.synchronize()
    for key in ("offsets", "perm", "active", "num_active"):
        assert np.array_equal(host(out[key]), ref[key]), key


# ------------------------------------------------------------------------------------------------ pack + FFN

def test_pack_weights_layout(L):
    rng = np.random.default_rng(0)
    E, F, H = 3, 96, 64
    Wg, Wu = (rng.integers(0, 65536, size=(E, F, H)).astype(np.uint16) for _ in range(2))
    Wd = rng.integers(0, 65536, size=(E, H, F)).astype(np.uint16)
    Wgu, Wdp = L.lynx_pack_weights(to_bf16_dev(Wg), to_bf16_dev(Wu), to_bf16_dev(Wd))
    torch.cuda.synchronize()
    gu_ref = np.stack([pack_reference(Wg), pack_reference(Wu)], axis=3)          # [E, F/16, H/32, 2, 64, 8]
    assert np.array_equal(bf16_bits(Wgu), gu_ref)
    assert np.array_equal(bf16_bits(Wdp), pack_reference(Wd))


def _ffn_case(L, T, H, F, N, k, S, Fs, seed, hot=None, std=0.05):
    rng = np.random.default_rng(seed)
    x = wl.f32_to_bf16_bits(rng.standard_normal((T, H)).astype(np.float32))
    Wg, Wu, Wd = wl.bf16_normal(rng, (N, F, H), std), wl.bf16_normal(rng, (N, F, H), std), wl.bf16_normal(rng, (N, H, F), std)
    Sg = Su = Sd = None
    if S:
        Sg, Su, Sd = (wl.bf16_normal(rng, (S, Fs, H), std), wl.bf16_normal(rng, (S, Fs, H), std),
                      wl.bf16_normal(rng, (S, H, Fs), std))
    hot = hot or N
    idx = np.stack([rng.permutation(hot)[:k] for _ in range(T)]).astype(np.int32)
    gate = rng.random((T, k)).astype(np.float32) + 0.1
    gate /= gate.sum(1, keepdims=True)
    y_ref = oracle.moe_ffn(x, Wg, Wu, Wd, idx, gate.astype(np.float64), Sg, Su, Sd)
    Wgu, Wdp = L.lynx_pack_weights(to_bf16_dev(Wg), to_bf16_dev(Wu), to_bf16_dev(Wd))
    Sgu = Sdp = None
    if S:
        Sgu, Sdp = L.lynx_pack_weights(to_bf16_dev(Sg), to_bf16_dev(Su), to_bf16_dev(Sd))
    idx_d = dev(idx)
    p = L.lynx_permute(idx_d, N)
    # workspace and output start as NaN / -1 patterns: nothing may depend on what a fresh allocation happens to hold
    ws = L.new_workspace(T, H, F, N, k, S, Fs, "cuda")
    ws.view(torch.uint8).fill_(0xFF)
    y0 = torch.full((T, H), float("nan"), dtype=torch.float32, device="cuda")
    y = L.lynx_moe_ffn(to_bf16_dev(x), Wgu, Wdp, idx_d, dev(gate), p, N, F, Sgu, Sdp, S, Fs, workspace=ws, y=y0)
    torch.cuda.synchronize()
    err = row_rel_err(host(y), y_ref)
    assert np.all(np.isfinite(host(y)))
    assert err.max() <= Y_TOL, f"max row error {err.max():.3e}"
    return err.max()


FFN_CASES = [
    # T,   H,   F,  N, k, S, Fs, hot     what it covers
    (16, 512, 1024, 8, 2, 0, 0, None),   # the tiny configuration's shapes
    (1, 256, 320, 4, 2, 0, 0, None),     # single token; F/64 ragged (5 row tiles per workgroup column)
    (40, 256, 352, 4, 2, 0, 0, 2),       # 40 tokens on each of 2 experts (3 token tiles); K = 352: ragged last chunk
    (100, 128, 224, 6, 3, 1, 160, 3),    # 100 tokens per expert (8 token tiles) + one shared expert
    (300, 128, 96, 4, 2, 2, 64, 2),      # 300 tokens per expert: more than one 128-token block; two shared experts
    (7, 64, 32, 3, 3, 0, 0, None),       # k = N, smallest allowed F
    (64, 2048, 768, 16, 8, 0, 0, None),  # Qwen3-like row / column sizes
    (96, 512, 128, 256, 8, 0, 0, None),  # very small experts, nearly all 256 invoked: thousands of short workgroups
    (72, 1024, 256, 200, 4, 1, 128, None),  # the same with a shared expert
    # shared experts 18-20 times wider than the routed ones: their down projection is cut into K slices of whole weight
    # tiles, and 8 slices of ceil(19 / 8) = 3 tiles would leave the last one empty (its output rows must not be summed)
    (31, 64, 32, 8, 2, 2, 608, None),
    (8, 64, 32, 8, 2, 1, 576, None),
    (70, 128, 64, 8, 2, 1, 1216, None),
    # token rows shorter than one staged chunk (H = 32 and 64 against chunks of 128 and 256 columns), experts with
    # more than 128 tokens (a second pass with few tokens): every load of a token row must stay inside the row
    (189, 32, 512, 13, 2, 0, 0, 3),
    (150, 64, 96, 5, 2, 1, 32, 2),
    # the last, partial round of gate/up workgroups is cut into workgroups of one row tile: all of them (48 live
    # workgroups), the 64 past a full round of 256 (40 experts x 8), with F / 16 no multiple of 4 (row tiles past the
    # last row), with crowded experts on the staged path among them, with a shared expert in front, and at most 16
    # tokens (gate/up and down as two launches); batches of at most 32 tokens, beyond which it is not done
    (32, 128, 128, 24, 4, 0, 0, None),
    (32, 64, 512, 40, 8, 0, 0, None),
    (31, 64, 96, 30, 5, 0, 0, None),
    (32, 64, 160, 20, 8, 0, 0, 10),
    (24, 128, 192, 28, 6, 1, 128, None),
    (12, 256, 224, 18, 3, 0, 0, None),
    (64, 64, 512, 40, 8, 0, 0, None),
    # down-projection work items of two and four 64-row units (many invoked experts x many row units), with crowded
    # experts cut into token blocks that go to workgroups of their own, direct and staged experts mixed
    (200, 1024, 128, 64, 8, 0, 0, None),
    (130, 512, 64, 48, 6, 1, 64, 20),
    (48, 768, 96, 100, 10, 0, 0, None),
    # beyond 64 tokens a down workgroup covers 128 rows and its waves walk two row tiles each: hidden sizes that are
    # no multiple of 128 (10 and 14 row tiles: the last workgroup of an expert has one and three waves with rows),
    # direct and staged experts mixed, with and without a shared expert
    (100, 160, 96, 6, 3, 0, 0, 3),
    (90, 224, 64, 5, 2, 1, 96, 2),
    (256, 96, 128, 12, 4, 0, 0, 5),
]


@pytest.mark.parametrize("T,H,F,N,k,S,Fs,hot", FFN_CASES)
def test_moe_ffn(L, T, H, F, N, k, S, Fs, hot):
    _say(f"moe_ffn T={T} H={H} F={F} N={N} k={k} shared={S}x{Fs} hot={hot}")
    e = _ffn_case(L, T, H, F, N, k, S, Fs, seed=T + F, hot=hot)
    _say(f"  max row rel err {e:.3e}")


def test_moe_ffn_many_small_experts_and_one_crowded(L):
    """Nearly all of 256 very small experts invoked (direct path, thousands of short workgroups in one launch) while
    one expert holds every token and takes the staged path."""
    rng = np.random.default_rng(21)
    T, H, F, N, k = 64, 512, 128, 256, 8
    _say(f"moe_ffn T={T} H={H} F={F} N={N} k={k}: expert 0 has all tokens")
    x = wl.f32_to_bf16_bits(rng.standard_normal((T, H)).astype(np.float32))
    Wg, Wu, Wd = wl.bf16_normal(rng, (N, F, H), 0.05), wl.bf16_normal(rng, (N, F, H), 0.05), wl.bf16_normal(rng, (N, H, F), 0.05)
    idx = np.stack([np.concatenate([[0], 1 + rng.permutation(N - 1)[:k - 1]]) for _ in range(T)]).astype(np.int32)
    gate = rng.random((T, k)).astype(np.float32) + 0.1
    gate /= gate.sum(1, keepdims=True)
    assert len(np.unique(idx)) > 200
    y_ref = oracle.moe_ffn(x, Wg, Wu, Wd, idx, gate.astype(np.float64))
    Wgu, Wdp = L.lynx_pack_weights(to_bf16_dev(Wg), to_bf16_dev(Wu), to_bf16_dev(Wd))
    p = L.lynx_permute(dev(idx), N)
    y = host(L.lynx_moe_ffn(to_bf16_dev(x), Wgu, Wdp, dev(idx), dev(gate), p, N, F))
    torch.cuda.synchronize()
    err = row_rel_err(y, y_ref)
    assert np.all(np.isfinite(y)) and err.max() <= Y_TOL, f"max row error {err.max():.3e}"


def test_a_failed_wait_shows_in_y_and_status(L):
    """The one hand-over inside a launch (a down-projection workgroup waits for its expert's gate/up workgroups) is
    bounded.  Forced from the host: a poll limit of 0 and a count the counters never reach make every such wait give
    up at once, while every kernel still runs to its end.  The call must then not pass a result on: y all NaN, status 1.
    With the knobs back at their defaults the same call gives status 0 and the right y."""
    from paper_2411_08982_amd import binding as B
    cfg = wl.CONFIGS["tiny"]
    T = 40                                         # more than 16 tokens, moderate experts: both projections in one launch
    assert L.lynx_moe_ffn_launches(T, cfg.F) == 1
    alpha, beta = wl.PRESETS["moderate"]
    d = wl.make_layer(cfg, T)
    x, Wr, bias = to_bf16_dev(d["x"]), dev(d["Wr"]), dev(d["bias"])
    Wgu, Wdp = L.lynx_pack_weights(to_bf16_dev(d["Wg"]), to_bf16_dev(d["Wu"]), to_bf16_dev(d["Wd"]))
    try:
        L.lynx_debug_set(B.DEBUG_SPIN_LIMIT, 0)
        L.lynx_debug_set(B.DEBUG_TARGET_BIAS, 1 << 20)
        _say("failed wait, forced from the host: whole layer")
        b = L.lynx_moe_layer(x, Wr, bias, Wgu, Wdp, cfg.F, cfg.k, alpha, beta, 1)
        torch.cuda.synchronize()
        assert int(host(b.status)[0]) == 1 and np.isnan(host(b.y)).all()
        assert int(host(b.workspace.view(torch.int32))[B.WAIT_FLAG_WORD]) != 0
        _say("failed wait, forced from the host: lynx_moe_ffn")
        p = dict(offsets=b.offsets, perm=b.perm, active=b.active, num_active=b.num_active_perm)
        st = torch.full((1,), -7, dtype=torch.int32, device="cuda")
        y = L.lynx_moe_ffn(x, Wgu, Wdp, b.new_idx, b.new_gate, p, cfg.N, cfg.F, status=st)
        torch.cuda.synchronize()
        assert int(host(st)[0]) == 1 and np.isnan(host(y)).all()
    finally:
        L.lynx_debug_set(B.DEBUG_SPIN_LIMIT, -1)
        L.lynx_debug_set(B.DEBUG_TARGET_BIAS, 0)
    _say("the same calls with the defaults")
    b = L.lynx_moe_layer(x, Wr, bias, Wgu, Wdp, cfg.F, cfg.k, alpha, beta, 1, buffers=b)
    st = torch.full((1,), -7, dtype=torch.int32, device="cuda")
    p = dict(offsets=b.offsets, perm=b.perm, active=b.active, num_active=b.num_active_perm)
    y = L.lynx_moe_ffn(x, Wgu, Wdp, b.new_idx, b.new_gate, p, cfg.N, cfg.F, status=st)
    torch.cuda.synchronize()
    assert int(host(b.status)[0]) == 0 and int(host(st)[0]) == 0
    a = oracle.affinity_bin(host(b.logits), oracle.topk(host(b.logits), cfg.k)["idx"], alpha, beta, 1)
    y_ref = oracle.moe_ffn(d["x"], d["Wg"], d["Wu"], d["Wd"], a["new_idx"], a["new_gate"])
    assert row_rel_err(host(b.y), y_ref).max() <= Y_TOL and np.array_equal(host(y), host(b.y))


def test_moe_ffn_skips_invalid_pairs_without_fault(L):
    # an index outside [0,N) is documented as "pair skipped": the call must stay in bounds and finite
    rng = np.random.default_rng(4)
    T, H, F, N, k = 8, 64, 64, 4, 2
    x = wl.f32_to_bf16_bits(rng.standard_normal((T, H)).astype(np.float32))
    Wg, Wu, Wd = wl.bf16_normal(rng, (N, F, H), 0.05), wl.bf16_normal(rng, (N, F, H), 0.05), wl.bf16_normal(rng, (N, H, F), 0.05)
    idx = np.stack([rng.permutation(N)[:k] for _ in range(T)]).astype(np.int32)
    gate = np.full((T, k), 0.5, np.float32)
    bad = idx.copy()
    bad[2, 1] = -1
    bad[5, 0] = N + 3
    Wgu, Wdp = L.lynx_pack_weights(to_bf16_dev(Wg), to_bf16_dev(Wu), to_bf16_dev(Wd))
    p = L.lynx_permute(dev(bad), N)
    y = host(L.lynx_moe_ffn(to_bf16_dev(x), Wgu, Wdp, dev(bad), dev(gate), p, N, F))
    torch.cuda.synchronize()
    assert np.all(np.isfinite(y))
    g2 = gate.astype(np.float64).copy()
    g2[2, 1] = 0.0
    g2[5, 0] = 0.0
    good = np.where((bad < 0) | (bad >= N), 0, bad)                     # zero gate: the stand-in expert does not matter
    y_ref = oracle.moe_ffn(x, Wg, Wu, Wd, good.astype(np.int32), g2)
    assert row_rel_err(y, y_ref).max() <= Y_TOL


# ------------------------------------------------------------------------------------------------ whole layer

def _check_indices_in_range(new_idx, perm, offs, T, N, k):
    assert new_idx.min() >= -1 and new_idx.max() < N
    assert np.all(np.diff(offs) >= 0) and offs[0] >= 0 and offs[N] <= T * k
    assert offs[N] == int((new_idx >= 0).sum())
    valid = perm[:offs[N]]
    assert len(set(valid.tolist())) == len(valid)
    assert valid.size == 0 or (valid.min() >= 0 and valid.max() < T * k)


@pytest.mark.parametrize("T,N,k", [(8, 12, 3), (40, 70, 6)])
def test_non_finite_inputs_stay_in_bounds(L, T, N, k):
    """Inputs are assumed finite; a token whose logits are not gets an undefined selection, but every index the
    calls produce stays in range (or is -1 = no expert), the permutation stays a permutation of the valid pairs, and
    the tokens with finite inputs still get finite outputs."""
    rng = np.random.default_rng(T)
    H, F = 64, 64
    _say(f"non-finite inputs T={T} N={N} k={k}")
    Wg, Wu, Wd = wl.bf16_normal(rng, (N, F, H), 0.05), wl.bf16_normal(rng, (N, F, H), 0.05), wl.bf16_normal(rng, (N, H, F), 0.05)
    Wgu, Wdp = L.lynx_pack_weights(to_bf16_dev(Wg), to_bf16_dev(Wu), to_bf16_dev(Wd))
    bad_tokens = [1, 2, 3, 4, 5]
    good = [t for t in range(T) if t not in bad_tokens]
    # (a) the binning call alone, valid picks, logits with NaN and infinities
    z = wl.make_logits(T, N, seed=T)
    z[1, :] = np.nan
    z[2, 3] = np.inf
    z[3, 0] = -np.inf
    z[4, ::2] = np.nan
    z[5, :] = np.inf
    idx = np.stack([rng.permutation(N)[:k] for _ in range(T)]).astype(np.int32)
    a = L.lynx_affinity_bin(dev(z), dev(idx), 2.0, 2, 1)
    p = L.lynx_permute(a["new_idx"], N)
    torch.cuda.synchronize()
    _check_indices_in_range(host(a["new_idx"]), host(p["perm"]), host(p["offsets"]), T, N, k)
    # (b) the whole layer with hidden states that are not finite for some tokens: their logits, picks and gates are
    # whatever they are; the rest of the batch is served
    x = rng.standard_normal((T, H)).astype(np.float32)
    x[1, :] = np.nan
    x[2, 7] = np.inf
    x[3, :] = -np.inf
    x[4, ::3] = np.nan
    x[5, 0] = np.inf
    x[5, 1] = -np.inf
    Wr = (rng.standard_normal((N, H)) / np.sqrt(H)).astype(np.float32)
    b = L.lynx_moe_layer(to_bf16_dev(wl.f32_to_bf16_bits(x)), dev(Wr), None, Wgu, Wdp, F, k, 2.0, 2, 1)
    torch.cuda.synchronize()
    _check_indices_in_range(host(b.new_idx), host(b.perm), host(b.offsets), T, N, k)
    assert np.all(np.isfinite(host(b.y)[good]))
    assert np.all(np.isfinite(host(b.logits)[good]))


def test_moe_ffn_over_expert_shards_sums_to_the_whole(L):
    """How the path shards by expert: every shard runs the permutation and the FFN over its own experts only, with
    the pairs of the other shards' experts marked invalid (documented as skipped), and the partial outputs add up to
    the layer output.  Here the shards run one after the other on the one GPU; the sum stands in for the all-reduce."""
    rng = np.random.default_rng(11)
    T, H, F, N, k, shards = 40, 256, 128, 16, 4, 4
    x = wl.f32_to_bf16_bits(rng.standard_normal((T, H)).astype(np.float32))
    Wg, Wu, Wd = wl.bf16_normal(rng, (N, F, H), 0.05), wl.bf16_normal(rng, (N, F, H), 0.05), wl.bf16_normal(rng, (N, H, F), 0.05)
    idx = np.stack([rng.permutation(N)[:k] for _ in range(T)]).astype(np.int32)
    gate = rng.random((T, k)).astype(np.float32) + 0.1
    gate /= gate.sum(1, keepdims=True)
    y_ref = oracle.moe_ffn(x, Wg, Wu, Wd, idx, gate.astype(np.float64))
    xd, gd = to_bf16_dev(x), dev(gate)
    per = N // shards
    total = np.zeros((T, H), np.float64)
    for s in range(shards):
        lo = s * per
        local = np.where((idx >= lo) & (idx < lo + per), idx - lo, -1).astype(np.int32)
        Wgu, Wdp = L.lynx_pack_weights(to_bf16_dev(Wg[lo:lo + per]), to_bf16_dev(Wu[lo:lo + per]), to_bf16_dev(Wd[lo:lo + per]))
        ld = dev(local)
        p = L.lynx_permute(ld, per)
        y = host(L.lynx_moe_ffn(xd, Wgu, Wdp, ld, gd, p, per, F))
        torch.cuda.synchronize()
        assert np.all(np.isfinite(y))
        assert int(host(p["offsets"])[per]) == int((local >= 0).sum())      # the shard took exactly its own pairs
        total += y
    assert row_rel_err(total, y_ref).max() <= Y_TOL


def _layer_case(L, cfg, T, alpha, beta, enable, data=None):
    d = data or wl.make_layer(cfg, T)
    x, Wr, bias = to_bf16_dev(d["x"]), dev(d["Wr"]), dev(d["bias"])
    Wgu, Wdp = L.lynx_pack_weights(to_bf16_dev(d["Wg"]), to_bf16_dev(d["Wu"]), to_bf16_dev(d["Wd"]))
    Sgu = Sdp = None
    if cfg.n_shared:
        Sgu, Sdp = L.lynx_pack_weights(to_bf16_dev(d["Sg"]), to_bf16_dev(d["Su"]), to_bf16_dev(d["Sd"]))
    b = L.lynx_moe_layer(x, Wr, bias, Wgu, Wdp, cfg.F, cfg.k, alpha, beta, enable, Sgu, Sdp, cfg.n_shared, cfg.F_shared)
    torch.cuda.synchronize()
    # router: logits against the oracle's own; everything downstream on the GPU's logits (identical on both sides)
    r = oracle.route(d["x"], d["Wr"], d["bias"], cfg.k)
    z = host(b.logits)
    assert np.all(np.abs(z - r["logits"]) <= LOGIT_TOL * np.maximum(1.0, np.abs(r["logits"])))
    tk = oracle.topk(z, cfg.k)
    assert np.array_equal(host(b.topk_idx), tk["idx"])
    a = oracle.affinity_bin(z, tk["idx"], alpha, beta, enable)
    for key, got in (("new_idx", b.new_idx), ("cnt_before", b.cnt_before), ("cnt_after", b.cnt_after),
                     ("bin_hist", b.bin_hist), ("num_active", b.num_active)):
        assert np.array_equal(host(got), a[key]), key
    np.testing.assert_allclose(host(b.new_gate), a["new_gate"], rtol=GATE_TOL, atol=1e-7)
    p = oracle.permute(a["new_idx"], cfg.N)
    for key, got in (("offsets", b.offsets), ("perm", b.perm), ("active", b.active), ("num_active", b.num_active_perm)):
        assert np.array_equal(host(got), p[key]), key
    y_ref = oracle.moe_ffn(d["x"], d["Wg"], d["Wu"], d["Wd"], a["new_idx"], a["new_gate"], d["Sg"], d["Su"], d["Sd"])
    err = row_rel_err(host(b.y), y_ref)
    assert err.max() <= Y_TOL, f"max row error {err.max():.3e}"
    return a["num_active"], err.max()


@pytest.mark.parametrize("preset,enable", [("moderate", 1), ("aggressive", 1), ("moderate", 0)])
def test_layer_tiny_config(L, preset, enable):
    cfg = wl.CONFIGS["tiny"]
    alpha, beta = wl.PRESETS[preset]
    na, err = _layer_case(L, cfg, 16, alpha, beta, enable)
    _say(f"tiny layer {preset} enable={enable}: invoked {na.tolist()}, max row err {err:.3e}")


@pytest.mark.parametrize("name,T", [("qwen15moe", 8), ("dsv2lite", 16)])
def test_layer_small_shared_expert_configs(L, name, T):
    # real row/column sizes of the shared-expert families with the expert count cut down so the oracle finishes in seconds
    import dataclasses
    cfg = dataclasses.replace(wl.CONFIGS[name], N=12)
    alpha, beta = wl.PRESETS["aggressive"]
    na, err = _layer_case(L, cfg, T, alpha, beta, 1)
    _say(f"{name}-shaped (N=12) layer T={T}: invoked {na.tolist()}, max row err {err:.3e}")


@pytest.mark.parametrize("name,T,preset", [("tiny", 16, "moderate"), ("tiny", 1, "aggressive"), ("tiny", 37, "aggressive")])
def test_fused_layer_equals_separate_calls(L, name, T, preset):
    # lynx_moe_layer issues fused launches; every output must be bit-identical to the four separate calls
    cfg = wl.CONFIGS[name]
    alpha, beta = wl.PRESETS[preset]
    d = wl.make_layer(cfg, T)
    x, Wr, bias = to_bf16_dev(d["x"]), dev(d["Wr"]), dev(d["bias"])
    Wgu, Wdp = L.lynx_pack_weights(to_bf16_dev(d["Wg"]), to_bf16_dev(d["Wu"]), to_bf16_dev(d["Wd"]))
    b = L.lynx_moe_layer(x, Wr, bias, Wgu, Wdp, cfg.F, cfg.k, alpha, beta, 1)
    r = L.lynx_route(x, Wr, bias, cfg.k)
    a = L.lynx_affinity_bin(r["logits"], r["idx"], alpha, beta, 1)
    p = L.lynx_permute(a["new_idx"], cfg.N)
    y = L.lynx_moe_ffn(x, Wgu, Wdp, a["new_idx"], a["new_gate"], p, cfg.N, cfg.F)
    torch.cuda.synchronize()
    pairs = [(b.logits, r["logits"]), (b.topk_idx, r["idx"]), (b.topk_gate, r["gate"]), (b.topk_psum, r["psum"]),
             (b.new_idx, a["new_idx"]), (b.new_gate, a["new_gate"]), (b.cnt_before, a["cnt_before"]),
             (b.cnt_after, a["cnt_after"]), (b.bin_hist, a["bin_hist"]), (b.num_active, a["num_active"]),
             (b.offsets, p["offsets"]), (b.perm, p["perm"]), (b.active, p["active"]), (b.num_active_perm, p["num_active"]),
             (b.y, y)]
    for i, (u, v) in enumerate(pairs):
        assert torch.equal(u, v), i


# At most 16 tokens: the single routing workgroup, with the logits in it on one side of its line and without on the other
# (products of four tokens 32768, experts per wave, 64 experts, one token), several tasks per wave, hidden sizes that leave
# lanes and whole column groups idle, experts past 64 and 128, as many picks as experts, group-limited and sigmoid-gated.
@pytest.mark.parametrize("H,N,k,T,gate_fn,groups", [
    (4096, 8, 2, 1, 0, (1, 1)), (4096, 8, 2, 4, 1, (4, 2)), (4096, 8, 2, 5, 0, (1, 1)), (4128, 8, 8, 3, 0, (1, 1)), (32, 5, 5, 16, 0, (1, 1)),
    (544, 60, 4, 1, 0, (1, 1)), (96, 64, 16, 1, 1, (1, 1)), (512, 12, 3, 16, 0, (3, 2)), (640, 12, 3, 13, 1, (3, 1)), (672, 13, 2, 16, 0, (1, 1)),
    (1056, 24, 6, 8, 0, (1, 1)), (64, 65, 7, 2, 0, (5, 3)), (128, 97, 9, 11, 0, (1, 1)), (64, 256, 8, 16, 1, (8, 4)), (64, 256, 16, 9, 0, (1, 1))])
@pytest.mark.parametrize("alpha,beta,enable", [(4.0, 1, 1), (1.5, 6, 1), (0.0, 6, 1), (2.0, 2, 0)])   # alpha = 0: all in bin 0
def test_small_layer_equals_separate_calls(L, H, N, k, T, gate_fn, groups, alpha, beta, enable):
    cfg = wl.MoEConfig("small", H, 64, N, k, 0, 0, 1.0, 0.5, 0.2, (T,), 7)
    d = wl.make_layer(cfg, T)
    x, Wr, bias = to_bf16_dev(d["x"]), dev(d["Wr"]), dev(d["bias"])
    Wgu, Wdp = L.lynx_pack_weights(to_bf16_dev(d["Wg"]), to_bf16_dev(d["Wu"]), to_bf16_dev(d["Wd"]))
    buf = L.LayerBuffers(T, H, cfg.F, N, k, beta)
    buf.workspace.fill_(0xFF)
    b = L.lynx_moe_layer_grouped(x, Wr, bias, Wgu, Wdp, cfg.F, k, *groups, alpha, beta, gate_fn, enable, buffers=buf)
    r = L.lynx_route_grouped(x, Wr, bias, k, *groups, gate_fn)
    if groups[0] == 1:
        a = (L.lynx_affinity_bin_sigmoid if gate_fn else L.lynx_affinity_bin)(r["logits"], r["idx"], alpha, beta, enable)
    else:
        a = L.lynx_affinity_bin_grouped(r["logits"], k, *groups, alpha, beta, gate_fn, enable)
    p = L.lynx_permute(a["new_idx"], N)
    y = L.lynx_moe_ffn(x, Wgu, Wdp, a["new_idx"], a["new_gate"], p, N, cfg.F)
    torch.cuda.synchronize()
    names = ["logits", "topk_idx", "topk_gate", "topk_psum", "new_idx", "new_gate", "new_psum", "cnt_before", "cnt_after", "bin_hist",
             "num_active", "offsets", "perm", "active", "num_active_perm", "y"]
    other = [r["logits"], r["idx"], r["gate"], r["psum"], a["new_idx"], a["new_gate"], a["new_psum"], a["cnt_before"], a["cnt_after"],
             a["bin_hist"], a["num_active"], p["offsets"], p["perm"], p["active"], p["num_active"], y]
    for n, v in zip(names, other):
        assert torch.equal(getattr(b, n), v), n
    if groups[0] == 1:   # the remap itself against the oracle (the separate calls share its kernel up to 16 tokens)
        z = host(r["logits"])
        ref = oracle.affinity_bin(z, host(r["idx"]), alpha, beta, enable)
        for n in ("new_idx", "cnt_before", "cnt_after", "bin_hist", "num_active"):
            assert np.array_equal(host(getattr(b, n)).ravel(), np.asarray(ref[n]).ravel()), n


def test_layer_zero_tokens(L):
    cfg = wl.CONFIGS["tiny"]
    d = wl.make_layer(cfg, 0)
    Wgu, Wdp = L.lynx_pack_weights(to_bf16_dev(d["Wg"]), to_bf16_dev(d["Wu"]), to_bf16_dev(d["Wd"]))
    x = torch.empty((0, cfg.H), dtype=torch.bfloat16, device="cuda")
    b = L.lynx_moe_layer(x, dev(d["Wr"]), dev(d["bias"]), Wgu, Wdp, cfg.F, cfg.k, 2.0, 2, 1)
    torch.cuda.synchronize()
    assert host(b.num_active).tolist() == [0, 0] and host(b.num_active_perm).tolist() == [0]
    assert np.all(host(b.offsets) == 0) and np.all(host(b.active) == -1)


# The logits of small and large batches come from different kernels; both add chains of H / 64 fp32 terms (64 of them per logit, then six
# levels of a tree).  With rounding errors of at most u = 2^-24 of the partial sum, uniform and independent, the i-th step of a chain of
# terms of variance s^2 adds i s^2 u^2 / 3: n^2 / 6 for a chain of n = H / 64, 64 times that over the H s^2 of a logit is H / 384;
# every level of the tree adds u^2 / 3.
@pytest.mark.parametrize("T,H,N", [(64, 512, 128), (130, 2048, 64), (64, 2048, 128), (48, 7168, 256), (129, 4096, 128), (200, 1056, 60),
                                   (64, 4096, 64),
                                   (129, 2048, 8), (1024, 2048, 9), (1024, 4096, 11), (1024, 4096, 12), (63, 4128, 128)])   # either side of the line
def test_rounding_error_of_the_logits(L, T, H, N):
    _say(f"logits against 64 bits T={T} H={H} N={N}")
    g = torch.Generator(device="cuda").manual_seed(H + N)
    x = torch.randn(T, H, device="cuda", generator=g).to(torch.bfloat16)
    Wr = torch.randn(N, H, device="cuda", generator=g)
    z = L.lynx_route(x, Wr, None, 1)["logits"]
    exact = x.double() @ Wr.double().T
    err = float((z.double() - exact).norm() / exact.norm())
    assert err <= 2.0 ** -24 * (H / 384 + 2) ** 0.5, f"{err:.3e}"
