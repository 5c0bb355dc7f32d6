"""The expert FFN with the tokens of every expert prescribed, so that each path of the weight-streaming kernel is met at the
edges of its tiles: token counts around the column tiles and token blocks, row counts and contraction lengths that leave
remainders, in the three weight formats, against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
import workloads as wl
from gpu_util import dev, host, planned_blocks, row_rel_err, to_bf16_dev, token_blocks

pytestmark = pytest.mark.gpu

Y_TOL = 1e-2   # per token row: bf16 operands, fp32 sums, the intermediate vector rounded to bf16 (2^-9 per element)


@pytest.fixture(scope="module")
def L():
    assert torch.cuda.is_available()
    import paper_2411_08982_amd as L
    L.lib()
    return L


def run_case(L, fmt, T, counts, H, F, S, Fs, spare=0, tok_block=None):
    print(f"ffn paths {fmt} T={T} counts={counts} spare={spare} H={H} F={F} shared={S}x{Fs}", flush=True)
    k = len(counts)
    N = k + spare      # experts that no token picks
    rng = np.random.default_rng([T, H, F, sum(counts)])
    idx = np.full((T, k), -1, np.int32)      # column e: the tokens of expert e; -1 is a skipped pair
    for e, c in enumerate(counts):
        idx[rng.permutation(T)[:c], e] = e
    gate = rng.uniform(0.1, 1.0, (T, k)).astype(np.float32)
    every = np.tile(np.arange(k, dtype=np.int32), (T, 1))   # the oracle takes no skipped pairs: weight 0 instead
    gate_ref = np.where(idx >= 0, gate, 0.0)
    x = wl.f32_to_bf16_bits(rng.standard_normal((T, H)).astype(np.float32))
    mk = lambda *shape: wl.f32_to_bf16_bits((rng.standard_normal(shape) * 0.05).astype(np.float32))
    W = [mk(N, F, H), mk(N, F, H), mk(N, H, F)]
    Sw = [mk(S, Fs, H), mk(S, Fs, H), mk(S, H, Fs)] if S else None
    idx_d = dev(idx)
    p = L.lynx_permute(idx_d, N)
    ws = L.new_workspace(T, H, F, N, k, S, Fs)
    ws.fill_(0xFF)
    y = torch.full((T, H), float("nan"), dtype=torch.float32, device="cuda")
    status = torch.full((1,), -1, dtype=torch.int32, device="cuda")
    if fmt == "bf16":
        ref = oracle.moe_ffn(x, *W, every, gate_ref, *(Sw or ()))
        Sgu, Sdp = L.lynx_pack_weights(*map(to_bf16_dev, Sw)) if S else (None, None)
        L.lynx_moe_ffn(to_bf16_dev(x), *L.lynx_pack_weights(*map(to_bf16_dev, W)), idx_d, dev(gate), p, N, F, Sgu, Sdp, S, Fs,
                       workspace=ws, y=y, status=status)
    else:
        quantize, ffn, oq, offn = {
            "fp8": (L.lynx_quantize_weights_fp8, L.lynx_moe_ffn_fp8, oracle.quantize_rows_e4m3, oracle.moe_ffn_q8),
            "fp4": (L.lynx_quantize_weights_fp4, L.lynx_moe_ffn_fp4, oracle.quantize_mxfp4, oracle.moe_ffn_q4),
        }[fmt]
        codes, scales = zip(*(oq(w) for w in W))
        extra = ()
        if S:
            scodes, sscales = zip(*(oq(w) for w in Sw))
            extra = (*scodes, *sscales)
        ref = offn(x, *codes, *scales, every, gate_ref, *extra)
        ffn(to_bf16_dev(x), quantize(*map(to_bf16_dev, W)), idx_d, dev(gate), p, N, F,
            quantize(*map(to_bf16_dev, Sw)) if S else None, S, Fs, workspace=ws, y=y, status=status)
    torch.cuda.synchronize()
    got = host(y)
    assert host(status)[0] == 0
    assert tok_block is None or planned_blocks(ws) == token_blocks(counts, tok_block)
    assert np.all(np.isfinite(got))
    err = row_rel_err(got, ref).max()
    assert err <= Y_TOL, f"max row error {err:.3e}"


# More than 64 tokens.  With more than 64 per expert on average a gate/up unit is 128 rows and a wave owns two row tiles of
# it: row counts of 128 n + 32, 64 and 96 leave it a partly filled last unit.  Contraction lengths that end inside a chunk of
# the token stage and inside a turn of the weight ring.
LARGE = [
    # T, tokens per expert, H, F, shared experts, their width
    (65, (65, 64, 63, 33, 1), 256, 128, 0, 0),
    (130, (130, 129, 128, 127, 17), 384, 640, 0, 0),       # blocks of one expert: a full one and a remainder of 1 or 2
    (300, (300, 256, 257, 16, 32), 128, 384, 1, 256),      # 3 blocks (5 of 64); a shared expert over all tokens
    (97, (97, 0, 81, 5, 49), 512, 256, 1, 768),            # an expert that is not invoked; a wide shared expert (K slices)
    (80, (3, 20, 0, 33, 65), 640, 384, 0, 0),
]
# few tokens per expert on average (the unused experts count): units of 64 rows for every format
SPARSE = [(130, (130, 20, 65, 5), 384, 640, 1, 128, 8), (90, (17, 90, 33, 64, 1), 256, 256, 0, 0, 20)]
# More than eight experts: undivided K in the down projection for every format.  First with more than 64 tokens per expert on
# average; then with 32 to 64, where 128-row gate/up units begin for MXFP4 (experts times F past 32768) and not yet for
# bf16 and FP8, and just below each of the two lines.
MANY = [
    (90, (90, 88, 65, 64, 63, 33, 17, 16, 1), 384, 256, 1, 256, 0),
    (130, (130, 129, 128, 70, 66, 65, 64, 5, 2), 256, 640, 0, 0, 0),
    (130, (130, 20, 65, 5), 384, 2816, 1, 128, 8),        # 43 tokens per expert, 12 x 2816
    (130, (130, 66, 17, 64), 256, 2688, 0, 0, 8),         # 12 x 2688: too few rows
    (94, (94, 33, 64, 16), 256, 2816, 0, 0, 8),           # 31 tokens per expert
]
RAGGED = {"bf16": (32, 96), "fp8": (64, 64), "fp4": (0, 0)}   # added to H and F: the format's smallest steps


@pytest.mark.parametrize("fmt", ["bf16", "fp8", "fp4"])
@pytest.mark.parametrize("case", LARGE + SPARSE + MANY)
def test_large_batches(L, fmt, case):
    T, counts, H, F, S, Fs, *spare = case
    dH, dF = RAGGED[fmt]
    run_case(L, fmt, T, counts, H + dH, F + dF, S, Fs, *spare)


# At most 16 tokens per expert: 1, 2, 4, 8 or 16 token rows in LDS, as many columns at a time as fit (contractions that need
# one chunk, several, and a remainder), K in one, two and four slices with short or empty last ones, a shared expert beside it.
SMALL = [
    # T, tokens per expert, H, F, shared experts, their width
    (1, (1, 0, 1), 128, 256, 0, 0),
    (2, (2, 1), 2048, 384, 1, 128),
    (5, (5, 3, 1, 0, 2), 640, 2048, 0, 0),
    (8, (8, 7, 1, 3), 8192, 256, 1, 640),                      # gate/up in several chunks
    (8, (8, 4, 1, 2), 256, 16384, 0, 0),                       # down: four slices, several chunks each
    (11, (11, 9, 8, 2, 1, 4, 0, 6, 3, 5, 7), 1152, 1024, 2, 128),
    (16, (16, 15, 9, 1), 2176, 4096, 0, 0),
    (23, (16, 17, 1, 23, 8), 4096, 640, 0, 0),                 # both paths in one launch
    (90, (16, 13, 66, 3, 90, 81, 80), 384, 256, 0, 0),         # the same in the kernel for large batches, units of 128 rows
]


@pytest.mark.parametrize("fmt", ["bf16", "fp8", "fp4"])
@pytest.mark.parametrize("case", SMALL)
def test_few_tokens_per_expert(L, fmt, case):
    T, counts, H, F, S, Fs = case
    dH, dF = RAGGED[fmt]
    run_case(L, fmt, T, counts, H + dH, F + dF, S, Fs)


# An infinity in the last columns of a token row (of x, or of the intermediate vector, which can overflow bf16) is part of
# the token's sums and of nothing else.  The contractions end inside a chunk of the token stage: what the stage holds past
# the end meets weights that read as zero, and has to be zero itself (zero times infinity is NaN).
@pytest.mark.parametrize("where", ["x", "h"])
@pytest.mark.parametrize("fmt,H,F", [("bf16", 288, 416), ("fp8", 320, 448), ("fp4", 384, 640)])
@pytest.mark.parametrize("T,counts", [(40, (40, 17, 3)), (130, (130, 70, 65, 20, 8)), (70, (20, 33, 64))])
def test_infinity_past_a_ragged_contraction(L, fmt, H, F, T, counts, where):
    print(f"ffn infinity {fmt} T={T} counts={counts} H={H} F={F} in {where}", flush=True)
    k = N = len(counts)
    rng = np.random.default_rng([T, H, F])
    idx = np.full((T, k), -1, np.int32)
    for e, c in enumerate(counts):
        idx[rng.permutation(T)[:c], e] = e
    gate = rng.uniform(0.1, 1.0, (T, k)).astype(np.float32)
    # all positive: a sum with an infinity in it is +Inf, whatever the order
    pos = lambda *shape: np.abs(rng.standard_normal(shape)).astype(np.float32) * 0.02 + 0.05   # (no code of theirs is zero)
    x, Wg, Wu, Wd = pos(T, H), pos(N, F, H), pos(N, F, H), pos(N, H, F)
    if where == "x":
        hit = rng.permutation(T)[:T // 3]
        x[hit[:, None], H - 1 - rng.integers(0, 8, (hit.size, 1))] = np.inf
    else:
        hit = np.arange(T)
        Wg[:, F - 3] *= 1e21
        Wu[:, F - 3] *= 1e21
    hit = np.isin(np.arange(T), hit) & (idx >= 0).any(axis=1)
    W = [wl.f32_to_bf16_bits(w) for w in (Wg, Wu, Wd)]
    x = wl.f32_to_bf16_bits(x)
    idx_d = dev(idx)
    p = L.lynx_permute(idx_d, N)
    if fmt == "bf16":
        y = L.lynx_moe_ffn(to_bf16_dev(x), *L.lynx_pack_weights(*map(to_bf16_dev, W)), idx_d, dev(gate), p, N, F)
    else:
        quantize, ffn = {"fp8": (L.lynx_quantize_weights_fp8, L.lynx_moe_ffn_fp8),
                         "fp4": (L.lynx_quantize_weights_fp4, L.lynx_moe_ffn_fp4)}[fmt]
        y = ffn(to_bf16_dev(x), quantize(*map(to_bf16_dev, W)), idx_d, dev(gate), p, N, F)
    torch.cuda.synchronize()
    y = host(y)
    assert np.all(np.isposinf(y[hit])) and np.all(np.isfinite(y[~hit]))


# An engine's own assignment may send a token to one expert more than once (lynx_permute makes none such): more rows than
# tokens, in kernels that are chosen by the number of tokens.  F is long enough for four K slices in the down projection.
# (H = 160: the last 64-row unit of the staged path is shared by two down workgroups of which only one exists.)
@pytest.mark.parametrize("fmt,H,F", [("bf16", 256, 2048), ("bf16", 160, 2048), ("fp8", 256, 4096), ("fp4", 256, 8192)])
@pytest.mark.parametrize("T,per_expert", [(8, (4, 20, 0)), (8, (16, 0)), (7, (12, 2)), (8, (9, 7)), (5, (1, 9)), (8, (13, 11, 0)),
                                          (16, (121, 1, 1, 1, 1, 1, 1, 1))])   # (one token block more than experts)
def test_more_rows_than_tokens(L, fmt, H, F, T, per_expert):
    print(f"ffn rows {fmt} T={T} rows={per_expert} H={H} F={F}", flush=True)
    N, P = len(per_expert), sum(per_expert)
    k = P // T
    assert P == T * k
    rng = np.random.default_rng([T, H, F, *per_expert])
    flat = rng.permutation(np.repeat(np.arange(N, dtype=np.int32), per_expert))
    idx = flat.reshape(T, k)
    gate = rng.uniform(0.1, 1.0, (T, k)).astype(np.float32)
    x = wl.f32_to_bf16_bits(rng.standard_normal((T, H)).astype(np.float32))
    mk = lambda *shape: wl.f32_to_bf16_bits((rng.standard_normal(shape) * 0.05).astype(np.float32))
    W = [mk(N, F, H), mk(N, F, H), mk(N, H, F)]
    p = dict(offsets=dev(np.concatenate([[0], np.cumsum(per_expert)]).astype(np.int32)),
             perm=dev(np.argsort(flat, kind="stable").astype(np.int32)),
             active=dev(np.arange(N, dtype=np.int32)), num_active=dev(np.array([N], np.int32)))
    ws = L.new_workspace(T, H, F, N, k)
    ws.fill_(0xFF)
    # the oracle takes distinct experts per token: slot by slot
    by_slot = lambda f: sum(f(np.ascontiguousarray(idx[:, j:j + 1]), np.ascontiguousarray(gate[:, j:j + 1])) for j in range(k))
    if fmt == "bf16":
        ref = by_slot(lambda i, g: oracle.moe_ffn(x, *W, i, g))
        y = L.lynx_moe_ffn(to_bf16_dev(x), *L.lynx_pack_weights(*map(to_bf16_dev, W)), dev(idx), dev(gate), p, N, F,
                           workspace=ws)
    else:
        quantize, ffn, oq, offn = {
            "fp8": (L.lynx_quantize_weights_fp8, L.lynx_moe_ffn_fp8, oracle.quantize_rows_e4m3, oracle.moe_ffn_q8),
            "fp4": (L.lynx_quantize_weights_fp4, L.lynx_moe_ffn_fp4, oracle.quantize_mxfp4, oracle.moe_ffn_q4),
        }[fmt]
        codes, scales = zip(*(oq(w) for w in W))
        ref = by_slot(lambda i, g: offn(x, *codes, *scales, i, g))
        y = ffn(to_bf16_dev(x), quantize(*map(to_bf16_dev, W)), dev(idx), dev(gate), p, N, F, workspace=ws)
    torch.cuda.synchronize()
    assert np.all(np.isfinite(host(y)))
    err = row_rel_err(host(y), ref).max()
    assert err <= Y_TOL, f"max row error {err:.3e}"


# The K slices of a down workgroup as the knob sets them, where the library's rule would choose another number.
@pytest.mark.parametrize("fmt", ["bf16", "fp8", "fp4"])
@pytest.mark.parametrize("slices,case", [(4, (16, (16, 15, 9, 1), 384, 1024, 1, 640)), (4, (11, (11, 8, 3), 256, 4096, 0, 0)),
                                         (1, (8, (8, 5), 256, 2048, 1, 128)), (2, (130, (130, 77, 40, 12), 384, 640, 1, 256)),
                                         (1, (97, (97, 81, 5), 512, 256, 0, 0))])
def test_k_slices_set_by_the_knob(L, fmt, slices, case):
    from paper_2411_08982_amd import binding as B
    T, counts, H, F, S, Fs = case
    dH, dF = RAGGED[fmt]
    L.lynx_debug_set(B.DEBUG_DOWN_K_WAVES, slices)
    try:
        run_case(L, fmt, T, counts, H + dH, F + dF, S, Fs)
    finally:
        L.lynx_debug_set(B.DEBUG_DOWN_K_WAVES, 0)


# The kernel for token blocks of 256, set by its knob: passes of up to 64, 128, 192 and 256 tokens at their edges, several blocks, one
# token, an expert that is not invoked; contractions of one k-step, an odd number of them, and ends inside a turn of four; rows that
# leave waves and row tiles without work; shared experts with K slices; one launch with waits and (F past 4096) two.
WIDE = [
    (257, (257, 256, 255, 193, 1), 256, 512, 0, 0),
    (192, (192, 129, 128, 65, 64), 288, 352, 1, 384),
    (66, (66, 0, 1, 33), 32, 64, 0, 0),
    (600, (600, 513, 512, 31), 160, 96, 1, 1024),
    (130, (130, 97), 1056, 4128, 0, 0),
    (65, (17, 16), 64, 4384, 1, 4384),
    (1024, (1024, 700), 512, 640, 2, 320),
]


@pytest.mark.parametrize("case", WIDE)
def test_wide_kernel(L, case):
    from paper_2411_08982_amd import binding as B
    L.lynx_debug_set(B.DEBUG_WIDE_KERNEL, 1)
    try:
        run_case(L, "bf16", *case, tok_block=256)
    finally:
        L.lynx_debug_set(B.DEBUG_WIDE_KERNEL, 0)
    T, counts, *_ = case
    assert max(counts) <= 128 or token_blocks(counts, 256) < token_blocks(counts, 128)   # (the plan tells the kernels apart)


# The results for quantised experts past 4096 columns where one launch begins (8 to 64 tokens, 512 down workgroups of 32 rows) and
# just short of it (7 tokens; H = 1920: 480): direct and staged experts.  How many launches there are shows in the next test.
@pytest.mark.parametrize("fmt,T,H,F", [("fp8", 7, 2048, 4160), ("fp8", 8, 1920, 4160), ("fp8", 8, 2048, 4160), ("fp4", 8, 2048, 4224),
                                       ("fp8", 64, 4096, 4160)])
def test_huge_quantised_experts_in_one_launch(L, fmt, T, H, F):
    run_case(L, fmt, T, tuple(min(T, c) for c in (64, 20, 8, 7, 5, 3, 2, 1)), H, F, 0, 0)


# Which launch the down workgroups of huge quantised experts run in.  A poll limit of zero and a count that is never reached make
# every wait give up at once: status 1 where they are in the launch of the gate/up workgroups and wait for them, 0 where they
# follow it.  64-row workgroups (H / 64 per expert) fill the chip from 384 on, 32-row ones (8 tokens, FP8) from 512; the live count
# decides where k experts are too few and N are enough.
@pytest.mark.parametrize("fmt,T,H,F,N,k,live,waits", [
    ("fp8", 16, 4096, 4160, 8, 2, 6, 1), ("fp8", 16, 4096, 4160, 8, 2, 5, 0), ("fp4", 64, 4096, 4224, 8, 2, 6, 1),
    ("fp4", 64, 4096, 4224, 8, 2, 5, 0), ("fp8", 8, 4096, 4160, 8, 2, 4, 1), ("fp8", 8, 4096, 4160, 8, 2, 3, 0),
    ("fp8", 7, 4096, 4160, 8, 2, 8, 0), ("fp8", 65, 4096, 4160, 8, 2, 8, 0),      # outside the batch sizes of the rule
    ("fp8", 16, 4096, 4160, 6, 2, 6, 1), ("fp8", 16, 4032, 4160, 6, 2, 6, 0),     # N experts are just enough, and not (63 rows of 64)
    ("fp8", 16, 4096, 4160, 8, 6, 6, 1),                                          # k experts are enough: always one launch
    ("bf16", 16, 4096, 4128, 8, 2, 8, 0),
])
def test_launches_of_huge_quantised_experts(L, fmt, T, H, F, N, k, live, waits):
    from paper_2411_08982_amd import binding as B
    print(f"ffn launches {fmt} T={T} H={H} F={F} N={N} k={k} live={live}", flush=True)
    rng = np.random.default_rng([T, H, F, live])
    names = rng.permutation(N)[:live]
    idx = dev(np.stack([np.roll(names, t)[:k] for t in range(T)]).astype(np.int32))     # every one of them is picked
    gate = dev(rng.uniform(0.1, 1.0, (T, k)).astype(np.float32))
    gen = torch.Generator(device="cuda").manual_seed(T * live)
    mk = lambda *shape: torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(0.0, 0.05, generator=gen)
    pack, ffn = {"bf16": (L.lynx_pack_weights, L.lynx_moe_ffn), "fp8": (L.lynx_quantize_weights_fp8, L.lynx_moe_ffn_fp8),
                 "fp4": (L.lynx_quantize_weights_fp4, L.lynx_moe_ffn_fp4)}[fmt]
    W = pack(mk(N, F, H), mk(N, F, H), mk(N, H, F))
    W = tuple(W) if fmt == "bf16" else (W,)
    x = mk(T, H)
    p = L.lynx_permute(idx, N)
    ws = L.new_workspace(T, H, F, N, k)
    status = torch.full((1,), -1, dtype=torch.int32, device="cuda")
    call = lambda x: host(ffn(x, *W, idx, gate, p, N, F, workspace=ws.fill_(0xFF), status=status))
    y = call(x)
    assert host(status)[0] == 0 and np.all(np.isfinite(y)) and np.any(y)
    odd = torch.empty(T * H + 8, dtype=torch.bfloat16, device="cuda")[1:1 + T * H].view(T, H)   # always two launches
    odd.copy_(x)
    assert np.array_equal(call(odd), y)
    try:
        L.lynx_debug_set(B.DEBUG_SPIN_LIMIT, 0)
        L.lynx_debug_set(B.DEBUG_TARGET_BIAS, 1 << 20)
        call(x)
    finally:
        L.lynx_debug_set(B.DEBUG_SPIN_LIMIT, -1)
        L.lynx_debug_set(B.DEBUG_TARGET_BIAS, 0)
    assert host(status)[0] == waits


def test_overlapping_expert_ranges_stay_inside_the_plan(L):
    """expert_offsets that lynx_permute cannot have written: every second expert claims all pairs, which makes more token
    blocks than the work plan has records, and the last expert, behind them, a few (its pair ids would be filed).  What
    the plan does not hold is not computed; nothing may be written past its tables."""
    T, k, N, H, F = 64, 16, 140, 32, 4128             # F: two launches, no waits for blocks that the plan leaves out
    P = T * k
    print(f"ffn overlapping ranges T={T} k={k} N={N}", flush=True)
    assert L.lynx_moe_ffn_launches(T, F) == 2
    offsets = np.zeros(N + 1, np.int32)
    offsets[1:138:2] = P                              # 69 experts of 16 blocks: 1104 blocks, the plan holds 512
    offsets[138:] = [0, 0, 9]
    W = [torch.zeros(s, dtype=torch.bfloat16, device="cuda") for s in ((N, F, H), (N, F, H), (N, H, F))]
    idx = dev(np.tile(np.arange(k, dtype=np.int32), (T, 1)))
    p = dict(offsets=dev(offsets), perm=dev(np.arange(P, dtype=np.int32)), active=dev(np.arange(N, dtype=np.int32)),
             num_active=dev(np.array([N], np.int32)))
    ws = L.new_workspace(T, H, F, N, k)
    ws.fill_(0xFF)
    gate = torch.ones((T, k), dtype=torch.float32, device="cuda")
    L.lynx_moe_ffn(torch.ones((T, H), dtype=torch.bfloat16, device="cuda"), *L.lynx_pack_weights(*W), idx, gate, p, N, F,
                   workspace=ws)
    torch.cuda.synchronize()
    # words 20032 to 22080: the counters of shared experts, of which there are none
    assert np.all(host(ws.view(torch.int32))[20032:22080] == -1)


@pytest.mark.parametrize("fmt,H,F", [("bf16", 64, 128), ("fp8", 2048, 4160), ("fp4", 2048, 4224)])
def test_overlapping_expert_ranges_leave_nothing_to_wait_for(L, fmt, H, F):
    """Overlapping ranges with more token blocks (15 + 16 + 16) than the grid has workgroups for (32), where both projections
    are one launch: the third expert is left out whole, and no down workgroup waits for reports of blocks that do not exist.  All
    experts have the same weights and the second one holds every pair, so y is that of any valid assignment."""
    T = 64
    k = N = 16
    P = T * k
    print(f"ffn overlapping ranges, one launch: {fmt} T={T} k={k} N={N} H={H} F={F}", flush=True)
    rng = np.random.default_rng([H, F])
    mk = lambda *shape: to_bf16_dev(wl.f32_to_bf16_bits((rng.standard_normal(shape) * 0.05).astype(np.float32))).expand(N, -1, -1).contiguous()
    pack, ffn = {"bf16": (L.lynx_pack_weights, L.lynx_moe_ffn), "fp8": (L.lynx_quantize_weights_fp8, L.lynx_moe_ffn_fp8),
                 "fp4": (L.lynx_quantize_weights_fp4, L.lynx_moe_ffn_fp4)}[fmt]
    W = pack(mk(1, F, H), mk(1, F, H), mk(1, H, F))
    W = tuple(W) if fmt == "bf16" else (W,)
    x = to_bf16_dev(wl.f32_to_bf16_bits(rng.standard_normal((T, H)).astype(np.float32)))
    idx = dev(np.tile(np.arange(N, dtype=np.int32), (T, 1)))
    gate = dev(rng.uniform(0.1, 1.0, (T, k)).astype(np.float32))
    want = host(ffn(x, *W, idx, gate, L.lynx_permute(idx, N), N, F))
    offsets = np.array([0, 960] + [0, P] * 7 + [0], np.int32)      # experts 0, 2, 4, ...: [0, 960), then all pairs
    p = dict(offsets=dev(offsets), perm=dev(np.arange(P, dtype=np.int32)), active=dev(np.arange(N, dtype=np.int32)),
             num_active=dev(np.array([N], np.int32)))
    ws = L.new_workspace(T, H, F, N, k)
    ws.fill_(0xFF)
    status = torch.full((1,), -1, dtype=torch.int32, device="cuda")
    y = host(ffn(x, *W, idx, gate, p, N, F, workspace=ws, status=status))
    assert host(status)[0] == 0
    words = host(ws.view(torch.int32))
    assert list(words[9760:9763]) == [31, 1, 2]      # the plan's header: blocks, units per item, experts
    assert np.all(np.isfinite(y)) and row_rel_err(y, want).max() <= Y_TOL


@pytest.mark.parametrize("fmt", ["bf16", "fp8", "fp4"])
@pytest.mark.parametrize("T,counts,S", [(40, (40, 33, 9, 1), 1), (130, (130, 100, 20), 0), (7, (7, 3), 1)])
def test_token_rows_at_odd_places(L, fmt, T, counts, S):
    """x is a contiguous tensor that starts one, two or four elements into its storage: the same result, bit for bit."""
    H, F, N, k = 384, 256, len(counts), len(counts)
    print(f"ffn odd places {fmt} T={T} counts={counts}", flush=True)
    rng = np.random.default_rng([T, H, F])
    idx = np.full((T, k), -1, np.int32)
    for e, c in enumerate(counts):
        idx[rng.permutation(T)[:c], e] = e
    gate = dev(rng.uniform(0.1, 1.0, (T, k)).astype(np.float32))
    mk = lambda *shape: to_bf16_dev(wl.f32_to_bf16_bits((rng.standard_normal(shape) * 0.05).astype(np.float32)))
    pack, ffn = {"bf16": (L.lynx_pack_weights, L.lynx_moe_ffn), "fp8": (L.lynx_quantize_weights_fp8, L.lynx_moe_ffn_fp8),
                 "fp4": (L.lynx_quantize_weights_fp4, L.lynx_moe_ffn_fp4)}[fmt]
    W = pack(mk(N, F, H), mk(N, F, H), mk(N, H, F))
    Sw = pack(mk(S, F, H), mk(S, F, H), mk(S, H, F)) if S else None
    weights = lambda w: tuple(w) if fmt == "bf16" else (w,)
    idx_d = dev(idx)
    p = L.lynx_permute(idx_d, N)
    shared = (weights(Sw) if S else weights(None if fmt != "bf16" else (None, None))) + (S, F if S else 0)
    x = to_bf16_dev(wl.f32_to_bf16_bits(rng.standard_normal((T, H)).astype(np.float32)))
    want = host(ffn(x, *weights(W), idx_d, gate, p, N, F, *shared))
    assert np.all(np.isfinite(want)) and np.any(want)
    for off in (1, 2, 4):
        room = torch.empty(T * H + 8, dtype=torch.bfloat16, device="cuda")
        odd = room[off:off + T * H].view(T, H)
        odd.copy_(x)
        assert odd.is_contiguous() and odd.data_ptr() % 16 == 2 * off
        got = host(ffn(odd, *weights(W), idx_d, gate, p, N, F, *shared))
        assert np.array_equal(got, want), off
