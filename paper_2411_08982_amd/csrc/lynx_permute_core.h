// Token assignment from per-expert token bit sets (paper Sec. 4: the remapper hands every expert its tokens), shared by the
// stand-alone lynx_permute kernel and by the last workgroup of the fused remap kernel.
//
// A token holds k distinct experts, so an expert sees a token at most once: the membership of the batch
// in each expert is a T-bit set.  Pair counts are popcounts, and the stable position of pair (t, slot)
// inside its expert is the popcount of the bits below t.  No sort, no ordered atomics.
#pragma once

#include "lynx_plan.h"

namespace lynx {

template <int MAXW>   // capacity in 32-token words per expert
struct PermuteSharedT {
    unsigned member[LYNX_MAX_N * MAXW];   // member[e*W + w] bit b: token 32*w+b uses expert e
    uint16_t before[LYNX_MAX_N * MAXW];   // before[e*W + w] = tokens of expert e in the words below w
    int count[LYNX_MAX_N];
    uint2 place[LYNX_MAX_N];              // x: where the expert's pairs start; y: its block in the FFN's work plan, -1 = files no pair ids
    int invoked, pairs;
};
typedef PermuteSharedT<LYNX_MAX_T / 32> PermuteShared;

// Every thread of the workgroup calls this with sh.member filled (and visible: barrier before).
// With ps.units_gu > 0 it also writes the
// work plan of the expert FFN into the workspace ws (lynx_plan.h).
template <int THREADS, typename Shared>
__device__ __forceinline__ void permute_from_bitsets(Shared &sh, const int32_t *__restrict__ idx, int T, int N,
                                                     int k, int32_t *__restrict__ expert_offsets,
                                                     int32_t *__restrict__ perm, int32_t *__restrict__ active_experts,
                                                     int32_t *__restrict__ num_active, const PlanShape &ps = PlanShape{0, 0, 0, 0, 0},
                                                     int32_t *__restrict__ ws = nullptr)
{
    const int tid = threadIdx.x;
    const int W = (T + 31) / 32;
    const int P = T * k;
    if (tid < N) {
        int c = 0;
        for (int w = 0; w < W; ++w) {
            sh.before[tid * W + w] = (uint16_t)c;
            c += __popc(sh.member[tid * W + w]);
        }
        sh.count[tid] = c;
    }
    __syncthreads();
    // One wave: exclusive prefixes over the experts.  Pair offsets and rank among the invoked experts in one scan (the pair
    // count of the whole batch is at most LYNX_MAX_T * LYNX_MAX_K < 2^16: it leaves the upper half to the ranks), token blocks
    // in a second one beside it; and what follows from them alone.  (Two passes of one scan each with a barrier between them,
    // the lists written by everybody at the end, five reads of LDS per pair instead of three, and in remap_kernel the gates
    // ahead of the hand-over: that kernel 8.5 -> 7.9 us at 32 tokens and 128 experts, 15.1 -> 13.8 at 512 tokens.)
    static_assert(LYNX_MAX_T * LYNX_MAX_K < 65536 && LYNX_MAX_N < 32768, "packed prefix sums");
    if (tid < kWave) {
        const bool plan = ps.units_gu > 0;
        int carry_o = 0, carry_a = 0, carry_b = 0;
        for (int base = 0; base < N; base += kWave) {
            const int e = base + tid;
            const int c = (e < N) ? sh.count[e] : 0;
            const int a = c > 0 ? 1 : 0;
            const int nb = plan && a ? plan_token_blocks(c, ps.tok_block) : 0;
            const int s = wave_prefix_sum_i32(c | (a << 16));
            const int sb = wave_prefix_sum_i32(nb);
            const int off = carry_o + (s & 0xffff) - c, q0 = carry_b + sb - nb;
            if (e < N) {
                sh.place[e] = make_uint2((unsigned)off, plan && c <= kDirectMaxTokens && q0 < kPlanMaxBlocks ? (unsigned)q0 : ~0u);
                expert_offsets[e] = off;
            }
            if (a) active_experts[carry_a + (s >> 16) - a] = e;
            if (nb > 0) plan_write_records(e, c, off, q0, nb, ws);
            const int total = __builtin_amdgcn_readlane(s, kWave - 1);
            carry_o += total & 0xffff;
            carry_a += total >> 16;
            carry_b += __builtin_amdgcn_readlane(sb, kWave - 1);
        }
        if (tid == 0) {
            expert_offsets[N] = carry_o;
            num_active[0] = carry_a;
            sh.invoked = carry_a;
            sh.pairs = carry_o;
            if (plan) plan_write_header(ps, carry_b, carry_a, ws);
        }
    }
    __syncthreads();
    // (the indices are read with device-coherent loads: in the fused kernel another workgroup of this launch
    // wrote them; such loads go to memory, so several are requested before the first is used)
    constexpr int kBatch = 8;
    const unsigned inv = 0xffffffffu / (unsigned)k + 1u;   // p / k = high word of p * inv, for p < 2^16 and k > 1
    uint16_t *pairs = ps.units_gu > 0 ? reinterpret_cast<uint16_t *>(ws + kWsPlanPairs) : nullptr;
    for (int p0 = tid; p0 < P; p0 += THREADS * kBatch) {
        int ev[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const int p = p0 + u * THREADS;
            ev[u] = p < P ? load_coherent(idx + p) : -1;
        }
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const int p = p0 + u * THREADS, e = ev[u];
            if (e < 0 || e >= N) continue;
            const int t = k > 1 ? (int)__umulhi((unsigned)p, inv) : p;
            const int wt = t >> 5;
            const uint2 place = sh.place[e];
            const int i = sh.before[e * W + wt] + __popc(sh.member[e * W + wt] & ((1u << (t & 31)) - 1u));
            perm[(int)place.x + i] = p;   // < the pair count <= P by construction
            if (place.y != ~0u) pairs[place.y * kDirectMaxTokens + i] = (uint16_t)p;
        }
    }
    for (int e = sh.invoked + tid; e < N; e += THREADS) active_experts[e] = -1;
    for (int p = sh.pairs + tid; p < P; p += THREADS) perm[p] = -1;   // pairs whose expert is invalid stay unassigned
}

}  // namespace lynx
