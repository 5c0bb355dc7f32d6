// The device-built work plan of the grouped expert FFN.
//
// The number of experts a batch invokes after the remap, and how many tokens each of them got, are device-side
// values (paper Sec. 4: the remapper compacts the active list and hands every expert its tokens; Sec. 5.9 names the
// dispatch parameters for a variable number of activated experts as the open tuning point).  The host sizes the FFN
// grid for the most work the batch could cause; which workgroup does what is decided on the device from three small
// tables in the workspace that the token assignment writes as its last step:
//   hdr     [0] = B, the number of (expert, token block) pairs of the batch, [1] = units per down-projection work
//           item, [2] = invoked experts;
//   blk     [q] = {expert id | tokens << 16, offset of the expert's pairs in the permutation, token block, 0} for
//           block q < B, the invoked experts by ascending id, an expert's blocks in a row;
//   pairs   [q][i], 16 bits each: the (token, slot) pair id of the i-th token of block q, for the blocks of experts
//           with at most kDirectMaxTokens tokens (entries past the expert's tokens are not written).
// An expert with at most kDirectMaxTokens tokens is one token block; a larger one is cut into blocks of tok_block tokens (64, 128, or
// 256 in the wide kernel; one pass over the weights each), which go to workgroups of their own.  The work items of a projection are
// numbered block-major, unit-minor: item = block * units + unit, so a workgroup knows from its index alone which
// records to read, and one round trip to memory tells it its expert, its tokens and where their rows are: nothing
// it needs for its first weight and token loads depends on a second load.
// Three places write the tables, each from what it has at hand: routing_small_kernel (one block per expert, from the lanes),
// permute_from_bitsets (the last workgroup of remap_kernel, from the token bit sets) and plan_kernel (build_plan, from ranges
// that a caller passes in).
#pragma once

#include "lynx_common.h"

namespace lynx {

constexpr int kDirectMaxTokens = 16;         // experts with more tokens take the staged path
constexpr int kTokBlock = 64;                // tokens per pass of the staged path (batches of up to 64 tokens, quantised weights)
constexpr int kTokBlockBig = 128;            // the same for larger batches with bf16 weights (the wide kernel: kWideTokens, 256)

static_assert(LYNX_MAX_N + LYNX_MAX_T * LYNX_MAX_K / kTokBlock <= kPlanMaxBlocks, "the plan must hold every block of a batch");

// What the host knows of the FFN launch when the plan is built.
struct PlanShape {
    int units_gu;    // gate/up work items per (expert, token block): units of 64 or 128 of the F rows; 0 = build no plan
    int units_dn;    // down-projection row units per (expert, token block)
    int tok_block;   // tokens per block of an expert with more than kDirectMaxTokens
    int dn_cap;      // down items the grid is sized for: the device takes the fewest units per item that fit it
    int dn_m_max;    // most units per down item
    int shared_pairs;   // (shared expert, token block) pairs: completion counters to clear
    int max_blocks;     // (expert, token block) pairs that the FFN's grid has workgroups for, at most kPlanMaxBlocks
};

constexpr int kPlanB = 0, kPlanM = 1, kPlanNa = 2;   // words of the header

__host__ __device__ __forceinline__ int plan_token_blocks(int te, int tok_block)
{
    return te <= kDirectMaxTokens ? 1 : (te + tok_block - 1) / tok_block;
}

// Most (expert, token block) pairs a batch of T tokens with k picks each can have.  repeats: an assignment may send a token to one
// expert more than once (a caller's can; lynx_permute and the layer's routing make none such), so that an expert can
// have more rows than there are tokens.
inline int plan_max_blocks(int T, int N, int k, int tok_block, bool repeats)
{
    const long P = (long)T * k;
    const long experts = P < N ? P : N;
    if (T <= kDirectMaxTokens && !repeats) return (int)experts;
    return (int)(experts + P / tok_block);   // an expert with te rows has at most 1 + te / tok_block blocks
}

// Units per down item the device will choose for B blocks (same rule on the host, for the grid size).
__host__ __device__ __forceinline__ int plan_down_units_per_item(const PlanShape &ps, int B)
{
    int m = 1;
    while (m < ps.dn_m_max && (long)((ps.units_dn + m - 1) / m) * B > ps.dn_cap) m *= 2;
    return m;
}

// Down items the grid must hold for a batch with at most max_blocks blocks.
inline int plan_down_grid(const PlanShape &ps, int max_blocks)
{
    long worst = 0;
    for (int m = 1; m <= ps.dn_m_max; m *= 2) {
        // m is chosen when m/2 did not fit the cap and m does (or m is the largest): the most blocks with that choice
        const long per = (ps.units_dn + m - 1) / m;
        long b = m == ps.dn_m_max ? max_blocks : ps.dn_cap / per;
        if (b > max_blocks) b = max_blocks;
        if (per * b > worst) worst = per * b;
    }
    return (int)worst;
}

// The records of an expert with c > 0 pairs from offset off, blocks [q0, q0 + nb), and the header.
__device__ __forceinline__ void plan_write_records(int e, int c, int off, int q0, int nb, int32_t *__restrict__ ws)
{
    for (int j = 0; j < nb && q0 + j < kPlanMaxBlocks; ++j)
        *reinterpret_cast<int4 *>(ws + kWsPlanBlk + 4 * (q0 + j)) = make_int4(e | (c << 16), off, j, 0);
}
__device__ __forceinline__ void plan_write_header(const PlanShape &ps, int blocks, int invoked, int32_t *__restrict__ ws)
{
    ws[kWsPlanHdr + kPlanB] = min(blocks, kPlanMaxBlocks);
    ws[kWsPlanHdr + kPlanM] = plan_down_units_per_item(ps, blocks);
    ws[kWsPlanHdr + kPlanNa] = invoked;
}

// Builds the header and the block records from a caller's ranges.  Every thread of the workgroup calls it (one wave does the
// work); count[e] / offs[e] (pairs of expert e and where they start in the permutation) are in LDS and complete (barrier
// before).  blk0[e] (LDS) receives the first block of expert e, for the caller to file the pair ids under (barrier after).
// Ranges that overlap can make more blocks than the grid has workgroups for.  An expert is in the plan with all of its blocks
// or not at all (then none behind it is either): a down workgroup waits for the reports of every gate/up workgroup of
// its expert, and those of a block past the grid never come.
// ws = the routing part of the workspace.
__device__ __forceinline__ void build_plan(const PlanShape &ps, int N, const int *count, const int *offs, int *blk0,
                                           int32_t *__restrict__ ws)
{
    if (ps.units_gu <= 0) return;
    const int tid = threadIdx.x;
    if (tid >= kWave) return;
    int invoked = 0, blocks = 0, carry_b = 0;   // blocks: of the experts in the plan; carry_b: of all experts before these
    for (int base = 0; base < N; base += kWave) {
        const int e = base + tid;
        const int c = e < N ? count[e] : 0;
        const int nb = c > 0 ? plan_token_blocks(c, ps.tok_block) : 0;
        const int s = wave_prefix_sum_i32(nb);
        const int q0 = carry_b + s - nb;
        const bool in = c > 0 && q0 + nb <= ps.max_blocks;
        if (e < N) blk0[e] = in ? q0 : kPlanMaxBlocks;
        if (in) plan_write_records(e, c, offs[e], q0, nb, ws);
        invoked += __popcll(__ballot(in));
        blocks = max(blocks, wave_max_i32(in ? q0 + nb : 0));
        carry_b += __builtin_amdgcn_readlane(s, kWave - 1);
    }
    if (tid == 0) plan_write_header(ps, blocks, invoked, ws);
}

// Files pair id p, the i-th of expert e's te pairs, under the expert's block (experts on the direct path only).
__device__ __forceinline__ void plan_file_pair(const PlanShape &ps, const int *blk0, int e, int te, int i, int p,
                                               int32_t *__restrict__ ws)
{
    if (ps.units_gu <= 0 || te > kDirectMaxTokens) return;
    if (blk0[e] >= kPlanMaxBlocks) return;   // (not in the plan)
    reinterpret_cast<uint16_t *>(ws + kWsPlanPairs)[blk0[e] * kDirectMaxTokens + i] = (uint16_t)p;
}

}  // namespace lynx
