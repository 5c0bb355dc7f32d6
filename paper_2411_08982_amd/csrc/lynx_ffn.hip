// lynx_moe_ffn: grouped SwiGLU expert FFN over the invoked experts + gate-weighted combine, and the
// one-time weight re-layout it streams from.
//
// Decode is bound by streaming expert weights from HBM (paper Sec. 2.1: latency grows with the number
// of experts the batch activates), so the kernels are organised around the weight stream:
//   * weights are pre-packed so that a wave reads a 16-row x 32-column bf16 tile as one contiguous
//     1 KiB load (16 bytes per lane) that IS the A operand of v_mfma_f32_16x16x32_bf16;
//   * a wave owns 16 output rows and walks (a slice of) the contraction dimension with a ring of
//     prefetched tiles in registers, so each weight byte is fetched from HBM once per call;
//   * the tokens of the expert are the B operand, read from LDS.  Experts with few tokens (<= 16, the usual
//     decode case) put their rows there before the stream starts ("direct" path: one column tile, K split over
//     the waves where that pays); experts with many tokens stream the token tiles through LDS in chunks shared
//     by the four waves ("staged" path);
//   * the grid is fixed (most experts the batch can invoke + shared experts, times row tiles); a
//     workgroup whose rank is past the device-side num_active leaves at once, so nothing is read back
//     to the host;
//   * gate/up (with the SiLU-multiply epilogue) and down are ONE kernel whose grid holds the workgroups of
//     both; it is launched once (down workgroups wait for their expert's gate/up workgroups through
//     completion counters) or once per projection, whichever measured faster for the shape;
//   * weights are bf16, FP8 E4M3 with one scale per row, or MXFP4 with one scale per block of 32 columns (both
//     converted to bf16 in registers).
// Launches: the expert kernel (once or twice) and a small combine.

#include <atomic>
#include <type_traits>

#include "../../include/lynx_bench.h"
#include "lynx_plan.h"

namespace lynx {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kFfnThreads = 256;
constexpr int kFfnWaves = kFfnThreads / kWave;
constexpr int kPF = 8;                       // staged path: weight tiles in flight per wave and matrix
constexpr int kPFD = 8;                      // direct path: the same (most; see DirectDepth for the depth per format)
// Two LDS buffers for token rows.  They are two arrays, not halves of one: the compiler tells loads into the one from reads of
// the other by that, and does not wait for them.  They have to lie in the first 64 KiB, which loads into LDS can address.
// The compiler places them (by falling alignment, as it happens); the build compares the size of the kernel's LDS segment:
// anything ahead of them or between them would add a whole kStageAlign.
constexpr int kStageBuffer = 32768;
constexpr int kStageAlign = 4096;

// Token rows lie in LDS as 256-byte segments of sixteen 16-byte pieces in the order piece ^ (row % 16), so that the sixteen
// rows of an MFMA operand are read from different banks.  A segment holds four k-steps; the piece of k-step q of a segment
// that this lane's operand needs, for the tile layout of the weight format:
template <int WF>
__device__ __forceinline__ int stage_piece(int q)
{
    const int g = (int)((threadIdx.x & (kWave - 1)) >> 4);
    return WF == 0 ? q * 4 + g : WF == 1 ? (q >> 1) * 8 + g * 2 + (q & 1) : g * 4 + q;
}

// Optional per-workgroup timeline of the expert kernel (-DLYNX_TIMELINE; measurement builds only): for every workgroup
// four stamps of the chip-wide 100 MHz clock (start, item known, wait over, work done) and what it was (projection,
// workgroup index, XCC id), read back with lynx_debug_timeline.  The product build defines none of it.
#ifdef LYNX_TIMELINE
constexpr int kTimelineSlots = 1 << 15;
__device__ unsigned long long g_timeline[kTimelineSlots][6];
#define LYNX_TS_BEGIN(kind, b)                                                                                         \
    const int ts_slot_ = (int)blockIdx.x < kTimelineSlots ? (int)blockIdx.x : kTimelineSlots - 1;                      \
    if (threadIdx.x == 0) {                                                                                            \
        unsigned xcc_, hwid_;                                                                                          \
        asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(xcc_));                                          \
        asm volatile("s_getreg_b32 %0, hwreg(HW_REG_HW_ID)" : "=s"(hwid_));                                          \
        g_timeline[ts_slot_][0] = wall_clock64();                                                                      \
        g_timeline[ts_slot_][4] = ((unsigned long long)(kind) << 32) | (unsigned)(b);                                  \
        g_timeline[ts_slot_][5] = (xcc_ & 0xf) | ((unsigned long long)hwid_ << 8);                                     \
        g_timeline[ts_slot_][1] = g_timeline[ts_slot_][2] = g_timeline[ts_slot_][3] = 0;                               \
    }
#define LYNX_TS(i)                                                                                                     \
    if (threadIdx.x == 0) g_timeline[ts_slot_][i] = wall_clock64()
#else
#define LYNX_TS_BEGIN(kind, b)
#define LYNX_TS(i)
#endif

struct GemmParams {
    const uint16_t *W_routed;   // packed routed weights (gate/up interleaved, or down)
    const uint16_t *W_shared;   // packed shared-expert weights or NULL
    const float *sc_routed;     // FP8 weights: row scales, gate/up [N][2][F] or down [N][H]; MXFP4: the scale dwords; else unused
    const float *sc_shared;     // the same for the shared experts
    const uint16_t *B;          // gate/up: x [T,H]; down: h scratch
    void *out;                  // gate/up: h scratch (bf16); down: o scratch (fp32)
    const int32_t *perm;        // pair ids grouped by expert (the token assignment)
    const int32_t *plan;        // the routing part of the workspace: the work plan (lynx_plan.h)
    int T, N, k, n_shared;
    int R, K;                   // routed: output rows, contraction length
    int ldb_r, ldo_r, ldb_s, ldo_s;   // elements between B rows / output rows, routed and shared
    int Rs, Ks;                 // shared
    int tiles_r, tiles_s;       // row units per (routed expert, token block) / per shared work item
    int tiles_s_stride;         // tiles_s rounded up so that the token blocks of one shared row tile share an XCD
    int shared_tblocks;         // token blocks that a shared expert's tokens are divided into (1 = not divided)
    int tok_block;              // tokens per block: one pass of the staged path
    int routed_blocks, shared_blocks;   // grid = shared blocks first (the longest workgroups), then routed
    int shared_splits;          // K slices per shared expert (down projection only; each slice has its own output rows)
    int dn_m_max;               // most row units per down item that the plan may choose (1: always one)
    long long shared_h_base;    // element offset of the shared experts' h rows in the h scratch
};

// What a workgroup works on, resolved from blockIdx and the device-side routing tables.
struct WorkItem {
    const uint4 *W;      // packed weights of the expert
    const uint16_t *B;   // B-operand rows
    void *out;
    const float *sc;     // FP8 weights: this expert's row scales ([2][R] for gate/up, [R] for down); MXFP4: its scale dwords
    int R, K, tile, Te, off, shared_s, e;
    int te_all;          // all tokens of the expert (Te bounds this item's token block)
    int ldb, ldo;        // elements between B rows / output rows
    int tok0;            // first token of this work item's token block
    int kbeg, ksteps;    // slice of the contraction dimension this work item covers, in weight tiles (32 or 64 columns)
    int out_base;        // shared experts: first output row of this work item
    int pair;            // direct path, routed experts: the pair id of this lane's token column (lane % 16), -1 = none
    bool valid;
};

// Weight formats WF: 0 = bf16 (a 1 KiB tile is 16 rows x 32 columns), 1 = FP8 E4M3 (16 rows x 64 columns, converted to
// bf16 in registers; one fp32 scale per row applied to the accumulated sums), 2 = MXFP4 (16 rows x 128 columns:
// lane l holds row l%16, columns 32*(l/16) .. +31, which is exactly one scale block; converted to bf16 times the
// block's power-of-two scale in registers).  MXFP4 scale exponents: one dword per lane and four consecutive
// k-tiles (byte i = tile 4j+i), stored [row group][k-tile/4][lane][2], the 2 being gate|up, or the two row tiles of
// a down-projection row pair: a lane fetches both of its streams' scales with one 8-byte load.
template <int WF>
struct TileCols {
    static constexpr int value = 32 << WF;
};

// Dwords of MXFP4 scale exponents behind the weights of one expert's projection: row groups (gate/up: R/16 row
// tiles, both matrices; down: R/32 row pairs) x groups of four k-tiles x 64 lanes x 2.
__host__ __device__ __forceinline__ size_t mx_kt4(int K) { return (size_t)((K / 128 + 3) / 4); }
template <bool DUAL>
__host__ __device__ __forceinline__ size_t mx_scale_dwords(int R, int K)
{
    return (size_t)(DUAL ? R / 16 : R / 32) * mx_kt4(K) * 128;
}

// Which work item workgroup b of a projection is: one round trip to memory.  The shared experts' items come first
// (static: they see every token); the routed items follow in the plan's order, item = block * per + unit with
// per = the row units (gate/up) or groups of m row units (down) of one (expert, token block) pair.  The block's
// record, the header and the lane's pair id are requested together; their addresses follow from b alone.
// w.tile = the first row unit of the item, units = how many it covers.
template <bool DUAL, int WF>
__device__ __forceinline__ WorkItem resolve_item(const GemmParams &p, int b, int &units)
{
    constexpr int KC = TileCols<WF>::value;
    WorkItem w;
    w.sc = nullptr;
    w.valid = false;
    w.off = 0;
    w.Te = 0;
    w.te_all = 0;
    w.e = -1;
    w.shared_s = -1;
    w.tok0 = 0;
    w.pair = -1;
    w.B = p.B;
    w.out = p.out;
    units = 1;
    const uint16_t *Wbase;
    if (b >= p.shared_blocks) {
        const int idx = b - p.shared_blocks;
        const int32_t *__restrict__ plan = p.plan;
        // (down items of more than one row unit: their number per block is a device-side value, and the block
        // follows from it: a second round trip, only with that tuning knob set)
        const int m = (DUAL || p.dn_m_max <= 1) ? 1 : max(plan[kWsPlanHdr + kPlanM], 1);
        const int per = (p.tiles_r + m - 1) / m;
        const int q = min(idx / per, kPlanMaxBlocks - 1);
        const int B = plan[kWsPlanHdr + kPlanB];
        const int4 rec = *reinterpret_cast<const int4 *>(plan + kWsPlanBlk + 4 * q);
        const unsigned pv = reinterpret_cast<const uint16_t *>(plan + kWsPlanPairs)[q * kDirectMaxTokens + (lane_id() & 15)];
        if (B <= 0 || idx >= per * B) return w;   // (uniform: the whole workgroup leaves)
        // (the same for every lane: kept in scalar registers, and everything derived from them too)
        const int r0 = __builtin_amdgcn_readfirstlane(rec.x);
        const int e = r0 & 0xffff, te = (int)((unsigned)r0 >> 16);
        const int off = __builtin_amdgcn_readfirstlane(rec.y), tb = __builtin_amdgcn_readfirstlane(rec.z);
        if (e < 0 || e >= p.N || te <= 0 || off < 0 || off + te > p.T * p.k) return w;
        w.e = e;
        w.off = off;
        w.te_all = te;
        if (te > kDirectMaxTokens) {   // one pass of the staged path: tokens [tok0, Te) of the expert
            w.tok0 = tb * p.tok_block;
            w.Te = min(te, w.tok0 + p.tok_block);
            if (w.tok0 >= te) return w;
        } else {
            w.Te = te;
            w.pair = (int)pv;   // (checked where it is used)
        }
        w.tile = (idx % per) * m;
        units = min(m, p.tiles_r - w.tile);
        w.R = p.R;
        w.K = p.K;
        w.ldb = p.ldb_r;
        w.ldo = p.ldo_r;
        w.kbeg = 0;
        w.ksteps = w.K / KC;
        w.out_base = 0;
        Wbase = p.W_routed + (size_t)e * (((size_t)w.R * w.K * (DUAL ? 2 : 1)) >> WF);
        if (WF == 1) w.sc = p.sc_routed + (size_t)e * w.R * (DUAL ? 2 : 1);
        if (WF == 2) w.sc = p.sc_routed + (size_t)e * mx_scale_dwords<DUAL>(w.R, w.K);
    } else {
        // b = ((shared expert, K slice) * token blocks + token block) * stride + row tile.  Workgroups go to the
        // XCDs round-robin and the stride is a multiple of 8, so the token blocks of one row tile read their
        // common weights through one L2.
        w.tile = b % p.tiles_s_stride;
        const int vt = b / p.tiles_s_stride;
        const int v = vt / p.shared_tblocks;   // (shared expert, K slice)
        w.tok0 = (vt % p.shared_tblocks) * p.tok_block;
        w.shared_s = v / p.shared_splits;
        if (w.tile >= p.tiles_s || w.shared_s >= p.n_shared || w.tok0 >= p.T) return w;
        w.Te = p.shared_tblocks > 1 ? min(p.T, w.tok0 + p.tok_block) : p.T;   // tokens [tok0, Te)
        w.te_all = p.T;
        w.R = p.Rs;
        w.K = p.Ks;
        w.ldb = p.ldb_s;
        w.ldo = p.ldo_s;
        const int per = (w.K / KC + p.shared_splits - 1) / p.shared_splits;
        w.kbeg = (v % p.shared_splits) * per;
        w.ksteps = min(w.K / KC, w.kbeg + per) - w.kbeg;
        if (w.ksteps <= 0) return w;
        w.out_base = p.T * p.k + v * p.T;
        Wbase = p.W_shared + (size_t)w.shared_s * (((size_t)w.R * w.K * (DUAL ? 2 : 1)) >> WF);
        if (WF == 1) w.sc = p.sc_shared + (size_t)w.shared_s * w.R * (DUAL ? 2 : 1);
        if (WF == 2) w.sc = p.sc_shared + (size_t)w.shared_s * mx_scale_dwords<DUAL>(w.R, w.K);
        // shared experts keep their h rows in their own region of the scratch
        const size_t hbase = (size_t)p.shared_h_base + (size_t)w.shared_s * p.T * (DUAL ? w.ldo : w.ldb);
        if (DUAL)
            w.out = reinterpret_cast<uint16_t *>(p.out) + hbase;
        else
            w.B = p.B + hbase;
    }
    w.W = reinterpret_cast<const uint4 *>(Wbase);
    w.valid = true;
    return w;
}

// B row (element offset) and output row of the i-th token of the work item; -1 = none.
template <bool DUAL>
__device__ __forceinline__ void token_rows(const GemmParams &p, const WorkItem &w, int i, int &ro, int &orow)
{
    ro = -1;
    orow = -1;
    if (i >= w.Te) return;
    const int P = p.T * p.k;
    if (w.shared_s < 0) {
        const int pv = p.perm[w.off + i];
        const bool ok = pv >= 0 && pv < P;
        if (DUAL) {   // B row = x[token], out row = sorted position in h
            if (!ok) return;
            ro = (pv / p.k) * w.ldb;
            orow = w.off + i;
        } else {      // B row = h[sorted position] (known without the permutation), out row = pair id in o
            ro = (w.off + i) * w.ldb;
            orow = ok ? pv : -1;
        }
    } else if (DUAL) {   // shared: every token
        ro = i * w.ldb;
        orow = i;
    } else {
        ro = i * w.ldb;
        orow = w.out_base + i;
    }
}

// The same for this lane's token column on the direct path, from the pair id that came with the item: no load.
template <bool DUAL>
__device__ __forceinline__ void token_rows_direct(const GemmParams &p, const WorkItem &w, int &ro, int &orow)
{
    const int i = lane_id() & 15;
    ro = -1;
    orow = -1;
    if (i >= w.Te) return;
    if (w.shared_s < 0) {
        const bool ok = w.pair >= 0 && w.pair < p.T * p.k;
        if (DUAL) {
            if (!ok) return;
            ro = (w.pair / p.k) * w.ldb;
            orow = w.off + i;
        } else {
            ro = (w.off + i) * w.ldb;
            orow = ok ? w.pair : -1;
        }
    } else {
        ro = i * w.ldb;
        orow = DUAL ? i : w.out_base + i;
    }
}

__device__ __forceinline__ uint16_t f32_to_bf16_rne(float f)
{
    uint32_t u = __float_as_uint(f);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

__device__ __forceinline__ float silu_mul(float g, float u) { return (g / (1.0f + __expf(-g))) * u; }

// D fragment of v_mfma_f32_16x16x32: lane holds token column (lane & 15) and output rows
// 4*(lane >> 4) .. +3 of the wave's 16.  gate/up: h = silu(g) * u rounded to bf16; down: fp32.
// FP8 weights: the sums are scaled by the row scales first (sc: gate rows [R] then up rows [R], or the down rows).
template <bool DUAL, int NT, int WF>
__device__ __forceinline__ void epilogue(const f32x4 (&accg_in)[NT], const f32x4 (&accu_in)[NT], void *out, int ld, int row0,
                                         const int (&orow)[NT], const float *sc, int R)
{
    const int r = row0 + 4 * (lane_id() >> 4);
    f32x4 sg = {1.f, 1.f, 1.f, 1.f}, su = {1.f, 1.f, 1.f, 1.f};
    if (WF == 1) {
        const float4 a = *reinterpret_cast<const float4 *>(sc + r);
        sg = f32x4{a.x, a.y, a.z, a.w};
        if (DUAL) {
            const float4 b = *reinterpret_cast<const float4 *>(sc + R + r);
            su = f32x4{b.x, b.y, b.z, b.w};
        }
    }
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        if (orow[nt] < 0) continue;
        const f32x4 accg = WF == 1 ? accg_in[nt] * sg : accg_in[nt];
        const f32x4 accu = (WF == 1 && DUAL) ? accu_in[nt] * su : accu_in[nt];
        if (DUAL) {
            uint2 pk;
            pk.x = (uint32_t)f32_to_bf16_rne(silu_mul(accg[0], accu[0])) |
                   ((uint32_t)f32_to_bf16_rne(silu_mul(accg[1], accu[1])) << 16);
            pk.y = (uint32_t)f32_to_bf16_rne(silu_mul(accg[2], accu[2])) |
                   ((uint32_t)f32_to_bf16_rne(silu_mul(accg[3], accu[3])) << 16);
            // read by the down-projection workgroups of the same launch, possibly on another XCD
            store_coherent(reinterpret_cast<uint2 *>(reinterpret_cast<uint16_t *>(out) + (size_t)orow[nt] * ld + r), pk);
        } else {
            *reinterpret_cast<float4 *>(reinterpret_cast<float *>(out) + (size_t)orow[nt] * ld + r) =
                make_float4(accg[0], accg[1], accg[2], accg[3]);
        }
    }
}

// ---------------------------------------------------------------------------------------------------
// Weight streaming.  Both paths keep a ring of prefetched 1 KiB weight tiles per wave and stream in registers.  The loop
// bodies are branch-free on purpose: loads past the end of a run carry an offset out of range (nothing is fetched, the tile
// reads as zero), so that the compiler can count the outstanding loads and wait for exactly the oldest one instead of
// draining the queue.
// ---------------------------------------------------------------------------------------------------

// The offsets of the ring_load_* functions pass through an empty asm so that the compiler treats every ring load as a
// distinct, unmovable-by-value-numbering load: otherwise it merges the prefetch for the next turn of the ring
// with the loads of that turn and issues them only when they are needed.
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

// B operand (token rows).  For the down projection these are the intermediate vectors that gate/up workgroups
// of the same launch have written with device-coherent stores.  Plain (cached) loads are right for them: caches
// are invalidated when a kernel starts, a row is first touched after its expert's counter says it is complete,
// and rows start on 128-byte lines, so no cache on the reading side can hold an older copy of a line.  (Device-
// coherent loads instead would send every workgroup's re-reads of the same few rows to memory.)
//
// They are read through a buffer resource over the B array with a byte offset per lane, on their way to LDS.  A lane whose
// row holds no token carries an offset past the resource's range: the hardware returns zero for it and fetches nothing.
constexpr unsigned kNoToken = 0x80000000u;   // past any resource (the B arrays stay below 2 GiB, checked on the host)
typedef __amdgpu_buffer_rsrc_t BufferRsrc;
__device__ __forceinline__ BufferRsrc token_rows_resource(const uint16_t *B)
{
    // the array is the same for all lanes of a wave: hand the address over as scalars (a resource that the compiler
    // takes for a per-lane value costs a loop over its distinct values around every load)
    const unsigned long long a = reinterpret_cast<unsigned long long>(B);
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)a), hi = __builtin_amdgcn_readfirstlane((unsigned)(a >> 32));
    return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void *>(((unsigned long long)hi << 32) | lo), 0, 0x7fffffff,
                                             0x00020000);
}
__device__ __forceinline__ uint4 ring_load_b(BufferRsrc rs, unsigned off, int index)
{
    asm volatile("" : "+v"(index));
    const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rs, off + (unsigned)index * 16u, 0, 0);
    return make_uint4(v.x, v.y, v.z, v.w);
}

// Expert weights: a non-temporal load (a weight byte is read once per launch, and a stream that does not allocate in
// the caches on its way runs measurably closer to the HBM rate) through a buffer resource over the wave's run of weight
// tiles.  The ring is refilled without branches, so a wave nearing the end of its run still issues its refills; those
// carry an offset past the resource's range, for which the hardware returns zero and fetches nothing.  (Clamping them
// to the last tile instead re-read that tile once per ring slot: with the short runs of small experts, a down
// projection of 12 k-steps behind a ring of 8, two thirds more loads than the weights need.  A streaming probe with
// the same clamped ring reads 12 KiB runs at 5.9 TB/s and runs of 24 KiB and more at 7.0-7.2 TB/s.)
__device__ __forceinline__ BufferRsrc weights_resource(const uint4 *wave_base)
{
    // the run's first tile is the same for all lanes of a wave: hand the address over as scalars
    const unsigned long long a = reinterpret_cast<unsigned long long>(wave_base);
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)a), hi = __builtin_amdgcn_readfirstlane((unsigned)(a >> 32));
    return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void *>(((unsigned long long)hi << 32) | lo), 0, 0x7fffffff,
                                             0x00020000);
}
constexpr int kAuxNonTemporal = 2;
// index: in 16-byte units from this lane's piece of the run's first tile; live = false: nothing is fetched, zero returns
// KEEP: an ordinary cached load, for weights that another workgroup of the launch reads too
template <bool KEEP = false>
__device__ __forceinline__ uint4 ring_load_weights(BufferRsrc rs, int index, bool live)
{
    unsigned off = live ? ((unsigned)index + (unsigned)lane_id()) * 16u : kNoToken;
    asm volatile("" : "+v"(off));
    const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, KEEP ? 0 : kAuxNonTemporal);
    return make_uint4(v.x, v.y, v.z, v.w);
}

// 16 E4M3 codes (one lane's piece of a 64-column tile) -> two MFMA operands of 8 bf16 (columns 0-7 and 8-15 of
// the lane's group).  The hardware conversion gives fp32; an E4M3 value has 3 mantissa bits, so the upper half
// of the fp32 IS the bf16, exactly.
typedef float f32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t e4m3x2_to_bf16x2(uint32_t codes, bool upper)
{
    const f32x2 f = upper ? __builtin_amdgcn_cvt_pk_f32_fp8((int)codes, true) : __builtin_amdgcn_cvt_pk_f32_fp8((int)codes, false);
    return __builtin_amdgcn_perm(__float_as_uint(f.y), __float_as_uint(f.x), 0x07060302u);
}
__device__ __forceinline__ void e4m3x16_to_bf16(uint4 c, bf16x8 &lo, bf16x8 &hi)
{
    const uint4 l = make_uint4(e4m3x2_to_bf16x2(c.x, false), e4m3x2_to_bf16x2(c.x, true), e4m3x2_to_bf16x2(c.y, false),
                               e4m3x2_to_bf16x2(c.y, true));
    const uint4 h = make_uint4(e4m3x2_to_bf16x2(c.z, false), e4m3x2_to_bf16x2(c.z, true), e4m3x2_to_bf16x2(c.w, false),
                               e4m3x2_to_bf16x2(c.w, true));
    lo = __builtin_bit_cast(bf16x8, l);
    hi = __builtin_bit_cast(bf16x8, h);
}

// 32 E2M1 codes (one lane's piece of a 128-column MXFP4 tile: one scale block) -> four MFMA operands of 8 bf16
// (columns 8j .. 8j+7 of the block), each value already multiplied by the block scale.  The conversion
// instruction takes one byte (two codes, low nibble first) and the scale as a float; value * 2^k is exact in bf16.
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t e2m1x2_to_bf16x2(uint32_t codes, float scale, int byte)
{
    bf16x2 r;
    switch (byte) {   // the byte select is an immediate
    case 0: r = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(codes, scale, 0); break;
    case 1: r = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(codes, scale, 1); break;
    case 2: r = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(codes, scale, 2); break;
    default: r = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(codes, scale, 3); break;
    }
    return __builtin_bit_cast(uint32_t, r);
}
__device__ __forceinline__ bf16x8 e2m1x8_to_bf16(uint32_t codes, float scale)
{
    const uint4 v = make_uint4(e2m1x2_to_bf16x2(codes, scale, 0), e2m1x2_to_bf16x2(codes, scale, 1),
                               e2m1x2_to_bf16x2(codes, scale, 2), e2m1x2_to_bf16x2(codes, scale, 3));
    return __builtin_bit_cast(bf16x8, v);
}
// The scale of k-tile kt from the lane's dword of four exponents: 2^(E - 127) is the float with exponent field E.
__device__ __forceinline__ float mx_scale(uint32_t four, int kt) { return __uint_as_float(((four >> (8 * (kt & 3))) & 0xffu) << 23); }

// One weight tile of one stream -> its MFMA A operands (1, 2 or 4 k-steps of 32 columns).
template <int WF>
__device__ __forceinline__ void decode_tile(uint4 w, float scale, bf16x8 (&a)[1 << WF])
{
    if constexpr (WF == 0) {
        a[0] = __builtin_bit_cast(bf16x8, w);
    } else if constexpr (WF == 1) {
        e4m3x16_to_bf16(w, a[0], a[1]);
    } else {
        a[0] = e2m1x8_to_bf16(w.x, scale);
        a[1] = e2m1x8_to_bf16(w.y, scale);
        a[2] = e2m1x8_to_bf16(w.z, scale);
        a[3] = e2m1x8_to_bf16(w.w, scale);
    }
}

// Weight tiles in flight per wave and stream on the direct path (twice as many: equal or slower for every format, spills
// with bf16; half: 1-8 % slower).  A chunk of the token stage has to hold whole turns of the ring.
template <int WF>
struct DirectDepth {
    static constexpr int value = WF == 2 ? 4 : kPFD;
};

// Where a wave of the direct path streams from: needs the expert, not its tokens.  Two weight streams share every token
// fragment: gate and up tiles (interleaved: second = 64, step = 128) or, for the down projection, two consecutive row
// tiles (second = one row tile further, step = 64).
struct DirectPlan {
    const uint4 *Wb;     // the wave's first weight tile (the same for all lanes)
    const uint2 *Sl;     // MXFP4: this lane's scale dwords of the wave's row group, k-tile group 0
    int step, second;    // uint4 strides: next k-step, second stream
    int n;               // k-tiles of this wave
    int kt0;             // first k-tile actually read (0 for a wave without work)
    int rt;              // first 16-row tile
    bool rows_ok;
};

template <int WF>
struct WeightRing {
    static constexpr int D = DirectDepth<WF>::value;
    uint4 w0[D], w1[D];
    uint2 sq[D];   // MXFP4: the scale exponents of both streams (see the layout above)
};

// k-tiles per K slice of the item (the last slices may hold fewer, or none)
template <int KW>
__device__ __forceinline__ int slice_tiles(const WorkItem &w) { return (w.ksteps + KW - 1) / KW; }

template <bool DUAL, int KW, int WF>
__device__ __forceinline__ DirectPlan plan_direct(const WorkItem &w)
{
    constexpr int RW = kFfnWaves / KW;
    const int wv = wave_id();
    const int rw = wv / KW, kw = wv % KW;
    const int KT = w.K / TileCols<WF>::value;
    DirectPlan d;
    const int grp = w.tile * RW + rw;                  // row group of this wave
    d.rt = DUAL ? grp : 2 * grp;
    d.rows_ok = d.rt * 16 < w.R;                       // (down: R/16 is even, so the second tile exists too)
    const int per = slice_tiles<KW>(w);
    const int kb = w.kbeg + kw * per;
    d.n = max(min(w.kbeg + w.ksteps, kb + per) - kb, 0);
    const int rtc = d.rows_ok ? d.rt : 0;              // waves past the last row read tile 0 and store nothing
    d.kt0 = d.n > 0 ? kb : 0;
    d.step = DUAL ? 2 * kWave : kWave;
    d.second = DUAL ? kWave : KT * kWave;
    d.Wb = w.W + ((size_t)rtc * KT + d.kt0) * d.step;
    d.Sl = nullptr;
    if (WF == 2)
        d.Sl = reinterpret_cast<const uint2 *>(w.sc) + (size_t)(d.rows_ok ? grp : 0) * mx_kt4(w.K) * kWave + lane_id();
    return d;
}

__device__ __forceinline__ uint2 ring_load_scales(const uint2 *__restrict__ base, int index)
{
    asm volatile("" : "+v"(index));
    return base[index];
}

// Tile s of the wave's run into slot u; past the end of the run nothing is fetched and the tile reads as zero.
template <int WF>
__device__ __forceinline__ void load_slot(const DirectPlan &d, BufferRsrc rw, WeightRing<WF> &r, int u, int s)
{
    r.w0[u] = ring_load_weights(rw, s * d.step, s < d.n);
    r.w1[u] = ring_load_weights(rw, s * d.step + d.second, s < d.n);
    if (WF == 2) r.sq[u] = ring_load_scales(d.Sl, ((d.kt0 + max(min(s, d.n - 1), 0)) >> 2) * kWave);
}

template <int WF>
__device__ __forceinline__ void prefetch_weights(const DirectPlan &d, WeightRing<WF> &r)
{
    const BufferRsrc rw = weights_resource(d.Wb);
#pragma unroll
    for (int j = 0; j < DirectDepth<WF>::value; ++j) load_slot<WF>(d, rw, r, j, j);
}

// Direct path: experts with at most 16 tokens.  Bound by the weight stream (a plain read runs at 7.1 TB/s) and, in short
// launches, by the latency of its chain of loads.  The workgroup's waves are RW row groups x KW slices of K (a row group is
// one 16-row tile of gate and up, or two consecutive 16-row tiles of down, so that every token fragment feeds two MFMAs);
// the slices are summed through LDS at the end.
//
// The expert's token rows are staged in LDS, as many columns at a time as fit 32 KiB (twice, double buffered): all of them
// at once for most shapes, and then no barrier interrupts the stream.  (They used to travel with the weights through the
// same in-order queue: with 4-bit weights the fragments of a tile are 64 bytes per lane against the tile's 16, and the
// ring's registers held them too.  MXFP4, us per FFN call: Mixtral shapes 16 tokens 157 -> 128, 8 tokens 129 -> 112, 1 token
// 49 -> 43; FP8, Mixtral shapes 16 tokens 237 -> 228; bf16 within 1 %.)  R = the token count rounded up to a power of two: R rows of 512 / (KW * R) k-steps per
// slice; the other lanes of a fragment read a row again, and their results are never stored.
template <int KW>
struct TokenStage {
    int lr, lk;          // log2 of the rows R, of the k-steps (32 columns) per chunk
    __device__ __forceinline__ TokenStage(int te)
    {
        lr = te <= 1 ? 0 : 32 - __clz(te - 1);
        lk = 9 - (KW == 4 ? 2 : KW == 2 ? 1 : 0) - lr;
    }
    __device__ __forceinline__ int slice_bytes() const { return 64 << (lk + lr); }
};
constexpr int kStagePieces = 32 * 1024 / 16 / kFfnThreads;   // 16-byte pieces per thread and chunk

// Chunk c of the token rows into registers (ro: element offset of the row of token lane % 16, -1 = none); pieces of rows
// without a token or past the end of the slice arrive as zero.
template <int KW, int WF>
__device__ __forceinline__ void load_tokens(const WorkItem &w, const TokenStage<KW> &ts, BufferRsrc rb, int ro, int c,
                                            uint4 (&xr)[kStagePieces])
{
    constexpr int KC = TileCols<WF>::value;
    const int per = slice_tiles<KW>(w);
    // (one token: up to 4096 columns are a quarter of the pieces)
    const bool one = KW == 1 && ts.lr == 0 && (per << WF) * 4 <= kFfnThreads * kStagePieces / 4;
#pragma unroll
    for (int i = 0; i < kStagePieces; ++i) {
        if (i >= kStagePieces / 4 && one) break;
        const int q = threadIdx.x + kFfnThreads * i;             // [slice][row][piece]
        const int pc = q & ((4 << ts.lk) - 1), row = (q >> (ts.lk + 2)) & ((1 << ts.lr) - 1), kw = q >> (ts.lk + 2 + ts.lr);
        const int col = ((c << ts.lk) * 32) + pc * 8;            // column inside the slice
        const int tiles = min(per, w.ksteps - kw * per);         // of the slice
        const int r = __shfl(ro, row, kWave);
        xr[i] = ring_load_b(rb, (r >= 0 && col < tiles * KC) ? 2u * (unsigned)(r + (w.kbeg + kw * per) * KC + col) : kNoToken, 0);
    }
}
template <int KW>
__device__ __forceinline__ void store_tokens(const TokenStage<KW> &ts, int c, const uint4 (&xr)[kStagePieces], char *stage0, char *stage1)
{
    char *buf = (c & 1) ? stage1 : stage0;
#pragma unroll
    for (int i = 0; i < kStagePieces; ++i) {
        const int q = threadIdx.x + kFfnThreads * i;
        const int pc = q & ((4 << ts.lk) - 1), row = q >> (ts.lk + 2);   // (rows of all slices in a row)
        *reinterpret_cast<uint4 *>(buf + (row << (ts.lk + 6)) + (pc ^ (row & ((1 << ts.lr) - 1))) * 16) = xr[i];
    }
}

// The wave's products over its slice of K.  The ring arrives with its first turn of weight tiles requested and the stage
// with the first chunk of token rows.  Every wave makes the same number of turns.
template <int KW, int WF>
__device__ __forceinline__ void stream_direct(const WorkItem &w, const DirectPlan &d, const TokenStage<KW> &ts,
                                              WeightRing<WF> &r, BufferRsrc rb, int ro, char *stage0, char *stage1,
                                              f32x4 &acc0, f32x4 &acc1)
{
    constexpr int D = DirectDepth<WF>::value;
    constexpr int TS = 1 << WF;              // k-steps per weight tile
    const BufferRsrc rw = weights_resource(d.Wb);
    const int lane = lane_id();
    const int per = slice_tiles<KW>(w);
    const int C = (1 << ts.lk) / TS;         // tiles per chunk: a multiple of D
    const int chunks = (per + C - 1) / C;
    const int row = lane & ((1 << ts.lr) - 1);
    int xaddr[4];                            // this lane's place in its row, for each of a segment's four k-steps
#pragma unroll
    for (int q = 0; q < 4; ++q)
        xaddr[q] = (wave_id() % KW) * ts.slice_bytes() + (row << (ts.lk + 6)) + (stage_piece<WF>(q) ^ row) * 16;
    static_assert((D * TS) % 4 == 0, "a turn must hold whole segments");
    for (int c = 0; c < chunks; ++c) {
        uint4 xr[kStagePieces];
        const bool more = c + 1 < chunks;
        if (more) load_tokens<KW, WF>(w, ts, rb, ro, c + 1, xr);
        const char *buf = (c & 1) ? stage1 : stage0;
        auto read_b = [&](int kk) {   // k-step kk of the turn
            return __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(buf + (kk / 4) * 256 + xaddr[kk & 3]));
        };
        const int end = min(per, (c + 1) * C);
        for (int s0 = c * C; s0 < end; s0 += D, buf += D * TS * 64) {
            bf16x8 b[2][TS];
#pragma unroll
            for (int h = 0; h < TS; ++h) b[0][h] = read_b(h);
#pragma unroll
            for (int u = 0; u < D; ++u) {
                const int s = s0 + u;
                if (u + 1 < D) {
#pragma unroll
                    for (int h = 0; h < TS; ++h)
                        b[(u + 1) & 1][h] = read_b((u + 1) * TS + h);
                }
                bf16x8 a0[TS], a1[TS];
                const int kt = d.kt0 + max(min(s, d.n - 1), 0);
                decode_tile<WF>(r.w0[u], WF == 2 ? mx_scale(r.sq[u].x, kt) : 1.0f, a0);
                decode_tile<WF>(r.w1[u], WF == 2 ? mx_scale(r.sq[u].y, kt) : 1.0f, a1);
#pragma unroll
                for (int h = 0; h < TS; ++h) {
                    acc0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0[h], b[u & 1][h], acc0, 0, 0, 0);
                    acc1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1[h], b[u & 1][h], acc1, 0, 0, 0);
                }
                // ... then refill the slot (the scheduling fences keep the refill behind the last read of the slot,
                // so that it can land in the same registers and the ring needs no copies)
                __builtin_amdgcn_sched_barrier(0);
                load_slot<WF>(d, rw, r, u, s + D);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (more) {
            store_tokens<KW>(ts, c + 1, xr, stage0, stage1);
            __syncthreads();
        }
    }
}

// The K slices are summed through LDS and the results stored (orow: output row of this lane's token column).  The stage has
// been read by then: a barrier first.
template <bool DUAL, int KW, int WF>
__device__ __forceinline__ void direct_finish(const WorkItem &w, const DirectPlan &d, int orow, f32x4 acc0, f32x4 acc1, char *stage)
{
    const int lane = lane_id(), wv = wave_id();
    const int rw = wv / KW, kw = wv % KW;
    if (KW > 1) {
        f32x4 *r4 = reinterpret_cast<f32x4 *>(stage) + (size_t)rw * (KW - 1) * 2 * kWave + lane;   // [rw][kw-1][2][lane]
        __syncthreads();
        if (kw > 0) {
            r4[(size_t)(kw - 1) * 2 * kWave] = acc0;
            r4[(size_t)(kw - 1) * 2 * kWave + kWave] = acc1;
        }
        __syncthreads();
        if (kw == 0) {
#pragma unroll
            for (int j = 0; j < KW - 1; ++j) {
                acc0 += r4[(size_t)j * 2 * kWave];
                acc1 += r4[(size_t)j * 2 * kWave + kWave];
            }
        }
    }
    if (kw == 0 && d.rows_ok) {
        const f32x4 a0[1] = {acc0}, a1[1] = {acc1};
        const int orows[1] = {orow};
        if (DUAL) {
            epilogue<true, 1, WF>(a0, a1, w.out, w.ldo, d.rt * 16, orows, w.sc, w.R);
        } else {
            epilogue<false, 1, WF>(a0, a0, w.out, w.ldo, d.rt * 16, orows, w.sc, w.R);
            epilogue<false, 1, WF>(a1, a1, w.out, w.ldo, d.rt * 16 + 16, orows, w.sc, w.R);
        }
    }
}

// Staged path: the token tile is staged through LDS in chunks of KS k-steps of 32 columns, double buffered and shared by
// the four waves, each of which owns RT consecutive 16-row tiles (of gate and of up, or of down) and walks all of K.
// Every token fragment read from LDS feeds the S = RT (down) or 2 RT (gate/up) weight streams of the wave.
// The fragments are requested ahead of their products, in order: left to itself the compiler read one, waited for it and
// multiplied (every 64 cycles of MFMA behind a full LDS latency; with one column tile per fragment and stream, Mixtral
// shapes at 512 tokens 830 -> 758 us per layer).
// The token chunks go from memory to LDS directly (buffer loads with an LDS destination): no registers hold them, and a
// chunk of 32 KiB is requested a whole chunk ahead.  (Through registers the chunks were half that, requested as far ahead as
// the registers allowed: Mixtral shapes 1000 tokens 1104 -> 1079 us per layer, 128 tokens 467 -> 462; MXFP4 FFN of 100 tokens
// 193 -> 181, FP8 FFN of 512 tokens 638 -> 600.  Both ends of a buffer have to lie below 64 KiB of LDS: beyond it such loads
// were seen to land elsewhere.)
// D = weight tiles in flight per stream.  The sizes are bounded by the 256 registers of a wave at two workgroups per CU:
// sums S*NT*4, ring S*D*4, fragments.
template <int S, int NT, int WF>
struct StagedShape {
    static constexpr int KS = 32 / NT;                // k-steps of 32 columns per chunk
    static constexpr int TPC = KS >> WF;              // weight tiles per chunk
    static constexpr int D = S == 4 ? (WF == 0 && NT < 8 ? 8 : 4) : 2 * TPC < kPF ? 2 * TPC : kPF;
    static constexpr int BQ = S == 4 && NT == 8 ? 2 : 4;   // token fragments read ahead (the same at 2 and 4)
};

// Waits until at most N of the wave's loads are outstanding (they return in order).
template <int N>
__device__ __forceinline__ void wait_loads()
{
    constexpr int n = N < 63 ? N : 63;   // (the counter's field; a smaller count waits for more)
    __builtin_amdgcn_s_waitcnt((n & 15) | (n >> 4) << 14 | 7 << 4 | 15 << 8);   // loads only
}

// KEEP: the weights are read by another workgroup too (an expert with several token blocks): cached loads.
template <bool DUAL, int RT, int NT, int WF, bool KEEP>
__device__ __forceinline__ void expert_staged(const WorkItem &w, const int *rowoff, const int *outrow, char *stage0, char *stage1)
{
    constexpr int MATS = DUAL ? 2 : 1;
    constexpr int S = RT * MATS;
    typedef StagedShape<S, NT, WF> Shape;
    constexpr int D = Shape::D, KS = Shape::KS, TPC = Shape::TPC;
    constexpr int KC = TileCols<WF>::value;
    constexpr int TS = 1 << WF;                  // 32-column steps of the staged token tile per weight tile
    static_assert(NT * KS * 1024 <= kStageBuffer, "a chunk must fit its buffer");
    static_assert(TPC >= 1 && (2 * TPC) % D == 0, "two chunks must hold whole turns of the ring");
    constexpr int WSTEP = MATS * kWave;

    const int lane = lane_id(), wv = __builtin_amdgcn_readfirstlane(wave_id());
    const int KTrow = w.K / KC;                  // tiles between consecutive row tiles
    const int KT = w.ksteps, K = KT * KC;        // weight tiles and token columns of this item
    const int rt = (w.tile * kFfnWaves + wv) * RT;   // w.tile counts units of 64 * RT rows
    const bool wave_active = rt * 16 < w.R;      // idle waves read tile 0 (in bounds) and store nothing
    const int rtc = wave_active ? rt : 0;
    const int last = KT - 1;
    // the second of a wave's row tiles may lie past the last row (gate/up; R / 16 is even for down): it re-reads the first
    const int tile2 = (RT == 1 || rtc * 16 + 16 < w.R) ? KTrow * WSTEP : 0;

    // MXFP4: scale dwords of the wave's row groups (gate/up: one per row tile; down: one per row pair)
    constexpr int SG = DUAL ? RT : (RT + 1) / 2;
    const uint2 *Sl[SG];
#pragma unroll
    for (int g = 0; g < SG; ++g)
        Sl[g] = WF == 2 ? reinterpret_cast<const uint2 *>(w.sc) +
                              (size_t)(DUAL ? rtc + (tile2 ? g : 0) : rtc >> 1) * mx_kt4(w.K) * kWave + lane
                        : nullptr;
    const bool sc_second = !DUAL && RT == 1 && (rtc & 1);

    // Token rows: one load of a wave fetches 256 consecutive bytes of four rows (a load that gathers 64 bytes of sixteen rows
    // in operand order costs more than the staging saves).  Block (nt, seg) of a buffer: 16 rows x 256 bytes.
    // A row without a token carries an offset out of range: nothing is fetched, and its column is never stored.  So do the
    // columns past the end (the last chunk of a ragged K): they arrive in LDS as zeros.  The weights that they meet read as
    // zero too, but that alone would not do: zero times an infinity of the row is NaN.
    const BufferRsrc rb = token_rows_resource(w.B + (size_t)w.kbeg * KC);
    constexpr int SEG = KS / 4;                  // 256-byte segments of a row per chunk
    constexpr int LPW = NT * SEG * 4 / kFfnWaves;   // loads per wave and chunk: eight, SEG of each of its groups of four rows
    // The piece of its row that a lane fetches is piece0 ^ (its group's place among the four of a column tile) * 4; ro: the
    // byte offset of that piece in the first segment (past the range for a row without a token, whatever is added).
    const int piece0 = (lane & 15) ^ (lane >> 4);
    unsigned ro[LPW / SEG];
#pragma unroll
    for (int r = 0; r < LPW / SEG; ++r) {
        const int grp = wv * (LPW / SEG) + r;    // four rows of column tile grp / 4
        const int o = rowoff[grp * 4 + (lane >> 4)];
        ro[r] = (o >= 0 ? 2u * (unsigned)o : kNoToken) + (unsigned)(piece0 ^ ((grp & 3) * 4)) * 16u;
    }
    auto load_x = [&](char *buf, int c) {
        int wvx = wv;
        asm volatile("" : "+s"(wvx), "+s"(c));   // (addresses of every load kept in scalar registers would spill others)
#pragma unroll
        for (int i = 0; i < LPW; ++i) {
            const int grp = wvx * (LPW / SEG) + i / SEG, seg = i % SEG;
            const int col = (c * SEG + seg) * 128;   // first column of the segment
            const unsigned off = (piece0 ^ ((grp & 3) * 4)) * 8 < K - col ? ro[i / SEG] : kNoToken;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                rb, (__attribute__((address_space(3))) void *)(buf + ((grp >> 2) * SEG + seg) * 4096 + (grp & 3) * 1024), 16, off, 2 * col, 0, 0);
        }
    };
    int xaddr[4];                                // this lane's place in a block, for each of the block's four k-steps
#pragma unroll
    for (int q = 0; q < 4; ++q) xaddr[q] = (lane & 15) * 256 + (stage_piece<WF>(q) ^ (lane & 15)) * 16;
    // The wave's own pieces of the chunk requested last have landed, and then everybody's have, and nobody reads the other
    // buffer any more.  The count is of the loads that the wave has issued behind those pieces (`tiles` turns of load_w;
    // every load of the loop sits between scheduling fences).  The build counts them again in the machine code.
    // (Left to the compiler, which waited before a read of the last piece, the counts were the same but for MXFP4's first
    // chunks: nearly everything.  With the columns masked above, MXFP4 FFN of 100 tokens 173.6 -> 168.1 us.)
    constexpr int kLoadsPerTile = S + (WF == 2 ? SG : 0);
    auto chunk_ready = [&](auto tiles) {
        wait_loads<tiles.value * kLoadsPerTile>();
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("" ::: "memory");
    };

    const BufferRsrc rw = weights_resource(w.W + ((size_t)rtc * KTrow + w.kbeg) * WSTEP);
    uint4 wr[D][S];
    uint2 sq[D][SG];
    auto load_w = [&](int slot, int s) {   // stream m + MATS * r: matrix m of row tile r; past the end nothing is fetched
#pragma unroll
        for (int r = 0; r < RT; ++r)
#pragma unroll
            for (int m = 0; m < MATS; ++m)
                wr[slot][r * MATS + m] = ring_load_weights<KEEP>(rw, s * WSTEP + m * kWave + r * tile2, s <= last);
        if (WF == 2)
#pragma unroll
            for (int g = 0; g < SG; ++g) sq[slot][g] = ring_load_scales(Sl[g], ((w.kbeg + min(s, last)) >> 2) * kWave);
    };
    f32x4 acc[S][NT];
#pragma unroll
    for (int j = 0; j < S; ++j)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[j][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
    load_x(stage0, 0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < D; ++j) load_w(j, j);
    chunk_ready(std::integral_constant<int, D>());

    for (int s0 = 0; s0 < KT; s0 += 2 * TPC) {
#pragma unroll
        for (int half = 0; half < 2; ++half) {   // the two buffers are told apart at compile time
            if (half == 1 && s0 + TPC >= KT) break;
            const char *cur = half ? stage1 : stage0;
            char *nxt = half ? stage0 : stage1;
            load_x(nxt, s0 / TPC + half + 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int ut = 0; ut < TPC; ++ut) {
                const int u = (half * TPC + ut) % D;
                const int s = s0 + half * TPC + ut;
                // (tiles past the end of the run were not fetched and arrived as zeros; a wave without rows multiplies
                // tile 0 and stores nothing)
                const int kt = w.kbeg + min(s, last);
                bf16x8 a[S][TS];
#pragma unroll
                for (int j = 0; j < S; ++j) {
                    float sc = 1.0f;
                    if (WF == 2) {
                        const uint2 q = sq[u][DUAL ? j / MATS : j / 2];
                        sc = mx_scale((DUAL ? (j & 1) : RT == 1 ? (int)sc_second : (j & 1)) ? q.y : q.x, kt);
                    }
                    decode_tile<WF>(wr[u][j], sc, a[j]);
                }
                // token fragments in the order (k-step, token column), BQ of them requested ahead of their products
                constexpr int G = TS * NT, BQ = Shape::BQ < G ? Shape::BQ : G;
                auto read_b = [&](int i) {
                    return __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(
                        cur + ((i % NT) * SEG + (ut * TS + i / NT) / 4) * 4096 + xaddr[(ut * TS + i / NT) & 3]));
                };
                bf16x8 bq[BQ];
#pragma unroll
                for (int i = 0; i < BQ; ++i) bq[i] = read_b(i);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < G; ++i) {
#pragma unroll
                    for (int j = 0; j < S; ++j)
                        acc[j][i % NT] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[j][i / NT], bq[i % BQ], acc[j][i % NT], 0, 0, 0);
                    if (i + BQ < G) bq[i % BQ] = read_b(i + BQ);
                    __builtin_amdgcn_sched_barrier(0);
                }
                load_w(u, s + D);
                __builtin_amdgcn_sched_barrier(0);
            }
            chunk_ready(std::integral_constant<int, TPC>());
        }
    }
    if (!wave_active) return;
    int orow[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) orow[nt] = outrow[nt * 16 + (lane & 15)];
#pragma unroll
    for (int r = 0; r < RT; ++r) {
        if ((rt + r) * 16 >= w.R) break;
        epilogue<DUAL, NT, WF>(acc[r * MATS], acc[r * MATS + MATS - 1], w.out, w.ldo, (rt + r) * 16, orow, w.sc, w.R);
    }
}

// Tokens per pass of the staged path.  The large-batch kernels take 128 with bf16 weights.  With quantised weights the
// operands that a tile is converted to leave no registers for eight token columns beside four weight streams (40-60
// spilled): passes of 64, whose workgroups share an expert's weights through the L2 (see resolve_item).
constexpr int staged_tokens(int big, int wf) { return big && wf == 0 ? kTokBlockBig : kTokBlock; }

// One pass of the staged path over nb tokens.  Weights that other workgroups stream too (an expert of several token
// blocks) are read with cached loads: the later block finds them in the memory-side cache (Mixtral shapes, 1000 tokens,
// 1336 against 1230 us per layer).
template <bool DUAL, int RT, int BIG, int WF>
__device__ __forceinline__ void staged_pass(const WorkItem &w, int nb, const int *rowoff, const int *outrow, char *stage0,
                                            char *stage1)
{
    constexpr int TB = staged_tokens(BIG, WF);
    if (nb <= 32)
        expert_staged<DUAL, RT, 2, WF, false>(w, rowoff, outrow, stage0, stage1);
    else if (TB > 64 && nb <= 64)
        expert_staged<DUAL, RT, 4, WF, false>(w, rowoff, outrow, stage0, stage1);
    else if (BIG && w.te_all > TB)
        expert_staged<DUAL, RT, TB / 16, WF, BIG != 0>(w, rowoff, outrow, stage0, stage1);
    else
        expert_staged<DUAL, RT, TB / 16, WF, false>(w, rowoff, outrow, stage0, stage1);
}

// Both projections of every invoked and shared expert in ONE launch.  Grid: all gate/up workgroups, then
// all down workgroups; per projection the shared experts' items first, then the routed items in the order of the
// device-built plan (lynx_plan.h): live items are contiguous from the front of each part, and a workgroup past them
// leaves after one load.  A row unit is 16*RW rows of gate and up, or 32*RW rows of down, RW = 4 / KW.  An expert
// with at most kDirectMaxTokens tokens takes the direct path with the workgroup's four waves as RW row tiles x KW
// slices of K.  A larger expert takes the staged path, in which a workgroup covers 64 rows (128 in the large-batch kernels:
// see staged_row_tiles): where a direct workgroup covers fewer, one of those that share the rows does the work, one pass of
// up to 64 (128) tokens per item, and the others leave.  (The wide kernel has the same grid with units and blocks of its own.)  A down
// item covers m consecutive row units, m chosen on the device from the number of (expert, token block) pairs: few
// invoked experts get short items that fill the chip, many get fewer, longer ones, whose start-up (tables, first
// tiles) weighs less.  The gate/up part of the grid ends with spare workgroups: when the last round of live gate/up
// workgroups is small, each of its workgroups is replaced by four of one row tile (see ffn_kernel).
//
// A down workgroup needs the intermediate vectors h of its expert complete.  Every gate/up workgroup adds its
// row tiles (four, or one) to its expert's counter once its h stores have completed; a down workgroup requests its
// first weight tiles and then waits for the counter to reach the expert's row tiles.  Workgroups are dispatched in
// index order, so when a down workgroup runs, every gate/up workgroup has been dispatched, and those wait for
// nothing: the wait always ends.  It is bounded all the same: on running out the workgroup sets a flag in the
// workspace and goes on, so no wave can hang, and the combine kernel turns the flag into NaNs in y and a non-zero
// status word.  The gain: the down projection's start-up overlaps the tail of gate/up instead of following a launch
// boundary.
struct FfnParams {
    GemmParams gu, dn;
    int gu_blocks;
    int block0;       // index of this launch's first workgroup in the (gate/up, down) order
    int gu_split;     // 1: the last, partial round of gate/up workgroups is cut into single row tiles (see ffn_kernel)
    int wait;         // 0: the down workgroups of this launch follow a finished gate/up launch and do not wait
    int fill;         // > 0: down workgroups are in both of two launches and run in the first if at least so many are live
    int spin_limit;   // polls of a completion counter before a down workgroup gives up
    int target_bias;  // added to the count a down workgroup waits for (0; tests of the give-up path set it)
    int32_t *done;    // completion counters (kWsDone), zero before the launch
    int32_t *flags;
};

constexpr int kCus = 256;
constexpr int kSplitRound = kCus;    // workgroups per round of the dispatcher
constexpr int kSplitMaxRem = 128;    // largest partial round that is cut into single row tiles
constexpr int kSplitMaxTokens = 32;  // largest batch for which it is done
constexpr int kSpinLimit = 1 << 17;   // polls of a counter (about a microsecond each) before giving up

__device__ __forceinline__ int done_slot(const GemmParams &p, const WorkItem &w)
{
    return w.shared_s < 0 ? w.e * done_stride(p.N)
                          : kWsDoneWords + done_shared_slot(w.shared_s * p.shared_tblocks + w.tok0 / p.tok_block);
}

// Waits for this expert's (this token block's) intermediate vectors (down projection in the same launch as
// gate/up; gate/up workgroups report row tiles: four each, or one for a workgroup of a single tile).
__device__ __forceinline__ void wait_for_gate_up(const GemmParams &p, const WorkItem &w, const FfnParams &fp, const int32_t *counter)
{
    if (!fp.wait) return;
    const int items = w.shared_s < 0 ? fp.gu.tiles_r * plan_token_blocks(w.te_all, p.tok_block) : fp.gu.tiles_s;
    const int target = kFfnWaves * items + fp.target_bias;
    if (threadIdx.x == 0) {
        int polls = 0;
        while (load_coherent(counter) < target) {
            if (++polls > fp.spin_limit) {
                atomicOr(fp.flags, 1);
                break;
            }
            __builtin_amdgcn_s_sleep(8);
        }
    }
    __syncthreads();
}

// Reports that this workgroup's part of h is complete in memory.
__device__ __forceinline__ void report_gate_up(int32_t *counter, int row_tiles)
{
    wait_memory_complete();
    __syncthreads();
    if (threadIdx.x == 0) atomicAdd(counter, row_tiles);
}

// 16-row tiles per wave on the staged path.  Two in the large-batch kernels (gate/up, and down with undivided K): a token
// fragment read from LDS then feeds four MFMAs (gate/up) or two (down), and a unit of 128 rows stages the tokens half as
// often as two of 64.
constexpr int staged_row_tiles(bool dual, int kw, int big) { return big && (dual ? big == 2 : kw == 1) ? 2 : 1; }

// sub >= 0 (gate/up, KW = 4 only): the workgroup takes row tile `sub` of the four that workgroup b stands for.
template <bool DUAL, int KW, int BIG, int WF>
__device__ __forceinline__ void expert_work(const GemmParams &p, int b, const FfnParams &fp, char *stage0, char *stage1, int *rowoff,
                                            int *outrow, int sub = -1)
{
    constexpr int TB = staged_tokens(BIG, WF);   // tokens per pass
    int units;
    LYNX_TS_BEGIN(DUAL ? (sub >= 0 ? 2 : 1) : 0, b);
    WorkItem w = resolve_item<DUAL, WF>(p, b, units);
    if (!w.valid) return;
    if (sub >= 0) w.tile = w.tile * kFfnWaves + sub;
    int32_t *counter = fp.done + done_slot(p, w);
    if (DUAL && BIG == 2 && w.te_all <= kDirectMaxTokens) {   // the item's 128 rows as two direct units of 64
        w.tile *= 2;
        units = min(2, (w.R + 63) / 64 - w.tile);
    }
    const int unit0 = w.tile;
    LYNX_TS(1);
    auto wait_for_h = [&]() {
        if (!DUAL) wait_for_gate_up(p, w, fp, counter);
    };
    // (With K in four slices a chunk of sixteen rows holds half a turn of the ring of the quantised formats.  Such kernels are
    // for at most eight tokens, but an assignment that sends a token to one expert twice can still give it more rows.)
    constexpr int kDirectRows = KW == kFfnWaves && WF != 0 ? kDirectMaxTokens / 2 : kDirectMaxTokens;
    if (w.te_all <= kDirectRows) {
        // Direct path.  The weight stream starts before h is waited for, and the next unit's first tiles are requested
        // before this unit's results are exchanged and stored.
        const TokenStage<KW> ts(w.Te);
        const BufferRsrc rb = token_rows_resource(w.B);
        DirectPlan plan = plan_direct<DUAL, KW, WF>(w);
        WeightRing<WF> ring;
        int ro, orow;
        token_rows_direct<DUAL>(p, w, ro, orow);
        uint4 xr[kStagePieces];
        prefetch_weights<WF>(plan, ring);
        wait_for_h();
        LYNX_TS(2);
        load_tokens<KW, WF>(w, ts, rb, ro, 0, xr);
        for (int un = 0; un < units; ++un) {
            if (un > 0) {
                __syncthreads();   // the stage has been read
                load_tokens<KW, WF>(w, ts, rb, ro, 0, xr);
            }
            store_tokens<KW>(ts, 0, xr, stage0, stage1);
            __syncthreads();
            f32x4 acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f};
            stream_direct<KW, WF>(w, plan, ts, ring, rb, ro, stage0, stage1, acc0, acc1);
            const DirectPlan done = plan;
            if (un + 1 < units) {
                w.tile = unit0 + un + 1;
                plan = plan_direct<DUAL, KW, WF>(w);
                prefetch_weights<WF>(plan, ring);
            }
            direct_finish<DUAL, KW, WF>(w, done, orow, acc0, acc1, stage0);
        }
    } else {
        wait_for_h();
        LYNX_TS(2);
        // staged path.  The token tables of one pass: tokens [i0, i0 + nb) of the expert
        auto load_tables = [&](int i0, int nb) {
            const int tid = threadIdx.x;
            if (tid < TB) {
                int ro, orow;
                token_rows<DUAL>(p, w, tid < nb ? i0 + tid : w.Te, ro, orow);
                rowoff[tid] = ro;
                outrow[tid] = orow;
            }
            __syncthreads();
        };
        constexpr int kRT = staged_row_tiles(DUAL, KW, BIG);
        if constexpr (BIG) {
            // the item is one pass over one unit of 64 * kRT rows (straight-line on purpose: loops around the passes
            // cost registers that they do not have)
            const int nb = w.Te - w.tok0;
            load_tables(w.tok0, nb);
            staged_pass<DUAL, kRT, BIG, WF>(w, nb, rowoff, outrow, stage0, stage1);
        } else {
            // units of 64 rows.  A direct workgroup covers 16*RW rows (gate/up) or 32*RW rows (down).
            constexpr int kRowsPerWG = 16 * (kFfnWaves / KW) * (DUAL ? 1 : 2);
            constexpr int kUnits = kRowsPerWG >= 64 ? kRowsPerWG / 64 : 1;      // staged units per row unit
            constexpr int kShare = kRowsPerWG >= 64 ? 1 : 64 / kRowsPerWG;      // workgroups that share one staged unit
            // (a gate/up workgroup that shares its unit with others and leaves the work to one of them still reports
            // below: a down workgroup waits for the row tiles of all gate/up workgroups of its expert)
            // (shared experts see every token, so the host knows that they are staged and gives them one workgroup
            // per unit)
            const bool shared = w.shared_s >= 0;
            for (int un = 0; un < units; ++un) {
                const int tile = unit0 + un;
                // Of the workgroups that share a unit one does the work and the others leave.  Which one rotates with the
                // unit and the expert: the sharing workgroups have consecutive indices, so a fixed choice would put all
                // the staged work of the launch on the XCDs that the first of every four workgroups goes to (measured:
                // two of the eight XCDs ended their gate/up work at 44 us, the others at 31 us).
                // (Of the last unit's sharers some may not exist: R / 32 need not be even.)
                int owner = tile / kShare * kShare + (tile / kShare + w.e) % kShare;
                if (!DUAL && kShare > 1) owner = min(owner, p.tiles_r - 1);
                if (!shared && tile != owner) continue;
                const int s0 = shared ? tile : (tile / kShare) * kUnits;
                const int sn = shared ? 1 : kUnits;
                for (int su = 0; su < sn; ++su) {
                    w.tile = s0 + su;
                    if (w.tile * 64 >= w.R) break;
                    for (int i0 = w.tok0; i0 < w.Te; i0 += TB) {
                        const int nb = min(w.Te - i0, TB);
                        __syncthreads();   // the previous pass has read rowoff / outrow and the stage
                        load_tables(i0, nb);
                        staged_pass<DUAL, kRT, BIG, WF>(w, nb, rowoff, outrow, stage0, stage1);
                    }
                }
            }
        }
    }
    LYNX_TS(3);
    if (DUAL && fp.wait) report_gate_up(counter, KW == 1 ? kFfnWaves : 1);
}

// Workgroups per CU: the registers (256 per wave) and the LDS buffers both come to two.  The dispatcher fills a CU up to its
// occupancy limit before it moves on, so a third one would leave CUs idle in a grid that is small compared with the chip.
constexpr int kWgPerCu = 2;

template <int KWD, int BIG, int WF>
__global__ __launch_bounds__(kFfnThreads, kWgPerCu) void ffn_kernel(FfnParams fp)
{
    // staged token tile, or the K-slice partial sums
    constexpr int TB = staged_tokens(BIG, WF);
    __shared__ __attribute__((aligned(kStageAlign))) char stage0[kStageBuffer], stage1[kStageBuffer];
    __shared__ int rowoff[TB];   // staged path: element offset of each token's B row, -1 = none
    __shared__ int outrow[TB];   // staged path: output row of each token, -1 = none
    static_assert(2 * kStageBuffer <= 65536 && kStageBuffer % kStageAlign == 0 && sizeof(rowoff) + sizeof(outrow) < kStageAlign,
                  "loads into LDS address 64 KiB; the build checks the placement by the segment's size");
    constexpr int kLdsPerCu = 160 * 1024;
    static_assert(2 * kStageBuffer * kWgPerCu + kStageAlign <= kLdsPerCu && 2 * kStageBuffer * (kWgPerCu + 1) > kLdsPerCu,
                  "workgroups per CU");
    const int b = blockIdx.x + fp.block0;
    if (b < fp.gu_blocks) {
        // Gate/up workgroups take four row tiles, one per wave, and the dispatcher hands workgroups to the CUs
        // breadth first: L live workgroups put two on L mod 256 CUs and one on the rest, and while the stream is
        // HBM-bound the CUs share it evenly, so the CUs with two take twice as long (measured: Qwen3 shape, 312
        // workgroups: 21-24 us against 40-48 us), at the end on a fraction of the chip's waves.  When that last,
        // partial round is small, each of its workgroups is replaced by four workgroups of one row tile (the
        // four waves split K), which the dispatcher spreads over all CUs: at most one or two tiles more per CU.
        // The count of live workgroups is a device-side value, so the mapping is made here.
        // (bf16 weights only: in the kernels of the quantised formats the second code path costs spilled registers)
        int bb = b, sub = -1;
        if (WF == 0 && fp.gu_split) {
            const int live = fp.gu.shared_blocks + max(fp.gu.plan[kWsPlanHdr + kPlanB], 0) * fp.gu.tiles_r;
            const int full = live / kSplitRound * kSplitRound, rem = live - full;
            if (rem > 0 && rem <= kSplitMaxRem && full >= fp.gu.shared_blocks) {
                // The small workgroups come last in the grid: they fill the tail.  (Putting them first when everything
                // is resident at once was tried, so that the small one is the older workgroup on its CU: with the
                // device-built plan it is equal or slower, Qwen3 shapes 32 tokens 51.7 against 49.3 us, 16 tokens
                // 47.4 against 43.1.)
                if (b >= full) {
                    bb = full + (b - full) / kFfnWaves;
                    sub = (b - full) % kFfnWaves;
                    if (bb >= live) return;
                }
            }
        }
        if (WF != 0 || sub < 0)
            expert_work<true, 1, BIG, WF>(fp.gu, bb, fp, stage0, stage1, rowoff, outrow);
        else if constexpr (WF == 0)
            expert_work<true, kFfnWaves, BIG, WF>(fp.gu, bb, fp, stage0, stage1, rowoff, outrow, sub);
    } else {
        if (WF != 0 && fp.fill > 0) {   // (the same answer in every workgroup of both launches: see launch_shape)
            const int live = fp.dn.shared_blocks + max(fp.dn.plan[kWsPlanHdr + kPlanB], 0) * fp.dn.tiles_r;
            if ((live >= fp.fill) != (fp.wait != 0)) return;
        }
        expert_work<false, KWD, BIG, WF>(fp.dn, b - fp.gu_blocks, fp, stage0, stage1, rowoff, outrow);
    }
}

// ---------------------------------------------------------------------------------------------------
// Wide kernel (bf16 weights, batches whose experts hold more than 128 tokens on average): token blocks of 256, units of 128
// gate/up rows or 256 down rows, one workgroup of four waves per CU with 512 registers each.
// With blocks of 128 tokens such a batch is bound by what passes the L2: every block of an expert streams its weights again
// (Mixtral shapes, 1000 tokens: 6.6 GB, at the 7.2 TB/s that memory and the memory-side cache both deliver; with the weights read
// from one place, 1106 -> 740 us).  Twice the tokens per weight byte need 256 sums per lane, all of the accumulator registers,
// and leave one wave per SIMD, so nothing but the order of the instructions hides a latency:
//   * every token fragment read from LDS feeds four products (64 cycles of matrix work), BQ fragments ahead, also across
//     the end of a chunk, and everything that is not a product is issued between two products, one thing at a time;
//   * token rows travel through registers, requested two chunks (128 columns) before they are written to LDS, as far ahead as the
//     weights: loads return in order, so whatever is waited for earlier shortens the way of everything behind it;
//   * three LDS buffers and one barrier per chunk, in the middle of its products: a wave that is past it may write the
//     buffer after next while another still reads the last one.
// Mixtral shapes, 1000 tokens, us per layer 1106 -> 898 (gate/up 670 -> 510, down 417 -> 330): matrix cores busy half of the
// time a wave is there (8 of 10 states with the weights in the caches), gate/up 5.2 rounds of workgroups, down 208 of them, one
// to a CU.  On the way (where it ended at 875): products in fours with the rest behind them 1008, dealt out between them 957; a
// turn of two chunks without a way out in the middle 915; loads further apart 866 to 881.
// ---------------------------------------------------------------------------------------------------
constexpr int kWideTokens = 256;             // tokens per block
constexpr int kWideCols = 64;                // columns of a chunk: whole 128-byte lines of a token row
constexpr int kWideBuffer = kWideTokens * kWideCols * 2;

// One product.  Written out, because the compiler (left alone it keeps the sums in the other half of the registers, where they do
// not fit beside the operands, and spills hundreds) has to be told that they live in accumulator registers.  It does not know what
// is inside and inserts no waits between this and other instructions: settle_sums() stands between the sums and ordinary code, no
// sum is used again for 4 * NT products, and the operands come from loads.  The build checks in the machine code that no VALU
// instruction writes an operand in the two states before its use, and that nothing else reads or writes a sum (a copy or a spill that
// the compiler puts in) less than 19 states behind its product, in both cases across branches too.
__device__ __forceinline__ void mfma_acc(f32x4 &c, bf16x8 a, bf16x8 b)
{
    asm("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
}
// Between the products and ordinary instructions on the sums, in both directions: more states than the longest wait.
template <int S, int NT>
__device__ __forceinline__ void settle_sums(f32x4 (&acc)[S][NT])
{
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
#pragma unroll
    for (int j = 0; j < S; ++j)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) asm volatile("" : "+a"(acc[j][nt]));
    asm volatile("s_nop 15" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

template <bool DUAL, int NT>
__device__ __forceinline__ void expert_wide(const WorkItem &w, const int *rowoff, const int *outrow, char *stage)
{
    constexpr int MATS = DUAL ? 2 : 1, S = 4, RT = S / MATS;   // weight streams of a wave: RT row tiles of MATS matrices
    constexpr int D = 4;                         // k-steps (32 columns) in the weight ring: two chunks
    constexpr int LPT = NT / 2;                  // token loads per thread and chunk: 32 rows x 128 bytes each
    constexpr int BQ = NT < 8 ? 3 : 7;           // token fragments read ahead: 64 cycles of products each
    constexpr int WS = NT < 8 ? 1 : NT < 12 ? 2 : 3;   // fragments between the weight loads of a k-step
    constexpr int WSTEP = MATS * kWave;
    static_assert(NT % 2 == 0 && NT * 16 * kWideCols * 2 <= kWideBuffer, "a chunk must fit its buffer");

    const int tid = threadIdx.x, lane = lane_id(), wv = __builtin_amdgcn_readfirstlane(wave_id());
    const int KTrow = w.K / 32, KT = w.ksteps, K = KT * 32, last = KT - 1;
    const int rt = (w.tile * kFfnWaves + wv) * RT;
    const bool wave_active = rt * 16 < w.R;      // idle waves read tile 0 (in bounds) and store nothing
    const int rtc = wave_active ? rt : 0;
    int tile_at[RT];                             // row tiles past the last row re-read the wave's first
#pragma unroll
    for (int r = 0; r < RT; ++r) tile_at[r] = (rtc + r) * 16 < w.R ? r * KTrow * WSTEP : 0;

    const BufferRsrc rb = token_rows_resource(w.B + (size_t)w.kbeg * 32);
    const int piece = tid & 7;                   // 16-byte piece of a row's 128
    unsigned ro[LPT];                            // byte offset of this thread's piece in its rows, out of range = no token
#pragma unroll
    for (int i = 0; i < LPT; ++i) {
        const int o = rowoff[(tid >> 3) + 32 * i];
        ro[i] = o >= 0 ? 2u * (unsigned)o + (unsigned)piece * 16u : kNoToken;
    }
    u32x4 xr[2][LPT];
    auto load_x1 = [&](int set, int i, int c) {  // (columns past the end, and chunks, arrive as zeros)
        const bool in = c * kWideCols + piece * 8 < K;
        asm volatile("" : "+s"(c));
        xr[set][i] = __builtin_amdgcn_raw_buffer_load_b128(rb, in ? ro[i] : kNoToken, c * (kWideCols * 2), 0);
    };
    // A row's eight pieces lie in the order piece ^ (row % 8): eight rows of a fragment, and the row that eight lanes write, lie in
    // different banks.
    const int xst = (tid >> 3) * 128 + (piece ^ ((tid >> 3) & 7)) * 16;
    auto store_x1 = [&](int set, int i, char *buf) { *reinterpret_cast<u32x4 *>(buf + xst + i * 4096) = xr[set][i]; };
    int xaddr[2];                                // this lane's place in a fragment, for each of a chunk's two k-steps
#pragma unroll
    for (int q = 0; q < 2; ++q) xaddr[q] = (lane & 15) * 128 + ((q * 4 + (lane >> 4)) ^ (lane & 7)) * 16;

    const BufferRsrc rw = weights_resource(w.W + ((size_t)rtc * KTrow + w.kbeg) * WSTEP);
    uint4 wr[D][S];
    auto load_w1 = [&](int slot, int j, int s) {   // stream m + MATS * r: matrix m of row tile r; past the end nothing is fetched
        wr[slot][j] = ring_load_weights<true>(rw, s * WSTEP + (j % MATS) * kWave + tile_at[j / MATS], s <= last);
    };
    f32x4 acc[S][NT];
#pragma unroll
    for (int j = 0; j < S; ++j)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[j][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto barrier = [&]() {                       // this wave's writes to LDS are done; everybody's are behind it
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(15 | 3 << 14 | 7 << 4 | 0 << 8);   // LDS only
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };

    // (the order of the loop below, so that the compiler counts the same loads behind each one on both ways into it)
    auto load_wx = [&](int s, int set, int c) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            if (nt % WS == 0 && nt / WS < S) load_w1(s, nt / WS, s);
            if (nt % 2 == 1) load_x1(set, nt / 2, c);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
#pragma unroll
    for (int i = 0; i < LPT; ++i) load_x1(0, i, 0);
    __builtin_amdgcn_sched_barrier(0);
    load_wx(0, 1, 1);
#pragma unroll
    for (int j = 0; j < S; ++j) load_w1(1, j, 1);
    settle_sums(acc);
#pragma unroll
    for (int i = 0; i < LPT; ++i) store_x1(0, i, stage);
    load_wx(2, 0, 2);
    barrier();

    constexpr int G = 2 * NT;                    // fragments of a chunk: k-step i / NT, column tile i % NT
    constexpr int NB = BQ + 1;                   // fragment i lies in bq[i % NB]
    constexpr bool kEarly = NT / 2 <= BQ;        // the reads that run into the next chunk begin before half of the second k-step
    static_assert(G % NB == 0 && (kEarly ? BQ <= NT : NT / 2 - 1 + BQ < NT), "nothing of the next chunk is read ahead of the barrier");
    char *cur = stage, *nxt = stage + kWideBuffer, *far = stage + 2 * kWideBuffer;
    auto read_b = [&](int i) {
        const char *buf = i < G ? cur : nxt;
        const int j = i < G ? i : i - G;
        return __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(buf + xaddr[j / NT] + (j % NT) * 2048));
    };
    bf16x8 bq[NB];
#pragma unroll
    for (int i = 0; i < BQ; ++i) bq[i] = read_b(i);
    // (Two chunks a turn, also where the second one is all zeros: with a way out between them the compiler takes the loads of the
    // first for the newest at the top of the loop and waits for nearly all of them.)
    for (int c0 = 0; c0 < KT; c0 += 2 * 2) {
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            const int c = c0 / 2 + half;
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int slot = half * 2 + q;
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    // A wave is alone on its SIMD, and what it issues between two products costs nothing while the first one
                    // runs; behind four products in a row it does.  So everything else is dealt out between them.
                    const int i = q * NT + nt;
                    const bf16x8 b = bq[i % NB];
#pragma unroll
                    for (int j = 0; j < S; ++j) {
                        mfma_acc(acc[j][nt], __builtin_bit_cast(bf16x8, wr[slot][j]), b);
                        __builtin_amdgcn_sched_barrier(0);
                        if (j == 0) bq[(i + BQ) % NB] = read_b(i + BQ);
                        if (j == 1 && nt % WS == 0 && nt / WS < S) load_w1((slot + 3) % D, nt / WS, 2 * c + q + 3);   // the slot of the last k-step
                        if (q == 0 && j == 2 && nt >= NT / 2) store_x1(1 - half, nt - NT / 2, nxt);    // chunk c + 1
                        if (q == 1 && j == 2 && nt % 2 == 1) load_x1(1 - half, nt / 2, c + 3);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    if (kEarly ? q == 0 && nt == NT - 1 : q == 1 && nt == NT / 2 - 1) barrier();
                }
            }
            char *t = cur;
            cur = nxt;
            nxt = far;
            far = t;
        }
    }
    settle_sums(acc);
    if (!wave_active) return;
    int orow[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) orow[nt] = outrow[nt * 16 + (lane & 15)];
#pragma unroll
    for (int r = 0; r < RT; ++r) {
        if ((rt + r) * 16 >= w.R) break;
        epilogue<DUAL, NT, 0>(acc[r * MATS], acc[r * MATS + MATS - 1], w.out, w.ldo, (rt + r) * 16, orow, w.sc, w.R);
    }
}

template <bool DUAL>
__device__ __forceinline__ void wide_work(const GemmParams &p, int b, const FfnParams &fp, char *stage, int *rowoff, int *outrow)
{
    int units;
    LYNX_TS_BEGIN(DUAL ? 1 : 0, b);
    const WorkItem w = resolve_item<DUAL, 0>(p, b, units);
    if (!w.valid) return;
    int32_t *counter = fp.done + done_slot(p, w);
    LYNX_TS(1);
    if (!DUAL) wait_for_gate_up(p, w, fp, counter);
    LYNX_TS(2);
    const int nb = w.Te - w.tok0;
    if ((int)threadIdx.x < kWideTokens) {
        int ro, orow;
        token_rows<DUAL>(p, w, (int)threadIdx.x < nb ? w.tok0 + (int)threadIdx.x : w.Te, ro, orow);
        rowoff[threadIdx.x] = ro;
        outrow[threadIdx.x] = orow;
    }
    __syncthreads();
    if (nb <= 64)
        expert_wide<DUAL, 4>(w, rowoff, outrow, stage);
    else if (nb <= 128)
        expert_wide<DUAL, 8>(w, rowoff, outrow, stage);
    else if (nb <= 192)
        expert_wide<DUAL, 12>(w, rowoff, outrow, stage);
    else
        expert_wide<DUAL, 16>(w, rowoff, outrow, stage);
    LYNX_TS(3);
    if (DUAL && fp.wait) report_gate_up(counter, kFfnWaves);
}

__global__ __launch_bounds__(kFfnThreads, 1) void ffn_wide_kernel(FfnParams fp)
{
    static_assert(kWideTokens <= kFfnThreads, "a thread per token of the tables");
    __shared__ __attribute__((aligned(128))) char stage[3 * kWideBuffer];
    __shared__ int rowoff[kWideTokens], outrow[kWideTokens];
    const int b = blockIdx.x + fp.block0;
    if (b < fp.gu_blocks)
        wide_work<true>(fp.gu, b, fp, stage, rowoff, outrow);
    else
        wide_work<false>(fp.dn, b - fp.gu_blocks, fp, stage, rowoff, outrow);
}

// The plan from a caller's token assignment (lynx_moe_ffn after lynx_permute): the experts with a valid, non-empty
// range in expert_offsets are the invoked ones.  One workgroup; also clears the completion counters and the flags.
__global__ __launch_bounds__(256) void plan_kernel(const int32_t *__restrict__ offsets, const int32_t *__restrict__ perm, int N,
                                                   int P, PlanShape ps, int32_t *__restrict__ ws)
{
    __shared__ int count[LYNX_MAX_N], offs[LYNX_MAX_N], blk0[LYNX_MAX_N];
    const int tid = threadIdx.x;
    const int clear = kWsDoneWords + (ps.shared_pairs > 0 ? kWsDoneSharedWords : 0);
    for (int i = tid * 4; i < clear; i += 256 * 4) *reinterpret_cast<int4 *>(ws + kWsDone + i) = make_int4(0, 0, 0, 0);
    if (tid < 16) ws[kWsFlags + tid] = 0;
    if (tid < N) {
        const int o0 = offsets[tid], o1 = offsets[tid + 1];
        const bool ok = o0 >= 0 && o1 > o0 && o1 <= P;
        count[tid] = ok ? o1 - o0 : 0;
        offs[tid] = ok ? o0 : 0;
    }
    __syncthreads();
    build_plan(ps, N, count, offs, blk0, ws);
    __syncthreads();
    // the pair ids of the experts on the direct path, 16 threads per expert
    for (int e = tid / kDirectMaxTokens; e < N; e += 256 / kDirectMaxTokens) {
        const int i = tid % kDirectMaxTokens;
        if (i < count[e]) {   // (an id outside [0, P) is filed as 0xffff: no such pair, the row is skipped)
            const int pv = perm[offs[e] + i];
            plan_file_pair(ps, blk0, e, count[e], i, (pv >= 0 && pv < P) ? pv : 0xffff, ws);
        }
    }
}

// n values to an aligned place, from one that need not be (n a multiple of 32).
__global__ __launch_bounds__(256) void realign_kernel(const uint16_t *__restrict__ x, uint16_t *__restrict__ out, size_t n)
{
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) out[i] = x[i];
}

// y[t] = sum_j gate[t,j] * o[t*k+j] + sum_s o[P + s*T + t].  If a workgroup of the expert kernel gave up a bounded wait
// (flags != 0: some rows of o may then be computed from incomplete intermediate vectors) every element of y becomes NaN
// and *status (if given) 1, else *status 0: a failed hand-over cannot pass for a result.
__global__ __launch_bounds__(256) void combine_kernel(const float *__restrict__ o, const int32_t *__restrict__ idx,
                                                      const float *__restrict__ gate, int T, int H, int N, int k,
                                                      int n_shared, float *__restrict__ y,
                                                      const int32_t *__restrict__ flags, int32_t *__restrict__ status)
{
    const int t = blockIdx.y;
    const int h = (blockIdx.x * 256 + threadIdx.x) * 4;
    // Latency-bound: the rows' loads must not wait for the picks one by one, so eight are requested before the first is
    // used.  A pick outside [0, N) has no row: its load is not made and it adds nothing.
    const int32_t *it = idx + (size_t)t * k;
    const float *gt = gate + (size_t)t * k;
    const int failed_word = *flags;
    if (status && t == 0 && blockIdx.x == 0 && threadIdx.x == 0) *status = failed_word != 0 ? 1 : 0;
    if (h >= H) return;
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    constexpr int U = 8;
    for (int j0 = 0; j0 < k; j0 += U) {
        float4 v[U];
        float g[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int j = min(j0 + u, k - 1);
            const int e = it[j];
            const bool live = j0 + u < k && e >= 0 && e < N;
            g[u] = live ? gt[j] : 0.f;
            v[u] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (live) v[u] = *reinterpret_cast<const float4 *>(o + ((size_t)t * k + j) * H + h);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            acc.x = fmaf(g[u], v[u].x, acc.x);
            acc.y = fmaf(g[u], v[u].y, acc.y);
            acc.z = fmaf(g[u], v[u].z, acc.z);
            acc.w = fmaf(g[u], v[u].w, acc.w);
        }
    }
    for (int s = 0; s < n_shared; ++s) {
        const float4 v = *reinterpret_cast<const float4 *>(o + ((size_t)T * k + (size_t)s * T + t) * H + h);
        acc.x += v.x;
        acc.y += v.y;
        acc.z += v.z;
        acc.w += v.w;
    }
    if (failed_word != 0) {
        const float q = __int_as_float(0x7fc00000);
        acc = make_float4(q, q, q, q);
    }
    *reinterpret_cast<float4 *>(y + (size_t)t * H + h) = acc;
}

// Row-major -> streaming layout, one 16-byte piece per thread.
__global__ __launch_bounds__(256) void pack_kernel(const uint16_t *__restrict__ Wa, const uint16_t *__restrict__ Wb,
                                                   int nmat, int E, int R, int K, uint16_t *__restrict__ out)
{
    const int KT = K / 32;
    const size_t pieces = (size_t)E * (R / 16) * KT * nmat * kWave;
    const size_t q = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (q >= pieces) return;
    const int l = (int)(q % kWave);
    size_t rest = q / kWave;
    const int m = (int)(rest % nmat);
    rest /= nmat;
    const int kt = (int)(rest % KT);
    rest /= KT;
    const int rt = (int)(rest % (R / 16));
    const int e = (int)(rest / (R / 16));
    const uint16_t *src = (m == 0 ? Wa : Wb) + ((size_t)e * R + rt * 16 + (l & 15)) * K + kt * 32 + (l >> 4) * 8;
    *reinterpret_cast<uint4 *>(out + q * 8) = *reinterpret_cast<const uint4 *>(src);
}

// Nearest E4M3 code of v (ties to the even code, 448 and above to +-448, NaN to NaN), in integer and exact
// floating-point steps so that it does not depend on a conversion mode of the hardware.
__device__ __forceinline__ uint32_t e4m3_encode(float v)
{
    const uint32_t sgn = (__float_as_uint(v) >> 24) & 0x80u;
    if (v != v) return sgn | 0x7fu;
    const float a = fabsf(v);
    if (a >= 448.0f) return sgn | 0x7eu;
    uint32_t code;
    if (a < 0.015625f) {                       // below 2^-6: multiples of 2^-9
        code = (uint32_t)rintf(a * 512.0f);
    } else {
        const uint32_t bits = __float_as_uint(a);
        const int ex = (int)(bits >> 23) - 127;                              // a = m * 2^ex, m in [1, 2)
        const float m = __uint_as_float((bits & 0x007fffffu) | 0x3f800000u);
        const uint32_t q = (uint32_t)rintf((m - 1.0f) * 8.0f);               // exact product; 8 carries into the exponent
        code = ((uint32_t)(ex + 7) << 3) + q;
    }
    return sgn | min(code, 0x7eu);
}

// Row-wise FP8 quantisation straight into the streaming layout: one wave per (expert, matrix, row).  scale =
// amax / 448 (1 for an all-zero row), code = encode(w / scale), both divisions correctly rounded fp32.  A 1 KiB
// tile is 16 rows x 64 columns: lane l = row l%16, column group l/16 (16 consecutive columns = 16 bytes).
__global__ __launch_bounds__(256) void quantize_kernel(const uint16_t *__restrict__ Wa, const uint16_t *__restrict__ Wb,
                                                       int nmat, int E, int R, int K, uint8_t *__restrict__ out,
                                                       float *__restrict__ scales)
{
    const long row_id = (long)blockIdx.x * 4 + wave_id();   // (e, m, r)
    if (row_id >= (long)E * nmat * R) return;
    const int lane = lane_id();
    const int r = (int)(row_id % R);
    const int m = (int)((row_id / R) % nmat);
    const int e = (int)(row_id / ((long)R * nmat));
    const uint16_t *src = (m == 0 ? Wa : Wb) + ((size_t)e * R + r) * K;
    float amax = 0.f;
    for (int c = lane * 8; c < K; c += kWave * 8) {
        const uint4 v = *reinterpret_cast<const uint4 *>(src + c);
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            amax = fmaxf(amax, fabsf(__uint_as_float(w[i] << 16)));
            amax = fmaxf(amax, fabsf(__uint_as_float(w[i] & 0xffff0000u)));
        }
    }
    amax = wave_max(amax);
    const float sc = amax == 0.f ? 1.0f : __fdiv_rn(amax, 448.0f);
    if (lane == 0) scales[((size_t)e * nmat + m) * R + r] = sc;
    const int KT = K / 64;
    for (int c = lane * 16; c < K; c += kWave * 16) {   // 16 consecutive columns = one lane's piece of a tile
        uint32_t packed[4];
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            const uint4 v = *reinterpret_cast<const uint4 *>(src + c + half * 8);
            const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t lo = e4m3_encode(__fdiv_rn(__uint_as_float(w[i] << 16), sc));
                const uint32_t hi = e4m3_encode(__fdiv_rn(__uint_as_float(w[i] & 0xffff0000u), sc));
                const uint32_t two = lo | (hi << 8);
                if (i % 2 == 0)
                    packed[half * 2 + i / 2] = two;
                else
                    packed[half * 2 + i / 2] |= two << 16;
            }
        }
        const int kt = c / 64, g = (c % 64) / 16;
        const size_t piece = ((((size_t)e * (R / 16) + r / 16) * KT + kt) * nmat + m) * kWave + g * 16 + (r % 16);
        *reinterpret_cast<uint4 *>(out + piece * 16) = make_uint4(packed[0], packed[1], packed[2], packed[3]);
    }
}

// Nearest E2M1 code of q (already divided by the block scale): ties to the even code, magnitudes above 6 to 6.
// The thresholds are the midpoints of 0, 0.5, 1, 1.5, 2, 3, 4, 6; "<=" where the lower neighbour is the even code.
__device__ __forceinline__ uint32_t e2m1_encode(float q)
{
    const uint32_t sgn = (__float_as_uint(q) >> 31) << 3;
    const float a = fabsf(q);
    const uint32_t code = a <= 0.25f ? 0u : a < 0.75f ? 1u : a <= 1.25f ? 2u : a < 1.75f ? 3u : a <= 2.5f ? 4u : a < 3.5f ? 5u : a <= 5.0f ? 6u : 7u;
    return sgn | code;
}

// MXFP4 quantisation straight into the streaming layout: one wave per (expert, matrix, row), a lane per block of
// 32 columns.  Per block: E - 127 = floor(log2(amax)) - 2, clamped to [0, 254] (E = 127 for an all-zero block);
// code = encode(w * 2^(127 - E)), an exact scaling.  Weights: a 1 KiB tile is 16 rows x 128 columns, lane l = row
// l%16, block l/16, 16 bytes, byte j = columns 2j (low nibble) and 2j+1.  Scale exponents: byte kt%4 of dword
// [row group][kt/4][lane][which], (row group, which) = (row tile, matrix) for gate/up or (row pair, tile of the
// pair) for down.
__global__ __launch_bounds__(256) void quantize_fp4_kernel(const uint16_t *__restrict__ Wa, const uint16_t *__restrict__ Wb,
                                                           int nmat, int E, int R, int K, uint8_t *__restrict__ out,
                                                           uint8_t *__restrict__ scales)
{
    const long row_id = (long)blockIdx.x * 4 + wave_id();   // (e, m, r)
    if (row_id >= (long)E * nmat * R) return;
    const int lane = lane_id();
    const int r = (int)(row_id % R);
    const int m = (int)((row_id / R) % nmat);
    const int e = (int)(row_id / ((long)R * nmat));
    const uint16_t *src = (m == 0 ? Wa : Wb) + ((size_t)e * R + r) * K;
    const int KT = K / 128;
    const size_t KT4 = mx_kt4(K);
    const int groups = nmat == 2 ? R / 16 : R / 32;
    const int grp = nmat == 2 ? r / 16 : r / 32;
    const int which = nmat == 2 ? m : (r / 16) & 1;
    for (int c = lane * 32; c < K; c += kWave * 32) {
        uint32_t w[16];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint4 v = *reinterpret_cast<const uint4 *>(src + c + q * 8);
            w[4 * q] = v.x;
            w[4 * q + 1] = v.y;
            w[4 * q + 2] = v.z;
            w[4 * q + 3] = v.w;
        }
        float amax = 0.f;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            amax = fmaxf(amax, fabsf(__uint_as_float(w[i] << 16)));
            amax = fmaxf(amax, fabsf(__uint_as_float(w[i] & 0xffff0000u)));
        }
        int Eb = 127;
        if (amax > 0.f) {
            const uint32_t bits = __float_as_uint(amax);
            const int ef = (int)(bits >> 23);
            const int fl = ef != 0 ? ef - 127 : (31 - __clz((int)(bits & 0x007fffffu))) - 149;   // floor(log2(amax))
            Eb = min(max(fl - 2 + 127, 0), 254);
        }
        uint32_t packed[4];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const uint32_t lo = e2m1_encode(ldexpf(__uint_as_float(w[i] << 16), 127 - Eb));
            const uint32_t hi = e2m1_encode(ldexpf(__uint_as_float(w[i] & 0xffff0000u), 127 - Eb));
            const uint32_t byte = lo | (hi << 4);
            if (i % 4 == 0)
                packed[i / 4] = byte;
            else
                packed[i / 4] |= byte << (8 * (i % 4));
        }
        const int kt = c / 128, g = (c % 128) / 32;
        const int l = g * 16 + (r % 16);
        const size_t piece = ((((size_t)e * (R / 16) + r / 16) * KT + kt) * nmat + m) * kWave + l;
        *reinterpret_cast<uint4 *>(out + piece * 16) = make_uint4(packed[0], packed[1], packed[2], packed[3]);
        const size_t dword = (((size_t)e * groups + grp) * KT4 + kt / 4) * 128 + (size_t)l * 2 + which;
        scales[dword * 4 + (kt % 4)] = (uint8_t)Eb;
    }
}

// How many of a workgroup's four waves split the contraction dimension (the rest split rows).  Long
// per-wave streams amortise the fill and drain of the prefetch ring, so K is only split when the
// batch cannot invoke enough experts to give every CU several waves otherwise.
static int pick_k_waves(int K, int R, bool dual, int T, int max_experts, int bits_per_weight)
{
    // Gate/up: a wave streams a whole row tile of both matrices (2 * K * 32 bytes, contiguous); measured best
    // at every expert count.  It also makes a workgroup exactly one 64-row unit of the staged path.
    if (dual) return 1;
    // Down, more than 16 tokens: some expert may take the staged path, whose unit is 64 rows; two row groups
    // of 32 rows per workgroup cover exactly one (workgroups that only exist to be told they have nothing to
    // do are expensive).
    // Beyond 64 tokens (passes of up to 128 tokens): 128-row workgroups, whose staged passes give every wave two row
    // tiles that share each token fragment read from LDS (measured 2-4 % faster on every shape).
    // (not with quantised weights of at most eight experts whose 128-row workgroups are fewer than the CUs.  us per FFN call,
    // 128-row against 64-row workgroups, 100 tokens: 8 experts of 512 rows, F = 1024, FP8 17.5 against 16.5, MXFP4 16.6
    // against 16.0; 8 experts of 4096 rows, 256 workgroups, F = 14336, FP8 245 against 251, MXFP4 150 against 161.  The
    // limit of eight is part of the rule and not of the reason: with more experts and as few workgroups 64 rows are the
    // better ones too (16 experts of 1024 rows, F = 2048, 300 tokens, FP8 57.1 against 52.3), towards 256 workgroups it
    // goes either way (60 experts of 512 rows, FP8, 100 tokens 28.6 against 30.4, 600 tokens of F = 1408 55.6 against 53.0).)
    if (T > kTokBlock && !(bits_per_weight < 16 && max_experts <= 8 && (long)max_experts * R < 256 * 128)) return 1;
    if (T > kDirectMaxTokens) return 2;
    // Down, direct path only.  Measured: splitting K four ways pays when the batch can invoke so few experts
    // that whole row groups would leave the chip with too few, too long workgroups (Mixtral-like shapes); with
    // more experts two ways (64-row workgroups: 4-5 % faster than 128-row ones for DeepSeek-V2-Lite and
    // Qwen1.5-MoE shapes), unless the streams would get too short.
    const long group_bytes = (long)16 * K * 2 * bits_per_weight / 8;      // weight bytes behind one row group
    // Four only up to 8 tokens: with 16 rows per slice the token stage holds no more than a turn of the weight ring (less
    // with quantised weights, which cannot be; bf16, Mixtral shapes, 16 tokens: 427.7 us with four, 424.4 with two).
    int kw = max_experts <= 8 && T <= 8 ? 4 : 2;
    while (kw > 1 && group_bytes / kw < 32 * 1024) kw >>= 1;              // keep at least 32 KiB per wave
    return kw;
}

// Knobs that tuning runs and the test of the give-up path set through lynx_debug_set (lynx_bench.h); the defaults are
// what the library ships with.
struct Tunables {
    std::atomic<int> spin_limit{kSpinLimit};
    std::atomic<int> target_bias{0};
    std::atomic<int> dn_cap{768};      // down items the grid aims at (two per CU are resident: 512)
    std::atomic<int> dn_m_max{1};      // most row units per down item
    std::atomic<int> dn_kw{0};         // 0 = the rule of pick_k_waves, else the K slices of a down workgroup's waves
    std::atomic<int> wide{0};          // 1 = the wide kernel for every batch that it can take
};
static Tunables g_tune;

// Everything the host decides from the sizes alone.
struct FfnShape {
    int kwd;            // K slices of a down workgroup's waves
    int big;            // 0 = at most 64 tokens; 1, 2 = larger batches, gate/up units of 64 or of 128 rows; 3 = the wide kernel
    bool single;        // one launch for both projections
    int fill;           // > 0: two launches, and the device decides which of them runs the down workgroups (launch_shape)
    int tok_block;
    int rows_gu, rows_dn;   // rows of a gate/up unit, of a down workgroup
    int max_blocks;     // most (expert, token block) pairs of a batch
    PlanShape plan;
};

static bool single_launch(int T, int F) { return T >= 1 && (F + 63) / 64 <= 64; }   // (any batch size: see below)

// Quantised weights, huge experts, batches of 8 to 64 tokens: one launch all the same where the live down workgroups fill the
// chip.  They start in the slots that the last, partial round of gate/up workgroups leaves empty.  Too few of them lose: they go
// two to a CU as its slots come free, where a launch of their own spreads them, one to a CU.  us per layer, two launches
// against one, 8 experts of 4096 x 14336 of which so many are invoked:
//   FP8,   16 tokens, 64-row workgroups, 64 per expert:   2: 95 / 124   4: 143 / 154   5: 176 / 169   6: 194 / 185   8: 239 / 237
//   FP8,    8 tokens, 32-row workgroups, 128 per expert:  2: 82 / 98    3: 110 / 118   4: 133 / 130   6: 174 / 165   8: 221 / 216
//   MXFP4, 32 tokens, 64-row workgroups:                  2: 79 / 112   4: 101 / 118   5: 125 / 130   6: 129 / 127   8: 147 / 143
// and of 16 experts of 4096 x 8192, FP8, 64 tokens: 4: 107 / 123, 6: 138 / 133, 12: 234 / 225.  So the line lies at 384 live
// workgroups of 64 rows, 512 of 32.  How many are live, only the device knows: one launch where the fewest experts a
// batch can invoke (k) are enough, two where all of them are not, and otherwise down workgroups in both launches,
// of which those of one leave at once.  That costs 1 to 2.5 us of the one launch's gain, and up to 1.5 us beside two (the
// first line: 95.2, 143.4, 178.1, 187.8, 238.7).  bf16 weights gain 0 to 1.5 % with all eight experts and keep two.
static void launch_shape(FfnShape &s, int T, int F, int k, int max_experts, int format)
{
    s.single = single_launch(T, F);
    s.fill = 0;
    if (s.single || format == 0 || T < 8 || T > kTokBlock) return;
    const int enough = s.kwd == 4 ? 2 * kCus : 2 * kCus * 3 / 4;
    if ((long)s.plan.units_dn * max_experts < enough) return;
    if ((long)s.plan.units_dn * k >= enough)
        s.single = true;
    else
        s.fill = enough;
}

// The wide kernel pays with more than 128 tokens per expert on average, where its workgroups are long (a quarter of a wave's time
// is start and end at H = 2048) and several per CU.  us per FFN call, ffn_kernel against the wide one: Mixtral shapes, 300 tokens
// 602 against 657, 400 tokens 672 against 700, 520 tokens 757 -> 721, 700 tokens 837 -> 789, 1000 tokens 1142 -> 907; 12 experts of
// 4096 x 4096, 400 tokens 267 against 265, 1000 tokens 369 -> 319; 16 experts of 2048 x 2048 (four picks), 1000 tokens 169 against 169;
// 8 of them (two picks) 110 against 114; 8 experts of 2048 x 4096, 600 tokens 155 against 157.  us per layer: 60 experts of
// 4096 x 1536 (eight picks) 1024 tokens 639 -> 594, 32 of 4096 x 2048 and a shared one, 600 tokens 495 -> 437, 16 of 7168 x 2048
// (four picks) and a shared one, 1024 tokens 647 -> 535.
static bool wide_pays(int T, int H, int F, int N, int k, int format)
{
    if (format != 0 || T <= kTokBlock) return false;
    if (g_tune.wide.load()) return true;
    return H >= 4096 && (long)T * k > 128L * N && (long)F * T * k >= 240L * 128 * kWideTokens;
}

static FfnShape ffn_shape(int T, int H, int F, int N, int k, int n_shared, int format)
{
    FfnShape s;
    const int max_experts = (int)min((long)N, (long)T * k) + n_shared;
    s.kwd = pick_k_waves(F, H, false, T, max_experts, 16 >> format);
    const int forced = g_tune.dn_kw.load();
    if (forced == 1 || forced == 2 || (forced == 4 && T <= kDirectMaxTokens)) s.kwd = forced;
    // Gate/up units of 128 rows when the experts hold more than 64 tokens on average: fewer, longer workgroups that stage
    // the tokens half as often (Mixtral shapes, 1000 tokens: 1156 -> 1126 us; DeepSeek-V2-Lite shapes, 1000: 343 -> 333).
    // With fewer tokens the weight stream is the bound and the finer units fill the chip more evenly (Mixtral shapes, 128
    // tokens: 454 against 466 us, 256: 557 against 574).
    // MXFP4: from 32 tokens on average where the units fill the chip, since a unit's fixed work weighs more beside fewer
    // weight bytes (FFN calls: DeepSeek-V2-Lite shapes, 600 tokens 147 -> 137 us; Mixtral shapes, 200 tokens 252 -> 242;
    // Qwen1.5-MoE shapes, 500 tokens 128 -> 121; but Mixtral shapes, 100 tokens, 25 on average, 180 -> 183, and 8 experts of
    // 512 x 1024, 200 tokens, FP8 22.9 -> 25.3; FP8 with large experts -2 to +1 %).
    const bool sooner = format == 2 && (long)N * F >= 256L * 128 && (long)T * k >= 32L * N;
    const bool many = sooner || (long)T * k > (long)kTokBlock * N;
    s.big = T <= kTokBlock ? 0 : many ? 2 : 1;
    if (wide_pays(T, H, F, N, k, format)) {
        s.big = 3;
        s.kwd = 1;
    }
    s.tok_block = s.big == 3 ? kWideTokens : staged_tokens(s.big, format);
    s.max_blocks = plan_max_blocks(T, N, k, s.tok_block, false);
    s.plan.max_blocks = s.max_blocks;
    s.plan.shared_pairs = n_shared * (T > kDirectMaxTokens ? (T + s.tok_block - 1) / s.tok_block : 1);
    const int rows_dn = s.big == 3 ? 256 : 16 * (kFfnWaves / s.kwd) * 2;
    const int rows_gu = s.big == 3 ? 128 : 64 * staged_row_tiles(true, 1, s.big);
    s.rows_gu = rows_gu;
    s.rows_dn = rows_dn;
    s.plan.units_gu = (F + rows_gu - 1) / rows_gu;
    s.plan.units_dn = (H + rows_dn - 1) / rows_dn;
    launch_shape(s, T, F, k, max_experts, format);
    s.plan.tok_block = s.tok_block;
    // Longer down items only where the staged unit and the direct workgroup are the same 64 rows (two K slices).
    // (not in the large-batch kernels, whose items are single passes)
    s.plan.dn_m_max = s.kwd <= 2 && !s.big ? max(1, g_tune.dn_m_max.load()) : 1;
    s.plan.dn_cap = max(1, g_tune.dn_cap.load());
    return s;
}

PlanShape ffn_plan_shape(int T, int H, int F, int N, int k, int n_shared, int format)
{
    return ffn_shape(T, H, F, N, k, n_shared, format).plan;
}

static void set_tiles(GemmParams &p, int units_r, int rows_per_wg, int routed_items, int tok_block)
{
    p.tiles_r = units_r;
    // shared experts process all T tokens: staged (units of 64 rows, one per workgroup) when T is past the direct limit
    const int rows_shared = p.T > kDirectMaxTokens && p.T <= kTokBlock ? 64 : rows_per_wg;
    p.tiles_s = p.n_shared ? (p.Rs + rows_shared - 1) / rows_shared : 0;
    // ... and then a workgroup with all T tokens would make one pass per 64 tokens over the same weights and be by
    // far the longest of the launch: the passes go to workgroups of their own instead.
    p.tok_block = tok_block;
    p.shared_tblocks = p.T > kDirectMaxTokens ? (p.T + p.tok_block - 1) / p.tok_block : 1;
    p.tiles_s_stride = p.shared_tblocks > 1 ? (p.tiles_s + 7) / 8 * 8 : p.tiles_s;
    p.shared_blocks = p.n_shared * p.shared_splits * p.shared_tblocks * p.tiles_s_stride;
    p.routed_blocks = routed_items;
}

static unsigned grid_blocks(const GemmParams &p) { return (unsigned)(p.shared_blocks + p.routed_blocks); }

template <int KWD, int BIG, int WF>
static void launch_kernel(const FfnParams &fp, unsigned blocks, hipStream_t st)
{
    hipLaunchKernelGGL((ffn_kernel<KWD, BIG, WF>), dim3(blocks), dim3(kFfnThreads), 0, st, fp);
}

// One launch for both projections, or one each (the same kernel over its gate/up and its down workgroups)?
// Measured over the benchmark configurations: with experts of moderate size the single launch is 3-12 % faster beyond
// 16 tokens (the down projection fills the tail of gate/up and there is one start-up less) and 0-5 % faster up to 16
// (DeepSeek-V2-Lite shapes, 16 tokens: 87.6 -> 84.7 us per layer, remap off 150.0 -> 146.5; Qwen1.5-MoE shapes, 8
// tokens: 81.7 -> 81.7, remap off 92.3 -> 87.5); with huge experts it is
// equal or slower with bf16 weights (Mixtral shapes, 1 token 129 -> 140 us, 64 tokens equal, 200 tokens 505 -> 555: down
// workgroups that are few come to lie two to a CU) and faster with quantised ones between 8 and 64 tokens, if enough experts
// are invoked (launch_shape).

// Gate/up and down over all invoked and shared experts.  Batches of more than 64 tokens take the large-batch kernels, whose
// staged path makes passes of up to 128 tokens with bf16 weights, 64 with quantised ones, or the wide kernel with passes of up
// to 256 (wide_pays).
template <int WF>
static int launch_ffn(FfnParams fp, const FfnShape &sh, hipStream_t st)
{
    const GemmParams &d = fp.dn;
    set_tiles(fp.gu, sh.plan.units_gu, sh.rows_gu, sh.plan.units_gu * sh.max_blocks, sh.tok_block);
    set_tiles(fp.dn, sh.plan.units_dn, sh.rows_dn, plan_down_grid(sh.plan, sh.max_blocks), sh.tok_block);
    fp.gu.dn_m_max = fp.dn.dn_m_max = sh.plan.dn_m_max;
    // the split of the last round needs up to three more workgroups per workgroup it replaces
    // (not for batches of more than 32 tokens: more and more experts are then on the staged path, whose unit is the
    // whole workgroup of four row tiles, and three of the four small workgroups only find out that they leave;
    // measured equal or 3 us slower at 64 tokens, 3-8 us slower at 128 and 256)
    fp.gu_split = (WF == 0 && d.T <= kSplitMaxTokens && fp.gu.shared_blocks < kSplitRound) ? 1 : 0;
    fp.gu_blocks = (int)grid_blocks(fp.gu) + (fp.gu_split ? kSplitMaxRem * (kFfnWaves - 1) : 0);
    const unsigned dn_blocks = grid_blocks(fp.dn);
    // (live items are the first ones: the second of two launches that share them runs them only where they are fewer than fill)
    const unsigned dn_last = sh.fill > 0 ? min(dn_blocks, (unsigned)sh.fill) : dn_blocks;
    int rc = LYNX_OK;
    fp.fill = sh.fill;
    for (int part = 0; part < (sh.single ? 1 : 2) && rc == LYNX_OK; ++part) {
        const bool both = part == 0 && (sh.single || sh.fill > 0);
        fp.wait = both ? 1 : 0;
        fp.block0 = part == 0 ? 0 : fp.gu_blocks;
        const unsigned blocks = both ? (unsigned)fp.gu_blocks + dn_blocks : part == 0 ? (unsigned)fp.gu_blocks : dn_last;
        if (WF == 0 && sh.big == 3)
            hipLaunchKernelGGL(ffn_wide_kernel, dim3(blocks), dim3(kFfnThreads), 0, st, fp);
        else if (sh.big == 2 && sh.kwd == 1)
            launch_kernel<1, 2, WF>(fp, blocks, st);
        else if (sh.big == 2)
            launch_kernel<2, 2, WF>(fp, blocks, st);
        else if (sh.big && sh.kwd == 1)
            launch_kernel<1, 1, WF>(fp, blocks, st);
        else if (sh.big)
            launch_kernel<2, 1, WF>(fp, blocks, st);
        else if (sh.kwd == 4)
            launch_kernel<4, 0, WF>(fp, blocks, st);
        else if (sh.kwd == 2)
            launch_kernel<2, 0, WF>(fp, blocks, st);
        else
            launch_kernel<1, 0, WF>(fp, blocks, st);
        rc = check_launch("lynx_moe_ffn(gate/up, down)");
    }
    return rc;
}

}  // namespace lynx

extern "C" size_t lynx_workspace_bytes(int T, int H, int F, int N, int k, int n_shared, int F_shared)
{
    // (N does not enter: the tables per expert are reserved for LYNX_MAX_N experts)
    if (T < 0 || H < 0 || F < 0 || N < 0 || k < 0 || n_shared < 0 || F_shared < 0) return 0;
    if (n_shared == 0) F_shared = 0;
    return lynx::workspace_layout(T, H, F, k, n_shared, F_shared, lynx::shared_down_splits(F, n_shared, F_shared)).total;
}

extern "C" int lynx_moe_ffn_launches(int T, int F) { return lynx::single_launch(T, F) ? 1 : 2; }

extern "C" int lynx_debug_set(int what, int value)
{
    using namespace lynx;
    switch (what) {
    case LYNX_DEBUG_SPIN_LIMIT: g_tune.spin_limit.store(value < 0 ? kSpinLimit : value); return LYNX_OK;
    case LYNX_DEBUG_TARGET_BIAS: g_tune.target_bias.store(value); return LYNX_OK;
    case LYNX_DEBUG_DOWN_ITEM_CAP: g_tune.dn_cap.store(value <= 0 ? 768 : value); return LYNX_OK;
    case LYNX_DEBUG_DOWN_ITEM_UNITS: g_tune.dn_m_max.store(value <= 0 ? 1 : value); return LYNX_OK;
    case LYNX_DEBUG_DOWN_K_WAVES: g_tune.dn_kw.store(value <= 0 ? 0 : value); return LYNX_OK;
    case LYNX_DEBUG_WIDE_KERNEL: g_tune.wide.store(value <= 0 ? 0 : 1); return LYNX_OK;
    default: return fail(LYNX_ERR_INVALID_ARG, "lynx_debug_set: unknown knob %d", what);
    }
}

#ifdef LYNX_TIMELINE
// Measurement builds only: copies the timeline of the last expert-kernel launch to a HOST array of n x 6 uint64.
extern "C" int lynx_debug_timeline(unsigned long long *host_out, int n)
{
    if (n > lynx::kTimelineSlots) n = lynx::kTimelineSlots;
    return hipMemcpyFromSymbol(host_out, HIP_SYMBOL(lynx::g_timeline), (size_t)n * 6 * sizeof(unsigned long long)) == hipSuccess
               ? LYNX_OK
               : LYNX_ERR_HIP;
}
#endif

extern "C" int lynx_pack_weights(const uint16_t *Wg, const uint16_t *Wu, const uint16_t *Wd, int E, int H, int F,
                                 uint16_t *Wgu_packed, uint16_t *Wd_packed, void *stream)
{
    using namespace lynx;
    if (E < 0 || H <= 0 || F <= 0) return fail(LYNX_ERR_INVALID_ARG, "lynx_pack_weights: bad size");
    if ((H % 32) != 0 || (F % 32) != 0)
        return fail(LYNX_ERR_UNSUPPORTED, "lynx_pack_weights: H and F must be multiples of 32 (H=%d F=%d)", H, F);
    if (E == 0) return LYNX_OK;
    if (!Wg || !Wu || !Wd || !Wgu_packed || !Wd_packed) return fail(LYNX_ERR_INVALID_ARG, "lynx_pack_weights: null pointer");
    const size_t pieces_gu = (size_t)E * F * H * 2 / 8, pieces_d = (size_t)E * F * H / 8;
    if ((pieces_gu + 255) / 256 > 0x7fffffffull) return fail(LYNX_ERR_UNSUPPORTED, "lynx_pack_weights: too large for one call");
    hipLaunchKernelGGL(pack_kernel, dim3((unsigned)((pieces_gu + 255) / 256)), dim3(256), 0, (hipStream_t)stream, Wg, Wu,
                       2, E, F, H, Wgu_packed);
    int rc = check_launch("lynx_pack_weights(gate/up)");
    if (rc != LYNX_OK) return rc;
    hipLaunchKernelGGL(pack_kernel, dim3((unsigned)((pieces_d + 255) / 256)), dim3(256), 0, (hipStream_t)stream, Wd, Wd,
                       1, E, H, F, Wd_packed);
    return check_launch("lynx_pack_weights(down)");
}

namespace lynx {

// Every check of the FFN call that needs no device: sizes, limits, pointers.  lynx_moe_layer runs it before its
// routing kernels are enqueued, so that an error leaves nothing behind.
int moe_ffn_validate(const void *x_bf16, const void *Wgu_packed, const void *Wd_packed, const void *Sgu_packed,
                     const void *Sd_packed, int n_shared, int F_shared, const void *idx, const void *gate, const void *perm,
                     const void *offsets, int T, int H, int F, int N, int k, const void *y, const void *workspace,
                     const FfnScales *q8)
{
    if (T < 0 || H <= 0 || F <= 0 || N <= 0 || k <= 0 || n_shared < 0)
        return fail(LYNX_ERR_INVALID_ARG, "lynx_moe_ffn: bad size");
    if (n_shared > 0 && (F_shared <= 0 || !Sgu_packed || !Sd_packed))
        return fail(LYNX_ERR_INVALID_ARG, "lynx_moe_ffn: shared experts need F_shared > 0 and their weights");
    const int mult = q8 ? 32 << q8->format : 32;   // columns of a weight tile
    if ((H % mult) != 0 || (F % mult) != 0 || (n_shared > 0 && (F_shared % mult) != 0) || N > LYNX_MAX_N ||
        k > LYNX_MAX_K || T > LYNX_MAX_T || k > N)
        return fail(LYNX_ERR_UNSUPPORTED, "lynx_moe_ffn: need H,F,F_shared multiples of %d, k<=N<=%d, k<=%d, T<=%d", mult,
                    LYNX_MAX_N, LYNX_MAX_K, LYNX_MAX_T);
    if (q8 && (!q8->gu || !q8->d || (n_shared > 0 && (!q8->shared_gu || !q8->shared_d))))
        return fail(LYNX_ERR_INVALID_ARG, "lynx_moe_ffn_fp8: null scale pointer");
    if (T == 0) return LYNX_OK;
    if (!x_bf16 || !Wgu_packed || !Wd_packed || !idx || !gate || !offsets || !perm || !y || !workspace)
        return fail(LYNX_ERR_INVALID_ARG, "lynx_moe_ffn: null pointer");
    if (n_shared == 0) F_shared = 0;
    // (counted in blocks of 128 tokens, with quantised weights too: at most 768 pairs of them, 1536 of 64 tokens)
    const int tok_block = T > kTokBlock ? kTokBlockBig : kTokBlock;
    constexpr int kMaxSharedPairs = 768;
    static_assert(2 * kMaxSharedPairs <= kWsDoneSharedWords, "completion counters of the shared experts");
    if ((long)n_shared * ((T + tok_block - 1) / tok_block) > kMaxSharedPairs)
        return fail(LYNX_ERR_UNSUPPORTED, "lynx_moe_ffn: too many shared experts for this batch size (n_shared=%d T=%d)",
                    n_shared, T);
    const Workspace ws = workspace_layout(T, H, F, k, n_shared, F_shared, shared_down_splits(F, n_shared, F_shared));
    // (token rows are addressed with 32-bit byte offsets below 2 GiB)
    if (ws.h_elems >= 0x3fffffffull || (unsigned long long)T * H >= 0x3fffffffull || ws.o_elems >= 0x7fffffffull * 4)
        return fail(LYNX_ERR_UNSUPPORTED, "lynx_moe_ffn: scratch index would overflow 32 bits");
    return LYNX_OK;
}

// plan_ready: the caller has already had the completion counters in the workspace cleared and the work plan written
// on `stream` (the fused layer path does both in its routing kernels); otherwise a small launch does it here from
// expert_offsets.
int moe_ffn_impl(const uint16_t *x_bf16, const uint16_t *Wgu_packed, const uint16_t *Wd_packed, const uint16_t *Sgu_packed,
                 const uint16_t *Sd_packed, int n_shared, int F_shared, const int32_t *idx, const float *gate,
                 const int32_t *expert_offsets, const int32_t *perm, int T, int H, int F, int N, int k, float *y,
                 int32_t *status, void *workspace, void *stream, void *const *stage_events, bool plan_ready,
                 const FfnScales *q8)
{
    auto mark = [&](int i) -> int {
        if (!stage_events || !stage_events[i]) return LYNX_OK;
        const hipError_t err = hipEventRecord((hipEvent_t)stage_events[i], (hipStream_t)stream);
        return err == hipSuccess ? LYNX_OK : fail(LYNX_ERR_HIP, "lynx_moe_ffn_timed: hipEventRecord: %s", hipGetErrorString(err));
    };
    int rc = moe_ffn_validate(x_bf16, Wgu_packed, Wd_packed, Sgu_packed, Sd_packed, n_shared, F_shared, idx, gate, perm,
                              expert_offsets, T, H, F, N, k, y, workspace, q8);
    if (rc != LYNX_OK || T == 0) return rc;
    if (n_shared == 0) F_shared = 0;
    const int mult = q8 ? 32 << q8->format : 32;
    // K slices of a shared expert's down projection.  The workspace is sized for the most there can be; a slice holds
    // whole weight tiles, ceil(tiles / slices) of them, so fewer slices may already cover all tiles: an empty slice
    // would leave its output rows unwritten, and the combine adds every slice's rows.
    int splits = shared_down_splits(F, n_shared, F_shared);
    const Workspace ws = workspace_layout(T, H, F, k, n_shared, F_shared, splits);
    if (n_shared > 0) {
        const int kt = F_shared / mult;
        for (;;) {
            const int per = (kt + splits - 1) / splits;
            const int need = (kt + per - 1) / per;
            if (need == splits) break;
            splits = need;
        }
    }
    uint16_t *hbuf = reinterpret_cast<uint16_t *>(reinterpret_cast<char *>(workspace) + ws.h_off);
    float *obuf = reinterpret_cast<float *>(reinterpret_cast<char *>(workspace) + ws.o_off);
    int32_t *rws = reinterpret_cast<int32_t *>(workspace);
    hipStream_t st = (hipStream_t)stream;
    FfnShape shape = ffn_shape(T, H, F, N, k, n_shared, q8 ? q8->format : 0);
    if (!plan_ready) shape.max_blocks = shape.plan.max_blocks = plan_max_blocks(T, N, k, shape.tok_block, true);
    if (reinterpret_cast<uintptr_t>(x_bf16) % 16 != 0) {
        // Token rows of a tensor that starts at an odd place of its storage.  The loads into LDS take 16 bytes per lane and
        // are not known to take them from everywhere, so the rows are copied first: to the place of the per-pair outputs,
        // which the down projection writes, in a launch of its own then.
        hipLaunchKernelGGL(realign_kernel, dim3(1024), dim3(256), 0, st, x_bf16, reinterpret_cast<uint16_t *>(obuf), (size_t)T * H);
        rc = check_launch("lynx_moe_ffn(realign)");
        if (rc != LYNX_OK) return rc;
        x_bf16 = reinterpret_cast<const uint16_t *>(obuf);
        shape.single = false;
        shape.fill = 0;
    }
    if (!plan_ready) {
        hipLaunchKernelGGL(plan_kernel, dim3(1), dim3(256), 0, st, expert_offsets, perm, N, T * k, shape.plan, rws);
        rc = check_launch("lynx_moe_ffn(plan)");
        if (rc != LYNX_OK) return rc;
    }

    FfnParams fp;
    fp.done = rws + kWsDone;
    fp.flags = rws + kWsFlags;
    fp.gu_blocks = 0;
    fp.spin_limit = g_tune.spin_limit.load();
    fp.target_bias = g_tune.target_bias.load();
    GemmParams p;
    p.perm = perm;
    p.plan = rws;
    p.T = T;
    p.N = N;
    p.k = k;
    p.n_shared = n_shared;
    p.shared_splits = 1;
    p.shared_h_base = (long long)T * k * h_stride(F);
    // gate/up: rows = F, contraction = H
    p.W_routed = Wgu_packed;
    p.W_shared = Sgu_packed;
    p.B = x_bf16;
    p.out = hbuf;
    p.R = F;
    p.K = H;
    p.Rs = F_shared;
    p.Ks = H;
    p.sc_routed = q8 ? q8->gu : nullptr;
    p.sc_shared = q8 ? q8->shared_gu : nullptr;
    p.ldb_r = p.ldb_s = H;
    p.ldo_r = h_stride(F);
    p.ldo_s = h_stride(F_shared);
    fp.gu = p;
    // down: rows = H, contraction = F
    p.W_routed = Wd_packed;
    p.W_shared = Sd_packed;
    p.B = hbuf;
    p.out = obuf;
    p.R = H;
    p.K = F;
    p.Rs = H;
    p.Ks = F_shared;
    p.sc_routed = q8 ? q8->d : nullptr;
    p.sc_shared = q8 ? q8->shared_d : nullptr;
    p.ldb_r = h_stride(F);
    p.ldb_s = h_stride(F_shared);
    p.ldo_r = p.ldo_s = H;
    p.shared_splits = splits;
    fp.dn = p;
    rc = mark(0);
    if (rc != LYNX_OK) return rc;
    rc = !q8 ? launch_ffn<0>(fp, shape, st) : q8->format == 2 ? launch_ffn<2>(fp, shape, st) : launch_ffn<1>(fp, shape, st);
    if (rc != LYNX_OK) return rc;
    rc = mark(1);
    if (rc != LYNX_OK) return rc;
    rc = mark(2);
    if (rc != LYNX_OK) return rc;

    hipLaunchKernelGGL(combine_kernel, dim3((H / 4 + 255) / 256, T), dim3(256), 0, st, obuf, idx, gate, T, H, N, k,
                       n_shared * splits, y, fp.flags, status);
    rc = check_launch("lynx_moe_ffn(combine)");
    if (rc != LYNX_OK) return rc;
    return mark(3);
}

}  // namespace lynx

extern "C" int lynx_moe_ffn_timed(const uint16_t *x_bf16, const uint16_t *Wgu_packed, const uint16_t *Wd_packed,
                                  const uint16_t *Sgu_packed, const uint16_t *Sd_packed, int n_shared, int F_shared,
                                  const int32_t *idx, const float *gate, const int32_t *expert_offsets,
                                  const int32_t *perm, const int32_t *active_experts, const int32_t *num_active, int T,
                                  int H, int F, int N, int k, float *y, int32_t *status, void *workspace, void *stream,
                                  void *const *stage_events)
{
    (void)active_experts;   // the invoked experts are those with a non-empty range in expert_offsets
    (void)num_active;
    return lynx::moe_ffn_impl(x_bf16, Wgu_packed, Wd_packed, Sgu_packed, Sd_packed, n_shared, F_shared, idx, gate,
                              expert_offsets, perm, T, H, F, N, k, y, status, workspace, stream, stage_events, false,
                              nullptr);
}

extern "C" int lynx_moe_ffn_fp8(const uint16_t *x_bf16, const uint8_t *Wgu_q, const uint8_t *Wd_q, const float *scales_gu,
                                const float *scales_d, const uint8_t *Sgu_q, const uint8_t *Sd_q,
                                const float *shared_scales_gu, const float *shared_scales_d, int n_shared, int F_shared,
                                const int32_t *idx, const float *gate, const int32_t *expert_offsets, const int32_t *perm,
                                const int32_t *active_experts, const int32_t *num_active, int T, int H, int F, int N,
                                int k, float *y, int32_t *status, void *workspace, void *stream, void *const *stage_events)
{
    (void)active_experts;
    (void)num_active;
    const lynx::FfnScales q = {scales_gu, scales_d, shared_scales_gu, shared_scales_d, 1};
    return lynx::moe_ffn_impl(x_bf16, reinterpret_cast<const uint16_t *>(Wgu_q), reinterpret_cast<const uint16_t *>(Wd_q),
                              reinterpret_cast<const uint16_t *>(Sgu_q), reinterpret_cast<const uint16_t *>(Sd_q), n_shared,
                              F_shared, idx, gate, expert_offsets, perm, T, H, F, N, k, y, status, workspace, stream,
                              stage_events, false, &q);
}

extern "C" int lynx_quantize_weights_fp8(const uint16_t *Wg, const uint16_t *Wu, const uint16_t *Wd, int E, int H, int F,
                                         uint8_t *Wgu_q, uint8_t *Wd_q, float *scales_gu, float *scales_d, void *stream)
{
    using namespace lynx;
    if (E < 0 || H <= 0 || F <= 0) return fail(LYNX_ERR_INVALID_ARG, "lynx_quantize_weights_fp8: bad size");
    if ((H % 64) != 0 || (F % 64) != 0)
        return fail(LYNX_ERR_UNSUPPORTED, "lynx_quantize_weights_fp8: H and F must be multiples of 64 (H=%d F=%d)", H, F);
    if (E == 0) return LYNX_OK;
    if (!Wg || !Wu || !Wd || !Wgu_q || !Wd_q || !scales_gu || !scales_d)
        return fail(LYNX_ERR_INVALID_ARG, "lynx_quantize_weights_fp8: null pointer");
    const size_t rows_gu = (size_t)E * 2 * F, rows_d = (size_t)E * H;
    if ((rows_gu + 3) / 4 > 0x7fffffffull || (rows_d + 3) / 4 > 0x7fffffffull)
        return fail(LYNX_ERR_UNSUPPORTED, "lynx_quantize_weights_fp8: too large for one call");
    hipLaunchKernelGGL(quantize_kernel, dim3((unsigned)((rows_gu + 3) / 4)), dim3(256), 0, (hipStream_t)stream, Wg, Wu, 2, E,
                       F, H, Wgu_q, scales_gu);
    int rc = check_launch("lynx_quantize_weights_fp8(gate/up)");
    if (rc != LYNX_OK) return rc;
    hipLaunchKernelGGL(quantize_kernel, dim3((unsigned)((rows_d + 3) / 4)), dim3(256), 0, (hipStream_t)stream, Wd, Wd, 1, E,
                       H, F, Wd_q, scales_d);
    return check_launch("lynx_quantize_weights_fp8(down)");
}

extern "C" size_t lynx_fp4_scale_words(int E, int rows, int K, int gate_up)
{
    if (E < 0 || rows <= 0 || K <= 0) return 0;
    return (size_t)E * (gate_up ? lynx::mx_scale_dwords<true>(rows, K) : lynx::mx_scale_dwords<false>(rows, K));
}

extern "C" int lynx_quantize_weights_fp4(const uint16_t *Wg, const uint16_t *Wu, const uint16_t *Wd, int E, int H, int F,
                                         uint8_t *Wgu_q, uint8_t *Wd_q, uint32_t *scales_gu, uint32_t *scales_d,
                                         void *stream)
{
    using namespace lynx;
    if (E < 0 || H <= 0 || F <= 0) return fail(LYNX_ERR_INVALID_ARG, "lynx_quantize_weights_fp4: bad size");
    if ((H % 128) != 0 || (F % 128) != 0)
        return fail(LYNX_ERR_UNSUPPORTED, "lynx_quantize_weights_fp4: H and F must be multiples of 128 (H=%d F=%d)", H, F);
    if (E == 0) return LYNX_OK;
    if (!Wg || !Wu || !Wd || !Wgu_q || !Wd_q || !scales_gu || !scales_d)
        return fail(LYNX_ERR_INVALID_ARG, "lynx_quantize_weights_fp4: null pointer");
    const size_t rows_gu = (size_t)E * 2 * F, rows_d = (size_t)E * H;
    if ((rows_gu + 3) / 4 > 0x7fffffffull || (rows_d + 3) / 4 > 0x7fffffffull)
        return fail(LYNX_ERR_UNSUPPORTED, "lynx_quantize_weights_fp4: too large for one call");
    hipLaunchKernelGGL(quantize_fp4_kernel, dim3((unsigned)((rows_gu + 3) / 4)), dim3(256), 0, (hipStream_t)stream, Wg, Wu, 2,
                       E, F, H, Wgu_q, reinterpret_cast<uint8_t *>(scales_gu));
    int rc = check_launch("lynx_quantize_weights_fp4(gate/up)");
    if (rc != LYNX_OK) return rc;
    hipLaunchKernelGGL(quantize_fp4_kernel, dim3((unsigned)((rows_d + 3) / 4)), dim3(256), 0, (hipStream_t)stream, Wd, Wd, 1,
                       E, H, F, Wd_q, reinterpret_cast<uint8_t *>(scales_d));
    return check_launch("lynx_quantize_weights_fp4(down)");
}

extern "C" int lynx_moe_ffn_fp4(const uint16_t *x_bf16, const uint8_t *Wgu_q, const uint8_t *Wd_q, const uint32_t *scales_gu,
                                const uint32_t *scales_d, const uint8_t *Sgu_q, const uint8_t *Sd_q,
                                const uint32_t *shared_scales_gu, const uint32_t *shared_scales_d, int n_shared, int F_shared,
                                const int32_t *idx, const float *gate, const int32_t *expert_offsets, const int32_t *perm,
                                const int32_t *active_experts, const int32_t *num_active, int T, int H, int F, int N,
                                int k, float *y, int32_t *status, void *workspace, void *stream, void *const *stage_events)
{
    (void)active_experts;
    (void)num_active;
    const lynx::FfnScales q = {reinterpret_cast<const float *>(scales_gu), reinterpret_cast<const float *>(scales_d),
                               reinterpret_cast<const float *>(shared_scales_gu),
                               reinterpret_cast<const float *>(shared_scales_d), 2};
    return lynx::moe_ffn_impl(x_bf16, reinterpret_cast<const uint16_t *>(Wgu_q), reinterpret_cast<const uint16_t *>(Wd_q),
                              reinterpret_cast<const uint16_t *>(Sgu_q), reinterpret_cast<const uint16_t *>(Sd_q), n_shared,
                              F_shared, idx, gate, expert_offsets, perm, T, H, F, N, k, y, status, workspace, stream,
                              stage_events, false, &q);
}

extern "C" int lynx_moe_ffn(const uint16_t *x_bf16, const uint16_t *Wgu_packed, const uint16_t *Wd_packed,
                            const uint16_t *Sgu_packed, const uint16_t *Sd_packed, int n_shared, int F_shared,
                            const int32_t *idx, const float *gate, const int32_t *expert_offsets, const int32_t *perm,
                            const int32_t *active_experts, const int32_t *num_active, int T, int H, int F, int N, int k,
                            float *y, int32_t *status, void *workspace, void *stream)
{
    return lynx_moe_ffn_timed(x_bf16, Wgu_packed, Wd_packed, Sgu_packed, Sd_packed, n_shared, F_shared, idx, gate,
                              expert_offsets, perm, active_experts, num_active, T, H, F, N, k, y, status, workspace, stream,
                              nullptr);
}
