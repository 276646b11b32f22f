// The LDS-direct implicit-GEMM kernel, included by the files that instantiate it (conv_igemm.hip, gemm_ln.hip).
#pragma once
#include <atomic>

#include "activation.hpp"
#include "tiles.hpp"

namespace strait {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

enum { MODE_1X1 = 0, MODE_GATHER8 = 1, MODE_SCALAR = 2 };

// ------------------------------------------------------------------------------------------
// Deep-pipelined variant for the regular cases: dense 1x1 / GEMM, and filters whose channel count
// is a multiple of the 32-wide slice (so a slice never straddles two filter taps).
//
// conv_igemm_kernel (conv_igemm.hip) keeps one slice in flight per workgroup and spends most of its issue slots on
// per-lane gather arithmetic.  Here
//   - slices travel global -> LDS directly (buffer_load_dwordx4 ... lds: each lane names a 16-byte
//     chunk, the wave's 64 chunks land in 1 KB of consecutive LDS) through a ring of STAGES
//     buffers, one barrier per slice.  The operand fragments of a slice's first step are read right
//     after the barrier that hands the slice over, ahead of the MFMAs of the slice before it, and the
//     transfers that refill the freed buffer are issued between those MFMAs: a wavefront that is alone
//     on its SIMD keeps the MFMA pipe fed across the barrier (8192 x 768 x 3072 on 128 x 192: 46 -> 41.5 us;
//     what is left is LDS traffic, T per flop = 0.555 + 0.255 (LDS bytes per MFMA clock / 128) in 1 / PFLOP/s).
//     The last STAGES slices run in a loop of their own that requests nothing;
//   - the address of a chunk is split into a per-lane part fixed for the whole kernel (pixel or
//     channel row, chunk within the slice) held in a VGPR, and a part that is the same for the
//     whole workgroup (filter tap, channel base of the slice) kept in a scalar register and
//     advanced by scalar instructions: a weight load costs no vector instruction at all, an input
//     load one bit test and one select;
//   - whether tap (r,s) of an output pixel falls inside the image is precomputed per lane as a bit
//     mask over the taps; a tap outside, a row beyond M or a channel beyond Cout gets the offset
//     0x80000000, which the buffer's range check turns into zeros in LDS (no stale data, no branch);
//   - the hardware fixes the LDS position of lane i's chunk, so the bank-conflict-avoiding layout
//     is obtained from the other side: rows are 64 bytes (4 chunks) and lane i fetches logical
//     chunk (i & 3) ^ ((i >> 4) & 3) of its row, i.e. LDS holds chunk c of row r at position
//     c ^ ((r >> 2) & 3); any 16 consecutive rows read at one logical chunk then touch 16
//     distinct 16-byte bank groups;
//   - the loads are issued from inline assembly so that the waits are ours: "all but the newest
//     STAGES-2 slices have landed" before the barrier, rather than a wait for everything;
//   - tiles are dealt to the XCDs as rectangles (TileOrder): a batch of 8 sequences' Q/K/V product fetched its
//     3.5 MB of weights into all eight L2s before, and fetches a quarter of them into each now (13.6 -> 9.8 us).
typedef int intx4 __attribute__((ext_vector_type(4)));

constexpr unsigned OOB_OFFSET = 0x80000000u;       // beyond any buffer this kernel accepts

__device__ __forceinline__ intx4 make_rsrc(const void* base, unsigned bytes) {
    const unsigned long long a = (unsigned long long)base;
    intx4 r;
    r[0] = (int)(unsigned)a;
    r[1] = (int)((unsigned)(a >> 32) & 0xffffu);   // stride 0: raw buffer
    r[2] = (int)bytes;                              // num_records in bytes
    r[3] = 0x00020000;                              // 32-bit data format, offsets in bytes
    return r;
}

// One wave-wide transfer of 64 x 16 bytes: lane i's chunk at rsrc.base + voff + soff goes to
// LDS byte address lds_base + 16 i; lanes whose voff is out of range deposit zeros.
// (The offset is copied by a scalar instruction first: the compiler may have it from a vector one, v_readlane of a spilled register, after which a
// transfer may not read it for five wait states, and it does not count them for inline assembly.  The copy is also the wait that m0 needs.)
__device__ __forceinline__ void dma16(intx4 rsrc, unsigned voff, unsigned soff, unsigned lds_base) {
    const unsigned m0v = __builtin_amdgcn_readfirstlane(lds_base);
    unsigned so;
    asm volatile("s_mov_b32 m0, %1\n\ts_mov_b32 %0, %4\n\tbuffer_load_dwordx4 %2, %3, %0 offen lds" : "=&s"(so) : "s"(m0v), "v"(voff), "s"(rsrc), "s"(soff) : "memory");
}
template <int N>
__device__ __forceinline__ void wait_loads_then_barrier() {
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

// The kernels that hold a patch of the input in LDS, the next slice's on its way while nine tap steps run, and stream weights through a ring: transfers of
// the patch (npw per wavefront and slice, as per step) in step t
constexpr int patch_share(int npw, int as, int t) { return npw - t * as < 0 ? 0 : (npw - t * as > as ? as : npw - t * as); }

constexpr int patch_wait(int npw, int as, int wi, int pre, int t) {     // transfers a wave may have in flight when tap step t starts
    int n = patch_share(npw, as, (t + 9 - pre) % 9);
    for (int k = 1; k < pre; ++k) n += wi + patch_share(npw, as, (t + 9 - k) % 9);
    return n;
}

// Waves per SIMD that the LDS footprint of a tile configuration allows (the register allocator is asked
// for that many: left to itself it splits accumulators into AGPRs and loses waves for nothing).
template <int BM, int BN, int BK, int WGM, int WGN, int STAGES>
constexpr int dma_tile_waves_per_simd() {
    constexpr int ring = STAGES * (BM + BN) * BK * 2, ctile = BM * (BN + 8) * 2;
    constexpr int lds = (ring > ctile ? ring : ctile) + 1024;
    constexpr int blocks = 160 * 1024 / lds;
    constexpr int w = blocks * WGM * WGN / 4;
    return w < 1 ? 1 : (w > 8 ? 8 : w);
}

// KG > 1: the workgroup holds KG groups of WGM x WGN wavefronts, all on the same output tile; group g reduces the g-th
// part of the slices in a ring of its own, the groups step through their parts together (the barriers are the
// workgroup's), and at the end groups 1.. hand their partial sums to group 0 through LDS, which adds them in group
// order and finishes the tile.  A split reduction without a second launch, for the small batches where one more
// launch costs as much as the convolution.
//
// RES: how a residual is added.  RES_LATE: to the rounded product, fetched as the tile is stored.  RES_EARLY: likewise, but requested right
// after the reduction, before the staging barrier: that takes its latency off the path between the last MFMA and the stores.
// RES_WIDE, for few outputs behind a long reduction: it goes through the staging tile first and is added in fp32, so that the
// sum is rounded once, as in the second launch of a split reduction and in conv_skinny.hip.  (A 128-token sequence through twelve
// encoder layers: relative error against 64-bit arithmetic 1.42e-3, with a rounding before the add 1.46e-3.)
// RES_F32, for products with a LayerNorm folded in: requested as RES_EARLY does, and added in fp32 to a tile that is staged in fp32, in two
// halves where it does not fit in LDS at once.  (RES_WIDE on large tiles: 3 to 4 % of a whole encoder or ViT pass.)
enum { RES_LATE = 0, RES_EARLY = 1, RES_WIDE = 2, RES_F32 = 3 };
// RES_F32: rows staged at a time
template <int BM, int BN>
constexpr int f32_stage_rows() { return BM * (BN + 4) * 4 + 4096 <= 160 * 1024 ? BM : BM / 2; }

// LN: a LayerNorm between two products takes part in both of them instead of being a launch that reads and writes the tensor between
// them (gemm_ln.hip).  The producer (LN_OUT; LN_RES: its residual is itself such a tensor, normalised here as it is added) leaves, for
// every row and 64 channels of its rounded output, their sum and the sum of squares about their own mean; the consumer (LN_IN) multiplies
// the tensor as it is by weights that already hold gamma and corrects each output by its row's mean and deviation:
//     sum_k ((x_k - mu) rs gamma_k + beta_k) w_nk + b_n  =  rs (sum_k x_k w'_nk) - rs mu c_n + b'_n
// with w' = fp16(gamma w), c_n = sum_k w'_nk (of the rounded w', so that the mean cancels exactly) and b' = b + w beta.  The statistics travel to LDS
// ahead of the first slice and are combined beside the last ones' MFMAs, so that no wait is added.
enum { LN_NONE = 0, LN_IN = 1, LN_OUT = 2, LN_RES = 3 };
constexpr int LN_MAX_PARTS = 16, LN_MAX_PARTS_256 = 12;  // groups of 64 channels that a row's statistics may come in; on tiles of 256 channels
// what a tile's channels need besides the bias, the rows' two numbers, the rows' `parts` statistics (whole transfers of 1 KB)
template <int BM, int LN>
__host__ __device__ constexpr unsigned ln_lds_bytes(int parts) {
    return LN == LN_IN || LN == LN_RES ? (LN == LN_IN ? 1024u : 2048u) + BM * 8u + (unsigned)(BM * parts * 8 + 1023) / 1024u * 1024u : 0u;
}
__device__ __forceinline__ float sum_of_8_lanes(float v) {     // of the aligned eight lanes that this one belongs to
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0xB1, 0xf, 0xf, true));    // lane ^ 1
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x4E, 0xf, 0xf, true));    // lane ^ 2
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x141, 0xf, 0xf, true));   // the other four
    return v;
}

// DEEP, for tiles of few MFMAs per wavefront and step: operands are read from LDS three steps ahead and not one, so that a step does not wait for
// LDS, and reads are in flight across the barrier; a stage is filled again one slice later.  1024 x 3072 x 768 with GELU on 128 x 128 tiles of 8
// wavefronts 11.7 -> 11.2 us, 2758 x 768 x 3072 on 96 x 128 22.7 -> 21.2, 1379 x 768 x 3072 on 128 x 64 17.6 -> 16.5 (on the 64 x 128 tile that it had before, 18.2; all without a LayerNorm).  What is
// left is the rate of the transfers, 60 to 75 B/ns per compute unit whatever the tile: rings of 6 or 8 stages change nothing.
// Short reductions on the 128 x 128 tile are better off without (3136 x 1024 x 256 with a residual 7.3 and 7.6): there from 512 on.
template <int BM, int BN, int BK, int WGM, int WGN>
constexpr bool dma_deep() { return BK == 64 && ((BM == 96 && BN == 128) || (BM == 128 && (BN == 128 || BN == 64) && WGM * WGN == 8)); }
template <int BM, int BN, int BK, int WGM, int WGN, int MODE, int STAGES, bool GELU, int RES, bool DUAL = false, int KG = 1, int LN = LN_NONE, bool DEEP = dma_deep<BM, BN, BK, WGM, WGN>()>
__global__ void __launch_bounds__(64 * WGM * WGN * KG, (KG > 1 ? WGM * WGN * KG / 4 : dma_tile_waves_per_simd<BM, BN, BK, WGM, WGN, STAGES>())) conv_igemm_dma_kernel(const ConvParams p) {
    static_assert(!DUAL || (MODE == MODE_1X1 && RES == RES_LATE && !GELU), "a second source belongs to a plain pointwise convolution");
    static_assert(LN == LN_NONE || (MODE == MODE_1X1 && !DUAL && (LN == LN_IN ? RES == RES_LATE : !GELU && RES == RES_F32)), "LayerNorm belongs to dense products");
    static_assert(KG == 1 || (!GELU && !DUAL && KG * STAGES * (BM + BN) * BK * 2 + 1024 <= 160 * 1024 && WGM * WGN * KG <= 16), "groups: LDS or workgroup limit");
    constexpr int CPRW = BK / 8;                       // 16-byte chunks per LDS row
    constexpr int RPI = 64 / CPRW;                     // rows covered by one wave-wide transfer
    constexpr int SWD = 16 / CPRW;                     // rows that share a bank window
    constexpr int NW = WGM * WGN, NT = 64 * NW;        // the waves form a WGM x WGN grid over the tile
    constexpr int TM = BM / WGM, TN = BN / WGN;
    constexpr int TMB = TM / 32, TNB = TN / 32;
    constexpr int XI = BM / (NW * RPI), WI = BN / (NW * RPI); // transfers per wave per slice
    static_assert((BK == 32 || BK == 64) && TM % 32 == 0 && TN % 32 == 0 && BM % (NW * RPI) == 0 && BN % (NW * RPI) == 0, "unsupported tile");
    static_assert((NW * RPI) % (SWD * CPRW) == 0, "the swizzle of a lane's row has to be the same in all of its transfers");
    constexpr int STAGE = (BM + BN) * BK;              // halfs per stage
    constexpr int LDC = BN + 8;
    static_assert(MODE == MODE_1X1 || MODE == MODE_GATHER8, "vector modes only");
    static_assert(STAGES >= 2 && STAGES * STAGE * 2 <= 160 * 1024 && BM * LDC * 2 <= 160 * 1024, "LDS limit");

    extern __shared__ __attribute__((aligned(1024))) half_t smem_all[];    // max(KG * STAGES * STAGE, BM * LDC) halfs
    const int group = KG > 1 ? __builtin_amdgcn_readfirstlane((int)threadIdx.x / NT) : 0;
    half_t* const smem = smem_all + group * (STAGES * STAGE);          // this group's ring
    const unsigned lds0 = (unsigned)(uintptr_t)smem;

    if (p.hp) __builtin_amdgcn_s_setprio(3);

    const int tid = (int)threadIdx.x - group * NT;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm0 = (wave % WGM) * TM, wn0 = (wave / WGM) * TN;
    const int l32 = lane & 31, lh = lane >> 5;

    const int logical = xcd_range(p.order.tiles * (KG > 1 ? 1 : p.ksplit), blockIdx.x);
    // split-K: the grid holds ksplit copies of the tile grid; copy z reduces slices [k_begin, k_end)
    int zsplit = 0, tile = logical;
    if (KG > 1) zsplit = group;
    else if (p.ksplit > 1) {
        zsplit = divide(logical, p.order.by_tiles);
        tile = logical - zsplit * p.order.tiles;
    }
    int tm, tn;
    place_tile(p.order, tile, tm, tn);
    const int m0 = tm * BM;
    const int n0 = tn * BN;

    // The input buffer starts `lead` elements before x so that the per-lane offset of an output
    // pixel (its window's top-left tap, which may lie in the padding) is never negative.
    const long long lead = (long long)p.pad_h * p.sH + (long long)p.pad_w * p.sW;
    const intx4 xrsrc = make_rsrc(p.x - lead, (unsigned)((p.x_elems + lead) * 2));
    const intx4 wrsrc = make_rsrc(p.w, (unsigned)((long long)p.Cout * p.ldw * 2));

    // ---- per-lane constants: row (lane >> 2) of each 16-row group, logical chunk cl ---------------
    const int rsub = lane / CPRW;
    const int cl = (lane % CPRW) ^ (((wave * RPI + rsub) / SWD) & (CPRW - 1));
    unsigned xoff[XI], tapmask[XI];
#pragma unroll
    for (int j = 0; j < XI; ++j) {
        const int m = m0 + (j * NW + wave) * RPI + rsub;
        xoff[j] = OOB_OFFSET;
        tapmask[j] = 0xffffffffu;
        if (m < p.M) {
            if (MODE == MODE_1X1 && p.stride_h == 1) {
                xoff[j] = (unsigned)(((long long)m * p.sW + cl * 8) * 2);
            } else {
                const int n = divide(m, p.by_pq), rem = m - n * p.PQ;
                const int pp = divide(rem, p.by_q), qq = rem - pp * p.Q;
                const int ih0 = pp * p.stride_h - p.pad_h, iw0 = qq * p.stride_w - p.pad_w;
                xoff[j] = (unsigned)(((long long)n * p.sN + (long long)(pp * p.stride_h) * p.sH +
                                      (long long)(qq * p.stride_w) * p.sW + cl * 8) * 2);
                if (MODE == MODE_GATHER8) {
                    tapmask[j] = taps_inside(p, ih0, iw0);
                }
            }
        }
    }
    // DUAL: the slices from p.C on come from the second tensor, addressed by output pixel with its own strides
    const intx4 xrsrc2 = DUAL ? make_rsrc(p.x2, (unsigned)(p.x2_elems * 2)) : xrsrc;
    unsigned xoff2[DUAL ? XI : 1];
    if (DUAL) {
#pragma unroll
        for (int j = 0; j < XI; ++j) {
            const int m = m0 + (j * NW + wave) * RPI + rsub;
            xoff2[j] = OOB_OFFSET;
            if (m < p.M) {
                const int n = divide(m, p.by_pq), rem = m - n * p.PQ;
                const int pp = divide(rem, p.by_q), qq = rem - pp * p.Q;
                xoff2[j] = (unsigned)(((long long)n * p.sN2 + (long long)(pp * p.stride2) * p.sH2 +
                                       (long long)(qq * p.stride2) * p.sW2 + cl * 8) * 2);
            }
        }
    }
    unsigned woff[WI];
#pragma unroll
    for (int j = 0; j < WI; ++j) {
        const int n = n0 + (j * NW + wave) * RPI + rsub;
        woff[j] = n < p.Cout ? (unsigned)(((long long)n * p.ldw + cl * 8) * 2) : OOB_OFFSET;
    }

    // ---- workgroup-uniform position of the slice being issued ---------------------------------
    const int nk_all = (p.Kg + BK - 1) / BK;
    const int kchunk = p.kchunk;
    const int k_begin = zsplit * kchunk;
    const int k_end = k_begin + kchunk < nk_all ? k_begin + kchunk : nk_all;
    // (the groups of one workgroup share its barriers: all of them take kchunk steps, slices past a group's part arrive as zeros)
    const int nk = KG > 1 ? kchunk : (k_end > k_begin ? k_end - k_begin : 0);
    const bool ragged_k = (p.Kg & (BK - 1)) != 0;      // only possible for 1x1 / GEMM
    int ki = k_begin;                                  // slice index
    int tap = 0, ts = 0, cb = 0;                       // filter tap, its column, channel base
    unsigned tap_off = 0;                              // byte offset of the tap: (r*sH + s*sW) * 2
    if (MODE == MODE_GATHER8 && k_begin > 0) {
        tap = divide(k_begin * BK, p.by_c);
        cb = k_begin * BK - tap * p.C;
        const int r0 = divide(tap, p.by_s);
        ts = tap - r0 * p.S;
        tap_off = (unsigned)(r0 * p.sH + ts * p.sW) * 2u;
    }
    const unsigned row_step = (unsigned)(p.sH - p.S * p.sW) * 2u;   // from the end of a filter row to the next

    // one transfer (j-th of this wave's XI + WI) of the slice being issued
    auto issue_one = [&](int stage, int j) __attribute__((always_inline)) {
        const unsigned sx = lds0 + (unsigned)(stage * STAGE) * 2u;
        const unsigned sw = sx + (unsigned)(BM * BK) * 2u;
        const bool live = ki < k_end;                  // slices past the end deposit zeros
        if (j < XI) {
            const bool second = DUAL && ki * BK >= p.C;   // workgroup-uniform
            const unsigned soff_x = LN != LN_NONE ? (unsigned)ki * p.x_slice : MODE == MODE_1X1 ? (unsigned)(second ? ki * BK - p.C : ki * BK) * 2u : tap_off + (unsigned)cb * 2u;
            unsigned v = xoff[j];
            if (DUAL && second) v = xoff2[j];
            if (MODE == MODE_GATHER8) v = ((tapmask[j] >> tap) & 1u) ? v : OOB_OFFSET;
            if (MODE == MODE_1X1 && ragged_k) v = (ki * BK + cl * 8 < p.Kg) ? v : OOB_OFFSET;
            if (!live) v = OOB_OFFSET;
            dma16(second ? xrsrc2 : xrsrc, v, live ? soff_x : 0u, sx + (unsigned)((j * NW + wave) * 1024));
        } else {
            const int jw = j - XI;
            unsigned v = woff[jw];                     // (a weight row's ragged end is followed by the next row, which may hold infinities)
            if (MODE == MODE_1X1 && ragged_k) v = (ki * BK + cl * 8 < p.Kg) ? v : OOB_OFFSET;
            dma16(wrsrc, live ? v : OOB_OFFSET, live ? (unsigned)ki * (BK * 2) : 0u, sw + (unsigned)((jw * NW + wave) * 1024));
        }
    };
    auto advance = [&]() __attribute__((always_inline)) {
        ++ki;
        if (MODE == MODE_GATHER8) {
            cb += BK;
            if (cb >= p.C) {
                cb = 0;
                ++tap;
                tap_off += (unsigned)p.sW * 2u;
                if (++ts == p.S) { ts = 0; tap_off += row_step; }
            }
        }
    };
    auto issue = [&](int stage) {
#pragma unroll
        for (int j = 0; j < XI + WI; ++j) issue_one(stage, j);
        advance();
    };

    floatx16 acc[TNB][TMB];
#pragma unroll
    for (int a = 0; a < TNB; ++a)
#pragma unroll
        for (int b = 0; b < TMB; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.f;

    // The tile's bias row goes to LDS with the very first transfer (channels past Cout, or no bias at all,
    // arrive as zeros), so that the epilogue does not start with a round trip to L2.
    constexpr int CTILE = RES == RES_F32 ? f32_stage_rows<BM, BN>() * (BN + 4) * 4 : BM * LDC * 2;
    constexpr unsigned BIAS_LDS = KG * STAGES * STAGE * 2 > CTILE ? KG * STAGES * STAGE * 2 : CTILE;   // byte offset
    static_assert(BN <= 256, "bias row: one transfer carries 256 floats");
    constexpr unsigned ROWS_LDS = BIAS_LDS + (LN == LN_IN ? 2048u : 3072u), PARTS_LDS = ROWS_LDS + BM * 8;   // LN_IN, LN_RES: [BM] float2; [BM][ln_parts]
    const int ln_parts = (LN == LN_IN ? p.Kg : p.Cout) >> 6;
    if (LN == LN_IN || LN == LN_RES) {
        // the tile's rows' statistics lie in one piece; rows past the end arrive as zeros
        static_assert(LN == LN_NONE || BM * 8 % 256 == 0, "alignment");
        const intx4 srsrc = make_rsrc(p.ln_stats, (unsigned)((long long)p.M * ln_parts * 8));
        const unsigned piece = (unsigned)(BM * ln_parts * 8), at = (unsigned)m0 * (unsigned)ln_parts * 8u;
        for (unsigned o = wave * 1024u; o < piece; o += NW * 1024u)
            dma16(srsrc, o + lane * 16u < piece ? at + o + lane * 16u : OOB_OFFSET, 0u, (unsigned)(uintptr_t)smem_all + PARTS_LDS + o);
    }
    auto channel_row = [&](const float* src, unsigned at) __attribute__((always_inline)) {
        const intx4 brsrc = make_rsrc(src, src ? (unsigned)p.Cout * 4u : 0u);
        const int c = n0 + lane * 4;
        dma16(brsrc, (src && lane * 4 < BN && c + 3 < p.Cout) ? (unsigned)c * 4u : OOB_OFFSET, 0u, (unsigned)(uintptr_t)smem_all + at);
    };
    if (wave == 0) {                                   // (every group fetches it, so that the wavefronts' transfer counts agree)
        channel_row(p.bias, BIAS_LDS);
        if (LN == LN_IN) channel_row(p.ln_csum, BIAS_LDS + 1024u);
        if (LN == LN_RES) { channel_row(p.ln_g, BIAS_LDS + 1024u); channel_row(p.ln_b, BIAS_LDS + 2048u); }
    }

#pragma unroll
    for (int i = 0; i < (DEEP ? STAGES - 1 : STAGES); ++i) if (i == 0 || i < nk) issue(i);

    const int swz = (l32 / SWD) & (CPRW - 1);
    constexpr int KS = BK / 16;
    half8 wf[DEEP ? KS : 2][TNB], xf[DEEP ? KS : 2][TMB];
    auto load_frags = [&](int buf, int stage, int ks) __attribute__((always_inline)) {
        const half_t* Xs = smem + stage * STAGE;
        const half_t* Ws = Xs + BM * BK;
        const int pos = ((ks * 2 + lh) ^ swz) * 8;
#pragma unroll
        for (int a = 0; a < TNB; ++a) wf[buf][a] = *(const half8*)(Ws + (wn0 + a * 32 + l32) * BK + pos);
#pragma unroll
        for (int b = 0; b < TMB; ++b) xf[buf][b] = *(const half8*)(Xs + (wm0 + b * 32 + l32) * BK + pos);
    };
    constexpr int NX = XI + WI, NM = TMB * TNB, PER = (NX + NM - 1) / NM;   // transfers per slice, MFMAs per step, transfers per MFMA
    // LN_IN, LN_RES: in every wavefront once the first slice is there
    auto ln_combine = [&]() __attribute__((always_inline)) {
    if (LN == LN_IN || LN == LN_RES) {
        // the row's mean and deviation from its parts (sum s, sum of squares q about the part's own mean): two threads a row, every other part each
        static_assert(LN == LN_NONE || LN == LN_OUT || NT >= 2 * BM, "two threads per row");
        const float2* parts = (const float2*)((const char*)smem_all + PARTS_LDS) + (tid >> 1) * ln_parts;
        float2 pt[LN_MAX_PARTS / 2];
        float s = 0.f, q = 0.f;
#pragma unroll
        for (int i = 0; i < LN_MAX_PARTS / 2; ++i) {
            const int k = 2 * i + (tid & 1);
            pt[i] = parts[k < ln_parts ? k : 0];
            s += k < ln_parts ? pt[i].x : 0.f;
        }
        s += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, s), 0xB1, 0xf, 0xf, true));
        const float mean = s / (float)(64 * ln_parts);       // (not times the reciprocal, which misses the number that a row of equal ones consists of: 7, 13, 14 and 15 parts)
#pragma unroll
        for (int i = 0; i < LN_MAX_PARTS / 2; ++i) {
            const float d = pt[i].x * (1.f / 64.f) - mean;
            q += 2 * i + (tid & 1) < ln_parts ? pt[i].y + 64.f * d * d : 0.f;
        }
        q += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, q), 0xB1, 0xf, 0xf, true));
        const float rs = __builtin_amdgcn_rsqf(q * p.ln_inv_n + p.ln_eps);
        // (a row of equal numbers is beta alone: nothing of the products' rounding may be scaled up)
        if (tid < 2 * BM && (tid & 1) == 0 && (KG == 1 || group == 0))
            *(float2*)((char*)smem_all + ROWS_LDS + (tid >> 1) * 8) = q == 0.f ? make_float2(0.f, 0.f) : make_float2(rs, -rs * mean);
    }
    };
    if constexpr (DEEP) {
        static_assert(KS == 4 && STAGES >= 4, "four steps a slice, and a stage that is being left");
        if (nk >= STAGES - 1) wait_loads_then_barrier<(STAGES - 2) * NX>(); else wait_loads_then_barrier<0>();
#pragma unroll
        for (int k = 0; k < 3; ++k) load_frags(k, 0, k);
        int rd = 0, fill = STAGES - 1;                 // stage in use, stage to fill (left by everyone at the barrier inside a slice)
        auto slice = [&](auto refillc, auto nextc) __attribute__((always_inline)) {
            constexpr bool REFILL = decltype(refillc)::value, NEXT = decltype(nextc)::value;
            const int nrd = rd + 1 == STAGES ? 0 : rd + 1;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                if (ks == 0) load_frags(KS - 1, rd, KS - 1);
                else if (NEXT) {
                    if (ks == 1) {
                        // slice kt + 1 has landed everywhere, and everyone has multiplied with slice kt - 1
                        if (REFILL) asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((STAGES - 3) * NX) : "memory");
                        else asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
                    }
                    load_frags(ks - 1, nrd, ks - 1);
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int q = 0; q < NM; ++q) {
                    const int a = q / TMB, b = q % TMB;
                    acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(wf[ks][a], xf[ks][b], acc[a][b], 0, 0, 0);
                    if (REFILL && ks > 0) {
                        constexpr int SLOTS = (KS - 1) * NM, EACH = (NX + SLOTS - 1) / SLOTS;   // transfers between two MFMAs
#pragma unroll
                        for (int j = ((ks - 1) * NM + q) * EACH; j < ((ks - 1) * NM + q + 1) * EACH && j < NX; ++j) issue_one(fill, j);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            if (REFILL) { advance(); fill = fill + 1 == STAGES ? 0 : fill + 1; }
            rd = nrd;
        };
        int kt = 0;
        for (; kt + STAGES - 1 < nk; ++kt) slice(std::true_type{}, std::true_type{});
        ln_combine();
        for (; kt + 1 < nk; ++kt) slice(std::false_type{}, std::true_type{});
        if (kt < nk) slice(std::false_type{}, std::false_type{});
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    } else {
    int rd = 0;
    if (nk >= STAGES) wait_loads_then_barrier<(STAGES - 1) * NX>(); else wait_loads_then_barrier<0>();
    load_frags(0, 0, 0);
    // main part: every step requests a further slice; tail: the last STAGES slices, nothing left to request
    const int nmain = nk - STAGES;
    for (int kt = 0; kt < nmain; ++kt) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const int frd = rd;
            if (ks + 1 < KS) load_frags((ks + 1) & 1, rd, ks + 1);
            else {
                wait_loads_then_barrier<(STAGES - 2) * NX>();   // slice kt + 1 has landed everywhere; slice kt's buffer is free
                rd = rd + 1 == STAGES ? 0 : rd + 1;
                load_frags((ks + 1) & 1, rd, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int q = 0; q < NM; ++q) {
                const int a = q / TMB, b = q % TMB;
                acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(wf[ks & 1][a], xf[ks & 1][b], acc[a][b], 0, 0, 0);
                if (ks == KS - 1) {
#pragma unroll
                    for (int j = q * PER; j < (q + 1) * PER && j < NX; ++j) issue_one(frd, j);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            if (ks == KS - 1) advance();
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    ln_combine();
    for (int kt = nmain > 0 ? nmain : 0; kt < nk; ++kt) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            if (ks + 1 < KS) load_frags((ks + 1) & 1, rd, ks + 1);
            else {
                wait_loads_then_barrier<0>();
                rd = rd + 1 == STAGES ? 0 : rd + 1;
                load_frags((ks + 1) & 1, rd, 0);                 // (after the last slice: whatever the buffer holds, not used)
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int q = 0; q < NM; ++q) {
                const int a = q / TMB, b = q % TMB;
                acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(wf[ks & 1][a], xf[ks & 1][b], acc[a][b], 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    }
    __syncthreads();                                   // LDS is free

    // ---- groups: partial sums of groups 1.. to group 0 through LDS, added in group order ----------------------
    if (KG > 1) {
        float* xch = (float*)smem_all;                 // [KG - 1][NW][TNB * TMB * 16][64 lanes]
        if (group > 0) {
            float* dst = xch + ((group - 1) * NW + wave) * (TNB * TMB * 16 * 64) + lane;
#pragma unroll
            for (int a = 0; a < TNB; ++a)
#pragma unroll
                for (int b = 0; b < TMB; ++b)
#pragma unroll
                    for (int v = 0; v < 16; ++v) dst[((a * TMB + b) * 16 + v) * 64] = acc[a][b][v];
        }
        __syncthreads();
        if (group == 0) {
            for (int g = 1; g < KG; ++g) {
                const float* src = xch + ((g - 1) * NW + wave) * (TNB * TMB * 16 * 64) + lane;
#pragma unroll
                for (int a = 0; a < TNB; ++a)
#pragma unroll
                    for (int b = 0; b < TMB; ++b)
#pragma unroll
                        for (int v = 0; v < 16; ++v) acc[a][b][v] += src[((a * TMB + b) * 16 + v) * 64];
            }
        }
        __syncthreads();                               // before the epilogue parks the output tile in the same memory
    }
    const bool finisher = KG == 1 || group == 0;       // the other groups only keep the epilogue's barrier company

    // ---- split-K: fp32 partial sums to this copy's slab; a second kernel reduces and finishes ------
    if (p.ksplit > 1) {
        float* slab = p.ws + (long long)zsplit * p.M * p.Cout;
#pragma unroll
        for (int a = 0; a < TNB; ++a)
#pragma unroll
            for (int b = 0; b < TMB; ++b) {
                const int m = m0 + wm0 + b * 32 + l32;
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int n = n0 + wn0 + a * 32 + 8 * g + 4 * lh;
                    if (m < p.M && n < p.Cout) {
                        float4 v = make_float4(acc[a][b][4 * g], acc[a][b][4 * g + 1], acc[a][b][4 * g + 2], acc[a][b][4 * g + 3]);
                        *(float4*)(slab + (long long)m * p.Cout + n) = v;
                    }
                }
            }
        return;
    }

    // ---- epilogue (as the staged path of conv_igemm_kernel in conv_igemm.hip) --------------------------------------
    // ReLU / ReLU6 / none are one clamp with workgroup-uniform bounds; GELU is a separate instantiation
    // The epilogue's arithmetic after the bias is done on packed fp16 pairs: adding two fp16 numbers, or
    // clamping one against 0, 6 or an infinity, gives the same fp16 result whether it is done in fp16 or
    // in fp32 and then rounded, and it takes a quarter of the instructions (short-reduction layers spend
    // most of their instructions here).  Bias and residual are fetched where they are used: holding
    // them across the reduction would cost a wave per SIMD in registers.
    constexpr int CPR = BN / 8, NCH = BM * CPR / NT;
    half_t* Cs = smem_all;
    const bool fuse_act = RES == RES_WIDE || p.res == nullptr;
    const half_t lo = (p.act == ACT_RELU || p.act == ACT_RELU6) ? (half_t)0.f : (half_t)-INFINITY;
    const half_t hi = p.act == ACT_RELU6 ? (half_t)6.f : (half_t)INFINITY;
    const half_t lo1 = fuse_act ? lo : (half_t)-INFINITY, hi1 = fuse_act ? hi : (half_t)INFINITY;
    const half4 lo4 = {lo1, lo1, lo1, lo1}, hi4 = {hi1, hi1, hi1, hi1};
    const half8 lo8 = {lo, lo, lo, lo, lo, lo, lo, lo}, hi8 = {hi, hi, hi, hi, hi, hi, hi, hi};
    auto residual_chunk = [&](int i) {
        const int id = tid + i * NT;
        const int row = id / CPR, c8 = id - row * CPR;
        const int m = m0 + row, n = n0 + c8 * 8;
        half8 r;
#pragma unroll
        for (int j = 0; j < 8; ++j) r[j] = (half_t)0.f;
        if (m < p.M && n < p.Cout) r = *(const half8*)(p.res + (long long)m * p.ldy + n);
        return r;
    };
    const float* bias_s = (const float*)((const char*)smem_all + BIAS_LDS);
    auto bias4 = [&](int a, int g, float (&bv)[4]) {
        const float4 b4 = *(const float4*)(bias_s + wn0 + a * 32 + 8 * g + 4 * lh);
        bv[0] = b4.x; bv[1] = b4.y; bv[2] = b4.z; bv[3] = b4.w;
    };
    half8 rv[RES == RES_EARLY || RES == RES_F32 ? NCH : 1];
    if ((RES == RES_EARLY || RES == RES_F32) && !fuse_act && finisher) {
#pragma unroll
        for (int i = 0; i < NCH; ++i) rv[i] = residual_chunk(i);
    }
    if (RES == RES_WIDE) {
        if (finisher) {
#pragma unroll
            for (int i = 0; i < NCH; ++i) {
                const int id = tid + i * NT, row = id / CPR, c8 = id - row * CPR;
                *(half8*)(Cs + row * LDC + c8 * 8) = residual_chunk(i);
            }
        }
        __syncthreads();
    }
    float2 rows[LN == LN_IN ? TMB : 1];
    if (LN == LN_IN) {
#pragma unroll
        for (int b = 0; b < TMB; ++b) rows[b] = *(const float2*)((const char*)smem_all + ROWS_LDS + (wm0 + b * 32 + l32) * 8);
    }
    if (RES == RES_F32) {
        constexpr int SR = f32_stage_rows<BM, BN>(), PASSES = BM / SR, LDF = BN + 4;
        static_assert(RES != RES_F32 || (SR % TM == 0 && NCH % PASSES == 0), "a wavefront's rows are staged in one go");
        float* Fs = (float*)smem_all;
        // gamma and beta of a thread's eight channels, which are the same in all of its rows unless the tile's rows are no divisor of the workgroup
        constexpr bool SAME_C = NT % CPR == 0;
        float4 gq[2], bq[2];
        auto load_gb = [&](int c8) __attribute__((always_inline)) {
#pragma unroll
            for (int h = 0; h < 2; ++h) { gq[h] = *(const float4*)(bias_s + 256 + c8 * 8 + h * 4); bq[h] = *(const float4*)(bias_s + 512 + c8 * 8 + h * 4); }
        };
        if (LN == LN_RES && SAME_C) load_gb(tid % CPR);
#pragma unroll
        for (int ps = 0; ps < PASSES; ++ps) {
            if (finisher && wm0 / SR == ps) {
#pragma unroll
                for (int a = 0; a < TNB; ++a)
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        float bv[4];
                        bias4(a, g, bv);
#pragma unroll
                        for (int b = 0; b < TMB; ++b)
                            *(float4*)(Fs + (wm0 - ps * SR + b * 32 + l32) * LDF + wn0 + a * 32 + 8 * g + 4 * lh) =
                                make_float4(acc[a][b][4 * g] + bv[0], acc[a][b][4 * g + 1] + bv[1], acc[a][b][4 * g + 2] + bv[2], acc[a][b][4 * g + 3] + bv[3]);
                    }
            }
            __syncthreads();
            if (finisher)
#pragma unroll
            for (int i = ps * (NCH / PASSES); i < (ps + 1) * (NCH / PASSES); ++i) {
                const int id = tid + i * NT;
                const int row = id / CPR, c8 = id - row * CPR;
                const int m = m0 + row, n = n0 + c8 * 8;
                if (m >= p.M || n >= p.Cout) continue;
                float2 row_s;
                if (LN == LN_RES) row_s = *(const float2*)((const char*)smem_all + ROWS_LDS + row * 8);
                if (LN == LN_RES && !SAME_C) load_gb(c8);
                float o[8];
                half8 v;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const float4 f = *(const float4*)(Fs + (row - ps * SR) * LDF + c8 * 8 + h * 4);
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        float r = (float)rv[i][4 * h + j];
                        if (LN == LN_RES) r = __builtin_fmaf(__builtin_fmaf(r, row_s.x, row_s.y), (&gq[h].x)[j], (&bq[h].x)[j]);
                        v[4 * h + j] = (half_t)((&f.x)[j] + r);
                        o[4 * h + j] = (float)v[4 * h + j];
                    }
                }
                *(half8*)((half_t*)p.y + (long long)m * p.ldy + n) = v;
                // Cout is a multiple of 64: the eight lanes that hold 64 channels of a row are all here
                const float s = sum_of_8_lanes(((o[0] + o[1]) + (o[2] + o[3])) + ((o[4] + o[5]) + (o[6] + o[7])));
                const float mean = s * (1.f / 64.f);
                float q = 0.f;
#pragma unroll
                for (int j = 0; j < 8; ++j) { const float d = o[j] - mean; q += d * d; }
                q = sum_of_8_lanes(q);
                if ((c8 & 7) == 0) p.stats_out[(long long)m * (p.Cout >> 6) + (n >> 6)] = make_float2(s, q);
            }
            if (ps + 1 < PASSES) __syncthreads();
        }
        return;
    }
    if (finisher)
#pragma unroll
    for (int a = 0; a < TNB; ++a)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int cn = wn0 + a * 32 + 8 * g + 4 * lh;
            float bv[4];
            bias4(a, g, bv);
            float4 c1;                                 // LN_IN: column sums of the weights
            if (LN == LN_IN) c1 = *(const float4*)(bias_s + 256 + cn);
#pragma unroll
            for (int b = 0; b < TMB; ++b) {
                half4* const at = (half4*)(Cs + (wm0 + b * 32 + l32) * LDC + cn);
                half4 h, r;
                if (RES == RES_WIDE) r = *at;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    float v = LN == LN_IN ? __builtin_fmaf(acc[a][b][4 * g + j], rows[b].x, __builtin_fmaf(rows[b].y, (&c1.x)[j], bv[j])) : acc[a][b][4 * g + j] + bv[j];
                    if (RES == RES_WIDE) v += (float)r[j];
                    if (GELU) v = gelu_f(v);
                    h[j] = (half_t)v;
                }
                // (behind a folded LayerNorm: GELU or nothing, and no residual.  With GELU the clamp would be one of 20 instructions per element, which an epilogue of 256 x 256
                // has 256 of on each SIMD, 9 us with idle matrix cores: ViT 64 images 3678 -> 3629 us, encoder 2 x 64 5154 -> 5111, eight sequences 704 -> 698)
                *at = LN == LN_IN ? h : __builtin_elementwise_min(__builtin_elementwise_max(h, lo4), hi4);
            }
        }
    __syncthreads();
    if (!finisher) return;
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
        const int id = tid + i * NT;
        const int row = id / CPR, c8 = id - row * CPR;
        const int m = m0 + row, n = n0 + c8 * 8;
        if (m < p.M && n < p.Cout) {
            half8 v = *(const half8*)(Cs + row * LDC + c8 * 8);
            if (LN != LN_IN && !fuse_act) {
                const half8 r = RES == RES_EARLY ? rv[i] : residual_chunk(i);
                v = __builtin_elementwise_min(__builtin_elementwise_max(v + r, lo8), hi8);
            }
            if (LN == LN_IN && p.y_sliced) *(half8*)((half_t*)p.y + ((long long)(n >> 6) * p.M + m) * 64 + (n & 63)) = v;
            else *(half8*)((half_t*)p.y + (long long)m * p.ldy + n) = v;
        }
    }
}

// One launch of a kernel that takes ConvParams and `lds` bytes of dynamic LDS, of which `reserve`, the same in every call for a kernel, are asked for before
// its first.  (The kernel is a template argument, so that each has a flag of its own: variants of a tile all have the same type.)
template <void (*KERNEL)(ConvParams)>
static int launch_with_lds(const ConvParams& p, dim3 grid, dim3 block, unsigned lds, unsigned reserve, hipStream_t stream) {
    static std::atomic<bool> configured{false};            // (setting the attribute twice is harmless)
    if (!configured.load(std::memory_order_acquire) && reserve > 48 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(KERNEL), hipFuncAttributeMaxDynamicSharedMemorySize, (int)reserve);
        if (e != hipSuccess) { set_error("conv: cannot reserve %u bytes of LDS: %s", reserve, hipGetErrorString(e)); return -2; }
    }
    configured.store(true, std::memory_order_release);
    hipLaunchKernelGGL(KERNEL, grid, block, lds, stream, p);
    return 0;
}

// The tiles a layer is given to one of (conv_igemm.hip: choose_conv).
enum TileId { T256x256, T256x192, T192x128, T128x256, T128x128, T128x128_2, T96x128, T64x128, T256x128s, T128x64_2, T128x64_3,
              T64x64, T64x64s, T32x64, T64x64_g2, T32x64_g4, T128x64, T_DMA, T_SK16 = T_DMA, T_SK32, T_PATCH256x128, T_PATCH128x128, T_PATCH256x64,
              T_REG128x128, T_REG128x64, T_REG64x64, T_ESTIMATED, T_SLABS64 = T_ESTIMATED, T_SLABS64s, T_SMALL32x16, T_SMALL64x16, T_SMALL64x32, T_SMALL128x32, T_MID96x128, T_MID192x128,
              T_COUNT };                               // (slabs: slab_split; small, mid: small_us, mid_us)

bool gemm_ln_two_fit(int id, const ConvParams& p);     // whether two workgroups of a folded product's tile fit a compute unit (gemm_ln.hip)

}  // namespace strait
