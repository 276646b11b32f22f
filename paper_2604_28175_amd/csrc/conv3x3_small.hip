// 3x3, stride 1, padding 1, of the small images and batches a server forms (paper Section 3.2 step (2)): few outputs, a long reduction.
//
// What bounds such a layer is the operand bytes that one compute unit can bring into LDS (60 to 100 B/ns) and the barriers of its chain, not MFMA.
// The gathered kernel fetches every input pixel nine times and meets at a barrier per 64 reduction elements; the patch kernel of the large layers
// (conv_igemm.hip) has tiles that leave most units idle here, and 64-byte rows, which travel at half the rate of whole 128-byte lines.  So
//   - a workgroup of four wavefronts owns BM bordered pixels x BN channels, BN as small as 16: the weights, BN rows of a stage, are most of its bytes;
//   - per slice of 64 input channels it holds the patch of input pixels that its nine taps touch, and all nine taps of its channels' weights: one
//     barrier per slice, between which a wavefront reads operands and multiplies without meeting the others.  NST slices are in flight;
//   - pixels are numbered as in the patch kernel (v = (n (H+1) + y) (W+1) + x, borders shared between neighbours), rows in LDS are 128 bytes, 16-byte
//     chunk c of row r at c ^ ((r >> 1) & 7): any 16 consecutive rows read at one logical chunk touch 16 distinct bank groups;
//   - the wavefronts share the 64 channels of a slice out (tiles of 16 channels: two by two, and the pixels), so that each reads an operand for several
//     MFMAs; what they read of the patch and the weights is what a slice takes where the transfers keep up.  Their sums meet in LDS in order.
// Measured on MI355X, dependent launches in a row, before -> after, us: one image 56 x 56, 64 channels 6.5 -> 4.7, 28 x 28, 128 7.2 -> 5.0, 14 x 14, 256
// 7.6 -> 5.5, 7 x 7, 512 11.1 -> 6.9; eight images 28 x 28 8.4 -> 6.9, 14 x 14 9.3 -> 7.5, 7 x 7 13.1 -> 9.2.  210 layers of 1 to 32 images: 0.82 of the
// time, the worst 1.08.  ResNet-50 one image 352 -> 329 us, eight 527 -> 509.  (A tile of 128 x 64 for 64 channels, its filter in LDS whole: 8.2 us on
// eight 56 x 56 images against 8.3 gathered; not kept.)
#include <algorithm>
#include <atomic>

#include "conv_dma.hpp"

namespace strait {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef unsigned uintx2 __attribute__((ext_vector_type(2)));
typedef unsigned uintx4 __attribute__((ext_vector_type(4)));

template <int BM, int BN, int NST, int NPW, int KSPLIT>
__global__ void __launch_bounds__(256) conv3x3_small_kernel(const ConvParams p) {
    constexpr int NW = 4, MF = BN == 16 ? 16 : 32;     // extent of an MFMA block
    constexpr int PXB = BM / MF;                       // blocks of pixels
    constexpr int GROUPS = NW / KSPLIT, TMB = PXB / GROUPS, TNB = BN / MF;   // groups of wavefronts share the pixels out
    constexpr int STEPS = 64 * MF / 512 / KSPLIT;      // MFMAs (of 512 / MF reduction elements) per tap and block
    constexpr int WROWS = 9 * BN, WI = (WROWS + 31) / 32;
    constexpr unsigned PATCH = NPW * NW * 1024, STAGE = PATCH + WI * NW * 1024;
    static_assert((BN == 16 || BN == 32) && BM % MF == 0 && PXB % GROUPS == 0 && STEPS >= 1 && NST >= 2, "unsupported tile");
    static_assert(NST * STAGE <= 160 * 1024, "LDS limit");
    typedef typename std::conditional<MF == 16, floatx4, floatx16>::type accx;

    extern __shared__ __attribute__((aligned(1024))) char sm[];
    const unsigned lds0 = (unsigned)(uintptr_t)sm;
    if (p.hp) __builtin_amdgcn_s_setprio(3);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kh = wave % KSPLIT, pb = wave / KSPLIT * TMB;
    const int lr = lane & (MF - 1), lk = lane / MF;    // row of a block, chunk of a step

    const int Wp = p.W + 1, NI = divide(p.M, p.by_pq);
    int m0, n0;
    {
        int tm, tn;
        place_tile(p.order, xcd_range(p.order.tiles, blockIdx.x), tm, tn);
        m0 = tm * BM;
        n0 = tn * BN;
    }
    const intx4 xrsrc = make_rsrc(p.x, (unsigned)(p.x_elems * 2));
    const intx4 wrsrc = make_rsrc(p.w, (unsigned)((long long)p.Cout * p.ldw * 2));

    // ---- per-lane source offsets: a transfer brings eight rows, a lane 16 bytes of row lane >> 3
    unsigned aoff[NPW];
#pragma unroll
    for (int j = 0; j < NPW; ++j) {
        const int s = (j * NW + wave) * 8 + (lane >> 3);
        int img, yp, xp;
        bordered_place(p, m0 + s, Wp, img, yp, xp);
        const int lc = (lane & 7) ^ ((s >> 1) & 7);
        aoff[j] = img < NI && yp >= 1 && xp >= 1 ? (unsigned)(((long long)img * p.sN + (long long)(yp - 1) * p.sH + (long long)(xp - 1) * p.sW + lc * 8) * 2) : OOB_OFFSET;
    }
    // weight rows in LDS are numbered tap * BN + channel; this wavefront's part of transfer j: tap, channel offset
    unsigned woff;
    {
        const int row = wave * 8 + (lane >> 3), ch = row % BN;
        woff = (unsigned)(((long long)(n0 + ch) * p.ldw + ((lane & 7) ^ ((row >> 1) & 7)) * 8) * 2);
    }
    // Tiles of 32 channels request the biases of their lane's outputs here, so that no round trip follows the reduction: eight images 28 x 28 6.70 -> 6.39 us,
    // 14 x 14 7.37 -> 6.98.  Tiles of 16 ask at the end: with four registers to fetch the same costs them more than it saves (7 x 7 8.50 -> 8.90).
    constexpr bool EARLY = MF == 32;
    constexpr int BQ = EARLY ? 4 : 1;
    auto bias_at = [&](int ch) __attribute__((always_inline)) { return p.bias ? *(const float4*)(p.bias + n0 + ch + 4 * lk) : make_float4(0.f, 0.f, 0.f, 0.f); };
    float4 bias[TNB][BQ];
    if constexpr (EARLY) {
#pragma unroll
        for (int a = 0; a < TNB; ++a)
#pragma unroll
            for (int q = 0; q < BQ; ++q) bias[a][q] = bias_at(a * MF + 8 * q);
    }
    const int ncs = p.C >> 6;
    auto issue = [&](int stage, int cs) __attribute__((always_inline)) {
        const bool live = cs < ncs;
        const unsigned base = lds0 + (unsigned)stage * STAGE, so = live ? (unsigned)cs * 128u : 0u;
        // (opaque per slice: keeps the nine taps' offsets from being hoisted out of the loop, where they would not fit in the scalar registers)
        unsigned step = live ? (BN == 16 ? 4u : 2u) * (unsigned)p.C : 0u;
        asm volatile("" : "+s"(step));
        unsigned at = so + (BN == 16 && (wave >> 1) ? step / 2 : 0u);
#pragma unroll
        for (int j = 0; j < WI; ++j, at += step) {
            const bool ok = live && (BN != 16 || 2 * j + (wave >> 1) < 9);
            dma16(wrsrc, ok ? woff : OOB_OFFSET, ok ? at : 0u, base + PATCH + (unsigned)(j * NW + wave) * 1024u);
        }
#pragma unroll
        for (int j = 0; j < NPW; ++j) dma16(xrsrc, live ? aoff[j] : OOB_OFFSET, so, base + (unsigned)(j * NW + wave) * 1024u);
    };
    constexpr int NT = WI + NPW;
#pragma unroll
    for (int i = 0; i < NST; ++i) issue(i, i);

    accx acc[TNB][TMB];
#pragma unroll
    for (int a = 0; a < TNB; ++a)
#pragma unroll
        for (int b = 0; b < TMB; ++b) acc[a][b] = accx(0.f);

    unsigned wbase[STEPS];                             // this lane's chunk of weight row lr, step by step
#pragma unroll
    for (int k = 0; k < STEPS; ++k) wbase[k] = PATCH + (unsigned)lr * 128u + (unsigned)((((kh * STEPS + k) * (64 / MF) + lk) ^ ((lr >> 1) & 7)) << 4);
    int st = 0;
    for (int cs = 0; cs < ncs; ++cs) {
        if (cs == 0) wait_loads_then_barrier<(NST - 1) * NT>();
        else {
            wait_loads_then_barrier<(NST - 2) * NT>();
            issue(st == 0 ? NST - 1 : st - 1, cs - 1 + NST);   // into the stage that everyone has left
        }
        const char* S = sm + (unsigned)st * STAGE;
#pragma unroll
        for (int t = 0; t < 9; ++t) {
            const int tapoff = (t / 3) * Wp + (t % 3);
            half8 wf[STEPS][TNB], xf[STEPS][TMB];
#pragma unroll
            for (int b = 0; b < TMB; ++b) {
                const unsigned slot = (unsigned)((pb + b) * MF + lr + tapoff);
                const unsigned a0 = slot * 128u, sw = (slot >> 1) & 7u;
#pragma unroll
                for (int k = 0; k < STEPS; ++k)
                    xf[k][b] = *(const half8*)(S + (a0 + ((((unsigned)((kh * STEPS + k) * (64 / MF) + lk)) ^ sw) << 4)));
            }
#pragma unroll
            for (int a = 0; a < TNB; ++a)
#pragma unroll
                for (int k = 0; k < STEPS; ++k) wf[k][a] = *(const half8*)(S + wbase[k] + (t * BN + a * MF) * 128);
#pragma unroll
            for (int k = 0; k < STEPS; ++k)
#pragma unroll
                for (int a = 0; a < TNB; ++a)
#pragma unroll
                    for (int b = 0; b < TMB; ++b) {
                        if constexpr (MF == 16) acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(wf[k][a], xf[k][b], acc[a][b], 0, 0, 0);
                        else acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(wf[k][a], xf[k][b], acc[a][b], 0, 0, 0);
                    }
        }
        st = st + 1 == NST ? 0 : st + 1;
    }
    wait_loads_then_barrier<0>();                      // trailing (empty) transfers have landed; LDS is free

    // ---- the wavefronts' sums meet: block b of a group is finished by its wavefront b mod KSPLIT, which adds them in the order of the channels
    constexpr int AV = MF == 16 ? 4 : 16;
    // (with KSPLIT == 1 there is nothing to add)
    float* xch = (float*)sm;                           // [GROUPS][TMB][TNB][KSPLIT - 1][AV][64]
    static_assert(GROUPS * TMB * TNB * (KSPLIT - 1) * AV * 256 <= NST * STAGE, "exchange");
    auto part = [&](int b, int a, int src) __attribute__((always_inline)) {
        return xch + (((pb + b) * TNB + a) * (KSPLIT - 1) + (src < b % KSPLIT ? src : src - 1)) * AV * 64 + lane;
    };
#pragma unroll
    for (int b = 0; b < TMB; ++b)
        if (kh != b % KSPLIT) {
#pragma unroll
            for (int a = 0; a < TNB; ++a)
#pragma unroll
                for (int v = 0; v < AV; ++v) part(b, a, kh)[v * 64] = acc[a][b][v];
        }
    if (KSPLIT > 1) __syncthreads();
    const half_t lo = (p.act == ACT_RELU || p.act == ACT_RELU6) ? (half_t)0.f : (half_t)-INFINITY;
    const half_t hi = p.act == ACT_RELU6 ? (half_t)6.f : (half_t)INFINITY;
    const half4 lo4 = {lo, lo, lo, lo}, hi4 = {hi, hi, hi, hi};
    auto finish = [&](float v0, float v1, float v2, float v3, float4 b4) __attribute__((always_inline)) {
        const half4 h = {(half_t)(v0 + b4.x), (half_t)(v1 + b4.y), (half_t)(v2 + b4.z), (half_t)(v3 + b4.w)};
        return __builtin_elementwise_min(__builtin_elementwise_max(h, lo4), hi4);
    };
#pragma unroll
    for (int b = 0; b < TMB; ++b) {
        if (kh != b % KSPLIT) continue;
#pragma unroll
        for (int a = 0; a < TNB; ++a)
#pragma unroll
            for (int v = 0; v < AV; ++v) {
                float t = b % KSPLIT == 0 ? acc[a][b][v] : part(b, a, 0)[v * 64];
#pragma unroll
                for (int h = 1; h < KSPLIT; ++h) t += h == b % KSPLIT ? acc[a][b][v] : part(b, a, h)[v * 64];
                acc[a][b][v] = t;
            }
        int img, yy, xx;
        bordered_place(p, m0 + (pb + b) * MF + lr, Wp, img, yy, xx);
        const bool ok = img < NI && yy < p.H && xx < p.W;
        half_t* row = (half_t*)p.y + ((long long)(img * p.H + yy) * p.W + xx) * p.ldy + n0;
#pragma unroll
        for (int a = 0; a < TNB; ++a) {
            if constexpr (MF == 16) {
                const half4 h = finish(acc[a][b][0], acc[a][b][1], acc[a][b][2], acc[a][b][3], bias_at(0));
                if (ok) *(half4*)(row + 4 * lk) = h;
            } else {
                // the lane holds channels 8 g + 4 lk .. + 3 of its pixel; after the exchange with lane ^ 32, eight channels of one g
#pragma unroll
                for (int g = 0; g < 4; g += 2) {
                    const half4 e = finish(acc[a][b][4 * g], acc[a][b][4 * g + 1], acc[a][b][4 * g + 2], acc[a][b][4 * g + 3], bias[a][g]);
                    const half4 f = finish(acc[a][b][4 * g + 4], acc[a][b][4 * g + 5], acc[a][b][4 * g + 6], acc[a][b][4 * g + 7], bias[a][g + 1]);
                    const uintx2 eu = __builtin_bit_cast(uintx2, e), fu = __builtin_bit_cast(uintx2, f);
                    const auto x = __builtin_amdgcn_permlane32_swap(eu[0], fu[0], false, false);
                    const auto y = __builtin_amdgcn_permlane32_swap(eu[1], fu[1], false, false);
                    if (ok) *(uintx4*)(row + a * 32 + 8 * (g + lk)) = uintx4{x[0], y[0], x[1], y[1]};
                }
            }
        }
    }
}

// slots of a tile's patch
static int small_slots(int bm, int W) { return bm + 2 * (W + 1) + 2; }

template <int BM, int BN, int NST, int NPW, int KSPLIT>
static int launch_small_tile(const ConvParams& params, hipStream_t stream) {
    ConvParams p = params;
    const long long mv = (long long)(p.M / p.PQ) * (p.H + 1) * (p.W + 1), tiles_m = (mv + BM - 1) / BM;
    const int tiles_n = p.Cout / BN;
    set_tile_order(p, tiles_m, tiles_n, small_slots(BM, p.W), 9 * BN, 64, 1);
    constexpr unsigned lds = NST * (NPW + (9 * BN + 31) / 32) * 4 * 1024;
    auto kernel = conv3x3_small_kernel<BM, BN, NST, NPW, KSPLIT>;
    static std::atomic<bool> configured{false};
    if (!configured.load(std::memory_order_acquire)) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) { set_error("conv: cannot reserve %u bytes of LDS: %s", lds, hipGetErrorString(e)); return -2; }
    }
    configured.store(true, std::memory_order_release);
    hipLaunchKernelGGL(kernel, dim3((unsigned)(tiles_m * tiles_n)), dim3(256), lds, stream, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) { set_error("conv launch: %s", hipGetErrorString(e)); return -2; }
    return 0;
}

bool conv3x3_small_takes(const ConvParams& p, int bm, int bn) {
    if (p.C % 64 != 0 || p.Cout % bn != 0 || p.W < 4 || p.W > 64) return false;
    const long long mv = (long long)(p.M / p.PQ) * (p.H + 1) * (p.W + 1);
    if (mv >= (1LL << 24) - 4096 || (mv + bm - 1) / bm * (p.Cout / bn) > 0x7fffffffLL) return false;
    const int npw = (small_slots(bm, p.W) + 31) / 32;
    if (bm == 32) return bn == 16 && npw <= 4;
    if (bm == 64) return npw <= 6;
    return bm == 128 && bn == 32 && npw <= 8;
}

int launch_conv3x3_small(const ConvParams& p, int bm, int bn, hipStream_t stream) {
    if (!conv3x3_small_takes(p, bm, bn)) { set_error("conv: not a layer of the small 3x3 kernel"); return -5; }
    const int npw = (small_slots(bm, p.W) + 31) / 32;
#define STRAIT_SMALL(BM, BN, NST, NPW, KSPLIT) return launch_small_tile<BM, BN, NST, NPW, KSPLIT>(p, stream)
    if (bm == 32 && bn == 16) { if (npw <= 2) STRAIT_SMALL(32, 16, 5, 2, 2); STRAIT_SMALL(32, 16, 4, 4, 2); }
    if (bm == 64 && bn == 16) { if (npw <= 3) STRAIT_SMALL(64, 16, 5, 3, 2); STRAIT_SMALL(64, 16, 3, 6, 2); }
    if (bm == 64 && bn == 32) { if (npw <= 3) STRAIT_SMALL(64, 32, 3, 3, 4); STRAIT_SMALL(64, 32, 2, 6, 2); }
    if (bm == 128 && bn == 32) { if (npw <= 6) STRAIT_SMALL(128, 32, 2, 6, 1); STRAIT_SMALL(128, 32, 2, 8, 1); }
#undef STRAIT_SMALL
    set_error("conv: no such tile");
    return -5;
}

}  // namespace strait
