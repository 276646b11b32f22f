// 3x3, stride 1, padding 1, of layers between the small images and batches (conv3x3_small.hip) and the large ones (conv_igemm.hip: the patch kernel), whose
// tiles make one round of the compute units (paper Section 3.2 step (2), for the batch sizes a server forms).
//
// What bounds such a layer on the gathered kernel is the operand bytes that one compute unit can bring into LDS (50 to 75 B/ns), of which the input's, every
// pixel fetched nine times, are half: 192 x 128 tiles of a 56 x 56 layer with 256 channels bring 40 KB per 64 reduction elements and need 20.  The large
// layers' patch kernel has too few tiles here, and 64-byte rows, which travel at half the rate of whole 128-byte lines.  So
//   - a workgroup of eight wavefronts owns BM bordered pixels (numbered as there, v = (n (H+1) + y) (W+1) + x) x 128 channels, and holds, per slice of 64
//     input channels, the patch of pixels that its nine taps touch, in 128-byte rows, swizzled as in conv3x3_small.hip; the next slice's patch arrives in a
//     second buffer meanwhile;
//   - the weights, 64 input channels of one tap at a time, stream through a ring of NBS stages; one barrier per tap, between which a wavefront
//     multiplies 96 pixels x 32 (BM = 96) or 64 channels with half of the 64 input channels, the halves' sums meeting in LDS in order, and reads the
//     next tap's operands (1 us of 28 against reading them behind the barrier).
// What is left is the weights' way into LDS on the tile of 96, 19 KB a tap in 0.29 us, and the MFMAs with that beside them on the tile of 192.  (Tiles of
// 96 with 64 channels and a quarter of the input channels per wavefront, which read LDS 1.6 times less: the same a tap, 1 us more at the end.)
// Measured on MI355X, dependent launches in a row, before -> after, us: three images 56 x 56, 256 channels 23.3 -> 18.1, six 31.0 -> 28.1; six 28 x 28, 512
// 35.9 -> 28.2, twelve 53.2 -> 47.8; 24 images 14 x 14, 512 37.5 -> 29.0.  VGG-19 with six images 601 -> 566 us a pass.
#include <algorithm>
#include <atomic>

#include "conv_dma.hpp"

namespace strait {

template <int BM, int WGM, int WGN, int KSPLIT, int NPW, int NBS>
__global__ void __launch_bounds__(512, 2) conv3x3_mid_kernel(const ConvParams p) {
    constexpr int NW = 8, NT = 512, BN = 128;
    constexpr int TM = BM / WGM, TMB = TM / 32, TNB = BN / WGN / 32, KSTEPS = 4 / KSPLIT, ACC = TNB * TMB * 16;
    static_assert(WGM * WGN * KSPLIT == NW && TM % 32 == 0, "unsupported tile");
    constexpr int WI = 2;                              // weight transfers per wave per tap: 128 rows, eight a transfer
    constexpr int AS = (NPW + 8 - NBS) / (9 - NBS);    // patch transfers per wave per tap (taps 0 .. 8 - NBS: before the next slice's first weights)
    constexpr int PATCH = NPW * NW * 1024, WSTAGE = BN * 128, RING = 2 * PATCH + NBS * WSTAGE;
    constexpr int LDC = BN + 8;
    constexpr unsigned BIAS_LDS = RING;
    static_assert(NBS >= 3 && NBS <= 8 && RING + 1024 <= 160 * 1024 && BM * LDC * 2 <= RING && KSPLIT / 2 * WGM * WGN * ACC * 256 <= RING, "LDS limit");

    extern __shared__ __attribute__((aligned(1024))) char sm[];
    const unsigned lds0 = (unsigned)(uintptr_t)sm;
    if (p.hp) __builtin_amdgcn_s_setprio(3);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, lh = lane >> 5;
    const int wn0 = wave % WGN * (TNB * 32), wm0 = wave / WGN % WGM * TM, kh = wave / (WGM * WGN);

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
    unsigned aoff[NPW], woff[WI];
#pragma unroll
    for (int j = 0; j < NPW; ++j) {
        const int s = (j * NW + wave) * 8 + (lane >> 3);
        int img, yp, xp;
        bordered_place(p, m0 + s, Wp, img, yp, xp);
        const int lc = (lane & 7) ^ ((s >> 1) & 7);
        aoff[j] = img < NI && yp >= 1 && xp >= 1 ? (unsigned)(((long long)img * p.sN + (long long)(yp - 1) * p.sH + (long long)(xp - 1) * p.sW + lc * 8) * 2) : OOB_OFFSET;
    }
#pragma unroll
    for (int j = 0; j < WI; ++j) {
        const int row = (j * NW + wave) * 8 + (lane >> 3);
        woff[j] = (unsigned)(((long long)(n0 + row) * p.ldw + ((lane & 7) ^ ((row >> 1) & 7)) * 8) * 2);
    }
    const int ncs = p.C >> 6;
    auto issue_w = [&](int stage, int tap, int cs) __attribute__((always_inline)) {
        const bool live = cs < ncs;
        const unsigned soff = live ? (unsigned)(tap * p.C + cs * 64) * 2u : 0u;
#pragma unroll
        for (int j = 0; j < WI; ++j)
            dma16(wrsrc, live ? woff[j] : OOB_OFFSET, soff, lds0 + (unsigned)(2 * PATCH + stage * WSTAGE + (j * NW + wave) * 1024));
    };
    auto issue_a = [&](int buf, int j, int cs) __attribute__((always_inline)) {
        const bool live = cs < ncs;
        dma16(xrsrc, live ? aoff[j] : OOB_OFFSET, live ? (unsigned)cs * 128u : 0u, lds0 + (unsigned)(buf * PATCH + (j * NW + wave) * 1024));
    };

    floatx16 acc[TNB][TMB];
#pragma unroll
    for (int a = 0; a < TNB; ++a)
#pragma unroll
        for (int b = 0; b < TMB; ++b) acc[a][b] = floatx16(0.f);
    if (wave == 0) {
        const intx4 brsrc = make_rsrc(p.bias, p.bias ? (unsigned)p.Cout * 4u : 0u);
        dma16(brsrc, p.bias && lane * 4 < BN ? (unsigned)(n0 + lane * 4) * 4u : OOB_OFFSET, 0u, lds0 + BIAS_LDS);
    }
#pragma unroll
    for (int j = 0; j < NPW; ++j) issue_a(0, j, 0);
#pragma unroll
    for (int t = 0; t < NBS; ++t) issue_w(t, t, 0);
    int cur = 0;                                       // ring stage of the tap that is multiplied, whose operands are in registers

    unsigned wbase[KSTEPS];                            // this lane's chunk of weight row wn0 + l32, step by step
#pragma unroll
    for (int k = 0; k < KSTEPS; ++k) wbase[k] = (unsigned)(wn0 + l32) * 128u + (unsigned)((((kh * KSTEPS + k) * 2 + lh) ^ ((l32 >> 1) & 7)) << 4);
    half8 wf[2][KSTEPS][TNB], xf[2][KSTEPS][TMB];           // operands of a tap and, on their way, of the next
    auto fetch = [&](auto setc, int stage, const char* Pa, int tapoff) __attribute__((always_inline)) {
        constexpr int SET = decltype(setc)::value;
        const char* Ws = sm + 2 * PATCH + stage * WSTAGE;
        unsigned a0[TMB], sw[TMB];
#pragma unroll
        for (int b = 0; b < TMB; ++b) {
            const unsigned slot = (unsigned)(wm0 + b * 32 + l32 + tapoff);
            a0[b] = slot * 128u;
            sw[b] = (slot >> 1) & 7u;
        }
#pragma unroll
        for (int k = 0; k < KSTEPS; ++k) {
#pragma unroll
            for (int a = 0; a < TNB; ++a) wf[SET][k][a] = *(const half8*)(Ws + wbase[k] + a * 32 * 128);
#pragma unroll
            for (int b = 0; b < TMB; ++b) xf[SET][k][b] = *(const half8*)(Pa + (a0[b] + ((((unsigned)((kh * KSTEPS + k) * 2 + lh)) ^ sw[b]) << 4)));
        }
    };
    // one tap: everyone has its operands in registers (so its weights' stage is free) and the next one's have landed
    auto tap_step = [&](auto tc, auto setc, int cs, int wp) __attribute__((always_inline)) {
        constexpr int T = decltype(tc)::value, SET = decltype(setc)::value;
        wait_loads_then_barrier<patch_wait(NPW, AS, WI, NBS - 1, T)>();
        const int next = cur + 1 == NBS ? 0 : cur + 1;
        fetch(std::integral_constant<int, 1 - SET>{}, next, sm + ((cs + (T + 1) / 9) & 1) * PATCH, ((T + 1) % 9 / 3) * wp + (T + 1) % 3);
        issue_w(cur, (T + NBS) % 9, cs + (T + NBS) / 9);
#pragma unroll
        for (int j = T * AS; j < (T + 1) * AS && j < NPW; ++j) issue_a((cs + 1) & 1, j, cs + 1);
        cur = next;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < KSTEPS; ++k)
#pragma unroll
            for (int a = 0; a < TNB; ++a)
#pragma unroll
                for (int b = 0; b < TMB; ++b) acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(wf[SET][k][a], xf[SET][k][b], acc[a][b], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto slice = [&](auto setc, int cs) __attribute__((always_inline)) {
        constexpr int S = decltype(setc)::value;
        int wp = Wp;                                   // opaque per slice: keeps the nine taps' operand addresses from being
        asm volatile("" : "+s"(wp));                   // hoisted out of the loop, where they would cost registers
#define STRAIT_TAP(T) tap_step(std::integral_constant<int, T>{}, std::integral_constant<int, (S + T) & 1>{}, cs, wp);
        STRAIT_TAP(0) STRAIT_TAP(1) STRAIT_TAP(2) STRAIT_TAP(3) STRAIT_TAP(4) STRAIT_TAP(5) STRAIT_TAP(6) STRAIT_TAP(7) STRAIT_TAP(8)
#undef STRAIT_TAP
    };
    wait_loads_then_barrier<(NBS - 1) * WI>();
    fetch(std::integral_constant<int, 0>{}, 0, sm, 0);
    int cs = 0;
    for (; cs + 1 < ncs; cs += 2) {                    // (an odd number of taps: the register sets change places from slice to slice)
        slice(std::integral_constant<int, 0>{}, cs);
        slice(std::integral_constant<int, 1>{}, cs + 1);
    }
    if (cs < ncs) slice(std::integral_constant<int, 0>{}, cs);
    wait_loads_then_barrier<0>();                      // trailing (empty) transfers have landed; LDS is free

    // the parts' sums are added to the first's, the upper half of them to the lower half at a time
#pragma unroll
    for (int half = KSPLIT / 2; half >= 1; half /= 2) {
        float* xch = (float*)sm + ((kh % half) * WGM * WGN + wave % (WGM * WGN)) * (ACC * 64) + lane;
        if (kh >= half && kh < 2 * half) {
#pragma unroll
            for (int a = 0; a < TNB; ++a)
#pragma unroll
                for (int b = 0; b < TMB; ++b)
#pragma unroll
                    for (int v = 0; v < 16; ++v) xch[((a * TMB + b) * 16 + v) * 64] = acc[a][b][v];
        }
        __syncthreads();
        if (kh < half) {
#pragma unroll
            for (int a = 0; a < TNB; ++a)
#pragma unroll
                for (int b = 0; b < TMB; ++b)
#pragma unroll
                    for (int v = 0; v < 16; ++v) acc[a][b][v] += xch[((a * TMB + b) * 16 + v) * 64];
        }
        __syncthreads();
    }

    // ---- bias, clamp, tile parked in LDS as [pixel][channel], 16-byte row segments out
    half_t* Cs = (half_t*)sm;
    const half_t lo = (p.act == ACT_RELU || p.act == ACT_RELU6) ? (half_t)0.f : (half_t)-INFINITY;
    const half_t hi = p.act == ACT_RELU6 ? (half_t)6.f : (half_t)INFINITY;
    const half4 lo4 = {lo, lo, lo, lo}, hi4 = {hi, hi, hi, hi};
    const float* bias_s = (const float*)(sm + BIAS_LDS);
    if (kh == 0) {
#pragma unroll
        for (int ag = 0; ag < 4 * TNB; ++ag) {
            const int a = ag >> 2, g = ag & 3, cn = wn0 + a * 32 + 8 * g + 4 * lh;
            const float4 b4 = *(const float4*)(bias_s + cn);
            const float bv[4] = {b4.x, b4.y, b4.z, b4.w};
#pragma unroll
            for (int b = 0; b < TMB; ++b) {
                half4 h;
#pragma unroll
                for (int j = 0; j < 4; ++j) h[j] = (half_t)(acc[a][b][4 * g + j] + bv[j]);
                *(half4*)(Cs + (wm0 + b * 32 + l32) * LDC + cn) = __builtin_elementwise_min(__builtin_elementwise_max(h, lo4), hi4);
            }
        }
    }
    __syncthreads();
    constexpr int CPR = BN / 8, NCH = BM * CPR / NT;
    static_assert(BM * CPR % NT == 0, "whole rows");
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
        const int id = tid + i * NT, row = id / CPR, c8 = id - row * CPR;
        int img, yy, xx;
        bordered_place(p, m0 + row, Wp, img, yy, xx);
        if (img < NI && yy < p.H && xx < p.W)
            *(half8*)((half_t*)p.y + ((long long)(img * p.H + yy) * p.W + xx) * p.ldy + n0 + c8 * 8) = *(const half8*)(Cs + row * LDC + c8 * 8);
    }
}

// slots of a tile's patch, in transfers of 64 per round of the wavefronts
static int mid_transfers(int bm, int W) { return (bm + 2 * (W + 1) + 2 + 63) / 64; }

template <int BM, int WGM, int WGN, int KSPLIT, int NPW, int NBS>
static int launch_mid_tile(const ConvParams& params, hipStream_t stream) {
    ConvParams p = params;
    const long long mv = (long long)(p.M / p.PQ) * (p.H + 1) * (p.W + 1), tiles_m = (mv + BM - 1) / BM;
    const int tiles_n = p.Cout / 128;
    set_tile_order(p, tiles_m, tiles_n, BM + 2 * (p.W + 1) + 2, 9 * 128, 64, 1);
    constexpr unsigned lds = 2 * NPW * 8 * 1024 + NBS * 128 * 128 + 1024;
    auto kernel = conv3x3_mid_kernel<BM, WGM, WGN, KSPLIT, NPW, NBS>;
    static std::atomic<bool> configured{false};
    if (!configured.load(std::memory_order_acquire)) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) { set_error("conv: cannot reserve %u bytes of LDS: %s", lds, hipGetErrorString(e)); return -2; }
    }
    configured.store(true, std::memory_order_release);
    hipLaunchKernelGGL(kernel, dim3((unsigned)(tiles_m * tiles_n)), dim3(512), lds, stream, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) { set_error("conv launch: %s", hipGetErrorString(e)); return -2; }
    return 0;
}

bool conv3x3_mid_takes(const ConvParams& p, int bm) {
    if (p.C % 64 != 0 || p.Cout % 128 != 0 || p.W < 4 || p.W > 64 || (bm != 96 && bm != 192)) return false;
    const long long mv = (long long)(p.M / p.PQ) * (p.H + 1) * (p.W + 1);
    return mv < (1LL << 24) - 4096 && (mv + bm - 1) / bm * (p.Cout / 128) <= 0x7fffffffLL && mid_transfers(bm, p.W) <= (bm == 96 ? 4 : 6);
}

int launch_conv3x3_mid(const ConvParams& p, int bm, hipStream_t stream) {
    if (!conv3x3_mid_takes(p, bm)) { set_error("conv: not a layer of the mid-size 3x3 kernel"); return -5; }
    const int npw = mid_transfers(bm, p.W);
    if (bm == 96) return npw <= 3 ? launch_mid_tile<96, 1, 4, 2, 3, 6>(p, stream) : launch_mid_tile<96, 1, 4, 2, 4, 5>(p, stream);
    if (npw <= 4) return launch_mid_tile<192, 2, 2, 2, 4, 5>(p, stream);
    return npw <= 5 ? launch_mid_tile<192, 2, 2, 2, 5, 4>(p, stream) : launch_mid_tile<192, 2, 2, 2, 6, 3>(p, stream);
}

}  // namespace strait
