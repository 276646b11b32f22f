// Convolutions and products with few outputs and a reduction worth sharing out: the late layers of small batches, fully
// connected layers, short token sequences (paper Section 3.2 step (2), for the batch sizes a server forms).
//
// What bounds such a layer is neither MFMA nor HBM but the chain of round trips of a workgroup and the operand bytes one
// compute unit can pull (about 40 B/ns when every byte is used once).  So
//   - a workgroup of four wavefronts owns a tile of only 16 pixels x 16 or 32 channels, which gives a hundred workgroups and
//     more even to a 7 x 7 image, and its wavefronts share the reduction out in contiguous parts, whole 64-element
//     super-slices (128 bytes of an operand row): no second launch adds partial sums, they meet in LDS;
//   - operands go from memory to registers in MFMA layout, not through LDS: every operand byte is used by one wavefront only,
//     so staging would add a round trip and no reuse.  A quarter-wavefront reads 64 contiguous bytes of a row;
//   - two register sets of two super-slices each alternate: one feeds v_mfma_f32_16x16x32_f16 while the other is on its way.
//     (More slices in flight, or eight wavefronts, came out the same or slower: the unit's request queue is full.)
//   - taps outside the image, rows and channels past the end and the slices past a wavefront's part take an offset beyond the
//     buffer, which reads as zeros.
// The partial sums are added in wavefront order, so results do not depend on scheduling.
//
// Measured on MI355X, dependent launches in a row, before (slab-split reduction and a second launch, or two groups of
// wavefronts in one workgroup) -> after, us: 3x3 256 -> 256 at 14 x 14, one image 11.7 -> 7.5; 3x3 128 -> 128 at 28 x 28 9.9 -> 6.5;
// 1x1 1024 -> 256 at 14 x 14 6.0 -> 4.4; 1x1 2048 -> 512 at 7 x 7 9.0 -> 6.1; 2048 -> 1000 classifier, 8 images 8.3 -> 5.5;
// 25088 -> 4096 for 6 rows 44.6 -> 38.3 (5.4 TB/s of weights); 960 -> 160 at 7 x 7, 5 images 6.4 -> 4.4.
#include "activation.hpp"
#include "tiles.hpp"

namespace strait {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef unsigned uintx4 __attribute__((ext_vector_type(4)));

constexpr unsigned SK_OOB = 0x80000000u;               // beyond any buffer these kernels accept

template <int TN, bool GATHER, bool DUAL>
__global__ void __launch_bounds__(256) conv_skinny_kernel(const ConvParams p) {
    constexpr int TM = 16, NB = TN / 16, NW = 4, U = 2;
    static_assert(TN == 16 || TN == 32, "tile");
    static_assert(!(GATHER && DUAL), "a second source belongs to a plain pointwise convolution");
    __shared__ float4 part[NW][NB][64];                // partial sums: [wavefront][16 channels][lane]
    if (p.hp) __builtin_amdgcn_s_setprio(3);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, lg = lane >> 4;

    int m0, n0;
    {
        int tm, tn;
        place_tile(p.order, xcd_range(p.order.tiles, blockIdx.x), tm, tn);
        m0 = tm * TM;
        n0 = tn * TN;
    }

    // the buffer starts `lead` elements before x, so that the offset of a window's top-left tap is never negative
    const long long lead = (long long)p.pad_h * p.sH + (long long)p.pad_w * p.sW;
    const auto xr = __builtin_amdgcn_make_buffer_rsrc((void*)(p.x - lead), 0, (int)((p.x_elems + lead) * 2), 0x00020000);
    const auto wr = __builtin_amdgcn_make_buffer_rsrc((void*)p.w, 0, (int)((long long)p.Cout * p.ldw * 2), 0x00020000);
    const auto xr2 = __builtin_amdgcn_make_buffer_rsrc((void*)(DUAL ? p.x2 : p.x), 0, DUAL ? (int)(p.x2_elems * 2) : 0, 0x00020000);

    // ---- this lane's operand rows: pixel l16 of the tile and channel l16 of each group of 16, bytes 16 lg .. of 64
    unsigned xoff = SK_OOB, xoff2 = SK_OOB, taps = 0xffffffffu, woff[NB];
    const int m = m0 + l16;
    if (m < p.M) {
        if (!GATHER && p.stride_h == 1) xoff = (unsigned)(((long long)m * p.sW + lg * 8) * 2);
        if (GATHER || p.stride_h != 1 || DUAL) {
            const int n = divide(m, p.by_pq), rem = m - n * p.PQ, pp = divide(rem, p.by_q), qq = rem - pp * p.Q;
            if (GATHER || p.stride_h != 1)
                xoff = (unsigned)(((long long)n * p.sN + (long long)(pp * p.stride_h) * p.sH + (long long)(qq * p.stride_w) * p.sW + lg * 8) * 2);
            if (DUAL) xoff2 = (unsigned)(((long long)n * p.sN2 + (long long)(pp * p.stride2) * p.sH2 + (long long)(qq * p.stride2) * p.sW2 + lg * 8) * 2);
            if (GATHER) {
                const int ih0 = pp * p.stride_h - p.pad_h, iw0 = qq * p.stride_w - p.pad_w;
                taps = taps_inside(p, ih0, iw0);
            }
        }
    }
#pragma unroll
    for (int a = 0; a < NB; ++a) {
        const int n = n0 + a * 16 + l16;
        woff[a] = n < p.Cout ? (unsigned)(((long long)n * p.ldw + lg * 8) * 2) : SK_OOB;
    }

    // ---- what this thread needs for the four channels of one pixel that it will finish: requested now, so that no further
    // round trip follows the reduction (one image, 2048 -> 512 channels 6.28 -> 6.24 us, 512 -> 2048 with its residual 4.63 -> 4.48, 1024 -> 256 4.04 -> 3.99)
    constexpr int NQ = TN / 4;                         // channel quads of a pixel
    const int cq = tid % NQ, px = tid / NQ;
    const int mo = m0 + px, no = n0 + cq * 4;
    const bool finishes = tid < TM * NQ && mo < p.M && no < p.Cout, whole = no + 4 <= p.Cout && ((p.Cout | p.ldy) & 3) == 0;
    const long long at = (long long)mo * p.ldy + no;
    float4 bias = make_float4(0.f, 0.f, 0.f, 0.f);
    half4 res = {(half_t)0.f, (half_t)0.f, (half_t)0.f, (half_t)0.f};
    if (finishes && whole) {
        if (p.bias) bias = *(const float4*)(p.bias + no);
        if (p.res) res = *(const half4*)(p.res + at);
    }
    // ---- this wavefront's part of the reduction: super-slices sl .. s1 - 1
    const int ns = p.Kg >> 6;
    const int q = ns / NW, rq = ns - q * NW;
    const int s0 = wave * q + (wave < rq ? wave : rq), s1 = s0 + q + (wave < rq ? 1 : 0);
    int sl = s0, tap = 0, ts = 0, cb = s0 * 64;
    unsigned tap_off = 0;
    const unsigned row_step = (unsigned)(p.sH - p.S * p.sW) * 2u;   // from the end of a filter row to the next
    if (GATHER) {
        tap = divide(cb, p.by_c);
        cb -= tap * p.C;
        const int r0 = divide(tap, p.by_s);
        ts = tap - r0 * p.S;
        tap_off = (unsigned)(r0 * p.sH + ts * p.sW) * 2u;
    }
    uintx4 wf[2][U][NB][2], xf[2][U][2];
    auto request = [&](int set) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool live = sl < s1;
            const unsigned wk = live ? (unsigned)sl * 128u : 0u;
            const bool second = DUAL && sl * 64 >= p.C;
            const unsigned xk = !live ? 0u : GATHER ? tap_off + (unsigned)cb * 2u : second ? wk - (unsigned)p.C * 2u : wk;
#pragma unroll
            for (int a = 0; a < NB; ++a)
#pragma unroll
                for (int h = 0; h < 2; ++h) wf[set][u][a][h] = __builtin_amdgcn_raw_buffer_load_b128(wr, (live ? woff[a] : SK_OOB) + 64u * h, wk, 0);
            unsigned v = DUAL && second ? xoff2 : xoff;
            if (GATHER) v = ((taps >> tap) & 1u) ? v : SK_OOB;
            if (!live) v = SK_OOB;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                if (DUAL && second) xf[set][u][h] = __builtin_amdgcn_raw_buffer_load_b128(xr2, v + 64u * h, xk, 0);
                else xf[set][u][h] = __builtin_amdgcn_raw_buffer_load_b128(xr, v + 64u * h, xk, 0);
            }
            ++sl;
            if (GATHER) {
                cb += 64;
                if (cb >= p.C) {
                    cb = 0;
                    ++tap;
                    tap_off += (unsigned)p.sW * 2u;
                    if (++ts == p.S) { ts = 0; tap_off += row_step; }
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);             // keeps the requests ahead of the MFMAs that follow
    };
    floatx4 acc[NB];
#pragma unroll
    for (int a = 0; a < NB; ++a) acc[a] = floatx4{0.f, 0.f, 0.f, 0.f};
    auto consume = [&](int set) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int a = 0; a < NB; ++a)
                    acc[a] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8, wf[set][u][a][h]), __builtin_bit_cast(half8, xf[set][u][h]), acc[a], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    };
    request(0);
    for (int s = s0; s < s1; s += 2 * U) {
        request(1);
        consume(0);
        request(0);
        consume(1);
    }

    // ---- partial sums meet in LDS; a thread finishes four channels of one pixel: lane (l16, lg) held channels 4 lg .. of pixel l16
#pragma unroll
    for (int a = 0; a < NB; ++a) part[wave][a][lane] = make_float4(acc[a][0], acc[a][1], acc[a][2], acc[a][3]);
    __syncthreads();
    if (!finishes) return;
    float4 v = part[0][cq >> 2][(cq & 3) * 16 + px];
#pragma unroll
    for (int w = 1; w < NW; ++w) {
        const float4 t = part[w][cq >> 2][(cq & 3) * 16 + px];
        v.x += t.x; v.y += t.y; v.z += t.z; v.w += t.w;
    }
    float o[4] = {v.x, v.y, v.z, v.w};
    if (whole) {
        if (p.bias) { o[0] += bias.x; o[1] += bias.y; o[2] += bias.z; o[3] += bias.w; }
        if (p.res) {
#pragma unroll
            for (int j = 0; j < 4; ++j) o[j] += (float)res[j];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) o[j] = apply_act(o[j], p.act);
        if (p.out_f32) *(float4*)((float*)p.y + at) = make_float4(o[0], o[1], o[2], o[3]);
        else {
            half4 h;
#pragma unroll
            for (int j = 0; j < 4; ++j) h[j] = (half_t)o[j];
            *(half4*)((half_t*)p.y + at) = h;
        }
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (no + j >= p.Cout) break;
            float t = o[j] + (p.bias ? p.bias[no + j] : 0.f);
            if (p.res) t += (float)p.res[at + j];
            t = apply_act(t, p.act);
            if (p.out_f32) ((float*)p.y)[at + j] = t;
            else ((half_t*)p.y)[at + j] = (half_t)t;
        }
    }
}

int launch_conv_skinny(const ConvParams& params, int tn, bool gather, hipStream_t stream) {
    ConvParams p = params;
    if (p.C % 64 != 0 || p.Kg % 64 != 0 || (tn != 16 && tn != 32)) { set_error("conv: not a layer of the small-output kernel"); return -5; }
    const long long tiles_m = (p.M + 15) / 16;
    const int tiles_n = (p.Cout + tn - 1) / tn;
    if (tiles_m * tiles_n > 0x7fffffffLL) { set_error("conv: bad grid (%lld tiles)", tiles_m * tiles_n); return -5; }
    set_tile_order(p, tiles_m, tiles_n, 16, tn, 64, 1);
    const dim3 grid((unsigned)(tiles_m * tiles_n)), block(256);
#define STRAIT_SK(TN)                                                                                                    \
    do {                                                                                                                \
        if (p.x2) hipLaunchKernelGGL((conv_skinny_kernel<TN, false, true>), grid, block, 0, stream, p);                  \
        else if (gather) hipLaunchKernelGGL((conv_skinny_kernel<TN, true, false>), grid, block, 0, stream, p);           \
        else hipLaunchKernelGGL((conv_skinny_kernel<TN, false, false>), grid, block, 0, stream, p);                      \
    } while (0)
    if (tn == 16) STRAIT_SK(16); else STRAIT_SK(32);
#undef STRAIT_SK
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) { set_error("conv launch: %s", hipGetErrorString(e)); return -2; }
    return 0;
}

}  // namespace strait
