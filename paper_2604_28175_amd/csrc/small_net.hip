// A whole small classifier in one launch (paper Section 3.2, all of step (2) and step (3)): three 3x3 convolutions with ReLU, of stride 1, 2 and 2 and 16, 32 and
// 64 channels, global average pooling, the fully connected layer, softmax, top-1 and the result's way to the host.
//
// Layer by layer such a network is nothing but launches: four dependent ones of 4 to 7 us, behind the input's copy, for 6 MFLOP an image.  Here a workgroup of eight wavefronts takes an
// image from the input to the host's buffer, all activations in LDS (77 KB at 32 x 32) with a border of zeros, so that no tap asks
// whether it is inside:
//   - a wavefront's weights, all three layers', are fragments of v_mfma_f32_16x16x32_f16 in registers (17 of them), requested before anything else;
//   - the image has its channels padded to eight in LDS: a filter row is four pixels of 16 bytes, one MFMA, whose fourth tap reads zeros (and not the
//     neighbouring pixel, whose infinities times a weight of zero would not be zero);
//   - 16 channels: an MFMA takes two taps, the tenth reads zeros; 32 channels: one tap;
//   - the last layer's activations are rounded to fp16 as everywhere, added up in the registers and never stored.
// Rounding points are those of the launches.  MI355X, from submission to result in us, those four launches / this: four 32 x 32 images 30.2 / 21.1, 32 images 35.0 / 25.9, 256 images
// 79.7 / 54.8.
// What is left: 12.7 us a launch in a trace, 3.5 of them until the weights and the image are there, 4 of LDS reads and chains of MFMAs, half of it at LDS's rate; the others are the launch
// itself, the head and the result's way to the host.
#include <algorithm>
#include <atomic>
#include <type_traits>

#include "classify_out.hpp"
#include "small_net.hpp"

namespace strait {

typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int SN_WAVES = 8, SN_C1 = 16, SN_C2 = 32, SN_C3 = 64;

struct SmallNetLds { int image, first, second, end; };     // halfs: where each activation ends
__host__ __device__ static inline SmallNetLds small_net_lds(int H, int W) {
    SmallNetLds l;
    l.image = (H + 2) * (W + 3) * 8;
    l.first = l.image + (H + 2) * (W + 2) * SN_C1;
    l.second = l.first + ((H + 1) / 2 + 2) * ((W + 1) / 2 + 2) * SN_C2;
    l.end = l.second;
    return l;
}

__device__ __forceinline__ float sum_of_16_lanes(float v) {    // of the aligned sixteen lanes that this one belongs to
    auto moved = [](float x, auto ctl) { return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), decltype(ctl)::value, 0xf, 0xf, true)); };
    v += moved(v, std::integral_constant<int, 0xB1>{});        // lane ^ 1
    v += moved(v, std::integral_constant<int, 0x4E>{});        // lane ^ 2
    v += moved(v, std::integral_constant<int, 0x141>{});       // the other four of eight
    v += moved(v, std::integral_constant<int, 0x140>{});       // the other eight
    return v;
}

template <bool V4>
__global__ void __launch_bounds__(64 * SN_WAVES, 2) small_net_kernel(const SmallNet p) {
    extern __shared__ __attribute__((aligned(16))) half_t sn_smem[];
    __shared__ float pooled[2][SN_C3];
    __shared__ __attribute__((aligned(16))) half_t feat[SN_C3];
    __shared__ float lg[256];
    __shared__ ClassifyReduce<SN_WAVES> red;
    if (p.out.hp) __builtin_amdgcn_s_setprio(3);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l16 = lane & 15, g = lane >> 4, row = blockIdx.x;
    const SmallNetLds at = small_net_lds(p.H, p.W);
    half_t *const xs = sn_smem, *const a1 = sn_smem + at.image, *const a2 = sn_smem + at.first;
    const int XP = p.W + 3, AP = p.W + 2, BP = p.Q1 + 2;    // pixels in a row of each

    // ---- the image's pixels are requested first, up to four a thread before any is waited for; then the weights
    // (what lies outside the image, or past its channels, has an offset beyond the buffer and reads as zero)
    const auto img = __builtin_amdgcn_make_buffer_rsrc((void*)(p.x + (size_t)row * p.H * p.W * p.C), 0, p.H * p.W * p.C * 2, 0x00020000);
    constexpr int AHEAD = 4;
    const int npix = (p.H + 2) * XP;
    unsigned short pix[AHEAD][4];
    auto request = [&](int i0) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < AHEAD; ++k) {
            const int i = i0 + k * 64 * SN_WAVES, yp = divide(i, p.by_xp), y = yp - 1, x = i - yp * XP - 1;
            const bool in = (unsigned)y < (unsigned)p.H && (unsigned)x < (unsigned)p.W;
            const unsigned at = in ? (unsigned)((y * p.W + x) * p.C) * 2u : 0x80000000u;
#pragma unroll
            for (int c = 0; c < 4; ++c) pix[k][c] = __builtin_amdgcn_raw_buffer_load_b16(img, c < p.C ? at + 2u * c : 0x80000000u, 0, 0);
        }
    };
    request(tid);
    // lane (l16, g) holds channel l16 of its group, reduction elements 8 g .. of 32
    const int cb1 = wave & 1, cb2 = wave & 3;
    half8 w0[3], w1[5], w2[9];
#pragma unroll
    for (int t = 0; t < 3; ++t) w0[t] = *(const half8*)(p.w0 + l16 * 96 + t * 32 + g * 8);
#pragma unroll
    for (int t = 0; t < 5; ++t) w1[t] = t == 4 && g >= 2 ? half8(0) : *(const half8*)(p.w1 + (cb1 * 16 + l16) * (9 * SN_C1) + t * 32 + g * 8);
#pragma unroll
    for (int t = 0; t < 9; ++t) w2[t] = *(const half8*)(p.w2 + (cb2 * 16 + l16) * (9 * SN_C2) + t * 32 + g * 8);
    const floatx4 b0 = *(const floatx4*)(p.b0 + 4 * g), b1 = *(const floatx4*)(p.b1 + cb1 * 16 + 4 * g), b2 = *(const floatx4*)(p.b2 + cb2 * 16 + 4 * g);
    const int sub = tid & 7, cls0 = tid >> 3;          // the head: a dot product is shared by 8 lanes, a chunk of 8 features each
    half8 wh = half8(0);
    if (cls0 < p.out.n) wh = *(const half8*)(p.out.w + (size_t)cls0 * p.out.ldw + sub * 8);
    for (int i = at.image / 8 + tid; i < at.end / 8; i += 64 * SN_WAVES) *(half8*)(sn_smem + i * 8) = half8(0);
    for (int i0 = tid; i0 < npix;) {
#pragma unroll
        for (int k = 0; k < AHEAD; ++k) {
            const int i = i0 + k * 64 * SN_WAVES;
            if (i < npix) *(uintx4*)(xs + i * 8) = uintx4{pix[k][0] | (unsigned)pix[k][1] << 16, pix[k][2] | (unsigned)pix[k][3] << 16, 0u, 0u};
        }
        i0 += AHEAD * 64 * SN_WAVES;
        if (i0 < npix) request(i0);
    }
    __syncthreads();

    const half4 zero4 = {(half_t)0.f, (half_t)0.f, (half_t)0.f, (half_t)0.f};
    auto relu = [&](floatx4 acc, floatx4 b) __attribute__((always_inline)) {
        const half4 h = {(half_t)(acc[0] + b[0]), (half_t)(acc[1] + b[1]), (half_t)(acc[2] + b[2]), (half_t)(acc[3] + b[3])};
        return __builtin_elementwise_max(h, zero4);
    };
    // Every wavefront works on several blocks of 16 pixels at a time: a block by itself is a chain of reads and MFMAs that wait for each other.
    // ---- 3 x 3, stride 1: a filter row an MFMA; the first pixel of each array is a border one, for lanes that are to read zeros
    {
        constexpr int NB = 4;
        const int n = p.H * p.W;
        for (int b = wave * (16 * NB); b < n; b += SN_WAVES * 16 * NB) {
            half8 xf[NB][3];
            int to[NB];
#pragma unroll
            for (int k = 0; k < NB; ++k) {
                const int px = b + k * 16 + l16, pc = px < n ? px : 0, y = divide(pc, p.by_w), x = pc - y * p.W;
                const half_t* src = xs + (g == 3 ? 0 : (y * XP + x + g) * 8);
                const int step = g == 3 ? 0 : XP * 8;
#pragma unroll
                for (int t = 0; t < 3; ++t) xf[k][t] = *(const half8*)(src + t * step);
                to[k] = px < n ? ((y + 1) * AP + x + 1) * SN_C1 + 4 * g : -1;
            }
            floatx4 acc[NB];
#pragma unroll
            for (int k = 0; k < NB; ++k) acc[k] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int t = 0; t < 3; ++t)
#pragma unroll
                for (int k = 0; k < NB; ++k) acc[k] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w0[t], xf[k][t], acc[k], 0, 0, 0);
#pragma unroll
            for (int k = 0; k < NB; ++k) if (to[k] >= 0) *(half4*)(a1 + to[k]) = relu(acc[k], b0);
        }
    }
    __syncthreads();
    // ---- 3 x 3, stride 2, from 16 channels: two taps an MFMA
    {
        constexpr int NB = 4;
        const int n = p.P1 * p.Q1;
        int off[5];
#pragma unroll
        for (int t = 0; t < 5; ++t) {
            const int lo = (2 * t / 3 * AP + 2 * t % 3) * SN_C1, hi = ((2 * t + 1) / 3 * AP + (2 * t + 1) % 3) * SN_C1;
            off[t] = (g >= 2 ? hi : lo) + (g & 1) * 8;
        }
        for (int b = (wave >> 1) * (16 * NB); b < n; b += SN_WAVES / 2 * 16 * NB) {
            half8 xf[NB][5];
            int to[NB];
#pragma unroll
            for (int k = 0; k < NB; ++k) {
                const int px = b + k * 16 + l16, pc = px < n ? px : 0, y = divide(pc, p.by_q1), x = pc - y * p.Q1;
                const half_t* src = a1 + (2 * y * AP + 2 * x) * SN_C1;
#pragma unroll
                for (int t = 0; t < 5; ++t) xf[k][t] = *(const half8*)(t == 4 && g >= 2 ? a1 : src + off[t]);
                to[k] = px < n ? ((y + 1) * BP + x + 1) * SN_C2 + cb1 * 16 + 4 * g : -1;
            }
            floatx4 acc[NB];
#pragma unroll
            for (int k = 0; k < NB; ++k) acc[k] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int t = 0; t < 5; ++t)
#pragma unroll
                for (int k = 0; k < NB; ++k) acc[k] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w1[t], xf[k][t], acc[k], 0, 0, 0);
#pragma unroll
            for (int k = 0; k < NB; ++k) if (to[k] >= 0) *(half4*)(a2 + to[k]) = relu(acc[k], b1);
        }
    }
    __syncthreads();
    // ---- 3 x 3, stride 2, from 32 channels, and the sum over the positions
    {
        constexpr int NB = 2;
        const int n = p.P2 * p.Q2;
        float s[4] = {0.f, 0.f, 0.f, 0.f};
        for (int b = (wave >> 2) * (16 * NB); b < n; b += SN_WAVES / 4 * 16 * NB) {
            half8 xf[NB][9];
#pragma unroll
            for (int k = 0; k < NB; ++k) {
                const int px = b + k * 16 + l16, pc = px < n ? px : 0, y = divide(pc, p.by_q2), x = pc - y * p.Q2;
                const half_t* src = a2 + (2 * y * BP + 2 * x) * SN_C2 + g * 8;
#pragma unroll
                for (int t = 0; t < 9; ++t) xf[k][t] = *(const half8*)(src + (t / 3 * BP + t % 3) * SN_C2);
            }
            // (two sums a block, of the first five taps and of the rest: half the chain)
            floatx4 acc[NB][2];
#pragma unroll
            for (int k = 0; k < NB; ++k) acc[k][0] = acc[k][1] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int t = 0; t < 5; ++t)
#pragma unroll
                for (int k = 0; k < NB; ++k) {
                    acc[k][0] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w2[t], xf[k][t], acc[k][0], 0, 0, 0);
                    if (t < 4) acc[k][1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w2[5 + t], xf[k][5 + t], acc[k][1], 0, 0, 0);
                }
#pragma unroll
            for (int k = 0; k < NB; ++k) {
                const half4 h = relu(acc[k][0] + acc[k][1], b2);
#pragma unroll
                for (int j = 0; j < 4; ++j) s[j] += b + k * 16 + l16 < n ? (float)h[j] : 0.f;
            }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) s[j] = sum_of_16_lanes(s[j]);
        if (l16 == 0) {
#pragma unroll
            for (int j = 0; j < 4; ++j) pooled[wave >> 2][cb2 * 16 + 4 * g + j] = s[j];
        }
    }
    __syncthreads();
    if (tid < SN_C3) feat[tid] = (half_t)((pooled[0][tid] + pooled[1][tid]) * (1.f / (float)(p.P2 * p.Q2)));
    __syncthreads();
    for (int cls = cls0; cls < p.out.n; cls += 8 * SN_WAVES) {
        if (cls != cls0) wh = *(const half8*)(p.out.w + (size_t)cls * p.out.ldw + sub * 8);
        const half8 f = *(const half8*)(feat + sub * 8);
        float s = 0.f;
#pragma unroll
        for (int j = 0; j < 8; ++j) s += (float)wh[j] * (float)f[j];
        s += __shfl_xor(s, 1, 8);
        s += __shfl_xor(s, 2, 8);
        s += __shfl_xor(s, 4, 8);
        if (sub == 0) lg[cls] = s + (p.out.bias ? p.out.bias[cls] : 0.f);
    }
    __syncthreads();
    float v[4];
    int cls[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) { cls[k] = V4 ? 4 * tid + k : tid + 64 * SN_WAVES * k; v[k] = cls[k] < p.out.n ? lg[cls[k]] : -INFINITY; }
    classify_end<SN_WAVES, V4, true>(p.out, row, v, cls, red);
}

// One workgroup a compute unit at a time (registers): 256 rows take 8 to 11 us, each further 256 as much again, where launches of their own take 8 us more per 1000
// images of 8 x 8, 18 of 16 x 16 and 43 of 32 x 32.  Kernels in us, launches / this: 8 x 8, 300 rows 21.6 / 16.6, 600 23.0 / 24.7, 1000 25.8 / 34.0; 16 x 16, 600
// 28.7 / 26.1, 1000 36.3 / 35.9; 32 x 32, 8 rows 20.2 / 11.1, 300 37.5 / 22.2, 1000 61.8 / 45.7.
constexpr int SN_MAX_LDS = 150 * 1024;
bool small_net_takes(int H, int W, int C, long long rows, int classes) {
    if (H < 1 || W < 1 || H > 256 || W > 256 || C < 1 || C > 4) return false;
    if (rows > 512 && H * W < 256) return false;
    return small_net_lds(H, W).end * 2 <= SN_MAX_LDS && classify_out_takes(rows, classes) && classify_out_pools(((H + 1) / 2 + 1) / 2 * (((W + 1) / 2 + 1) / 2), SN_C3, classes);
}

int launch_small_net(const SmallNet& params, hipStream_t stream) {
    SmallNet p = params;
    if (!p.x || !p.w0 || !p.w1 || !p.w2 || !p.b0 || !p.b1 || !p.b2 || !p.out.w || p.out.ldw < SN_C3 || p.out.ldw % 8 != 0 || !p.out.logits || !p.out.probs || !p.out.top1 ||
        !p.out.host || !p.out.ctl || !p.out.counter || !small_net_takes(p.H, p.W, p.C, p.out.rows, p.out.n)) {
        set_error("small network: invalid shape"); return -5;
    }
    if ((reinterpret_cast<uintptr_t>(p.w0) | reinterpret_cast<uintptr_t>(p.w1) | reinterpret_cast<uintptr_t>(p.w2) | reinterpret_cast<uintptr_t>(p.out.w) |
         reinterpret_cast<uintptr_t>(p.b0) | reinterpret_cast<uintptr_t>(p.b1) | reinterpret_cast<uintptr_t>(p.b2) | reinterpret_cast<uintptr_t>(p.out.logits) |
         reinterpret_cast<uintptr_t>(p.out.host) | (p.out.n % 4 == 0 ? reinterpret_cast<uintptr_t>(p.out.probs) : 0)) & 15) {
        set_error("small network: 16-byte aligned buffers required"); return -1;
    }
    p.P1 = (p.H + 1) / 2; p.Q1 = (p.W + 1) / 2; p.P2 = (p.P1 + 1) / 2; p.Q2 = (p.Q1 + 1) / 2;
    p.by_xp = divisor(p.W + 3); p.by_w = divisor(p.W); p.by_q1 = divisor(p.Q1); p.by_q2 = divisor(p.Q2);
    const unsigned lds = (unsigned)small_net_lds(p.H, p.W).end * 2;
    const bool v4 = p.out.n % 4 == 0;
    const void* const kernel = v4 ? reinterpret_cast<const void*>(small_net_kernel<true>) : reinterpret_cast<const void*>(small_net_kernel<false>);
    static std::atomic<bool> configured[2];
    if (!configured[v4].load(std::memory_order_acquire)) {
        const hipError_t e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, SN_MAX_LDS);
        if (e != hipSuccess) { set_error("small network: cannot reserve LDS: %s", hipGetErrorString(e)); return -2; }
    }
    configured[v4].store(true, std::memory_order_release);
    if (v4) hipLaunchKernelGGL(small_net_kernel<true>, dim3((unsigned)p.out.rows), dim3(64 * SN_WAVES), lds, stream, p);
    else hipLaunchKernelGGL(small_net_kernel<false>, dim3((unsigned)p.out.rows), dim3(64 * SN_WAVES), lds, stream, p);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) { set_error("small network launch: %s", hipGetErrorString(e)); return -2; }
    return 0;
}

}  // namespace strait
