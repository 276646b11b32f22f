// The end of a classifier's batch in one launch: softmax and top-1 of the logits, and the whole result's way to pinned host memory (paper Section 3.2,
// the last of step (2) and step (3)); in small networks also the global average pooling and the fully connected layer before them.
//
// Nothing here is bound by memory or arithmetic: a launch whose input comes from the launch before it takes 4 to 6 us for a round trip to memory and the
// hand-over, whatever it computes.  So a workgroup takes one sample from its logits (or its feature map) to the host's buffer, a thread holding four
// classes in registers, and the last workgroup to finish sets the flag that the host polls.  Results of one chunk only: a larger one leaves in
// pieces beside the kernels that follow.  The device's copy of the result is written too, and is there before the flag.
// Measured on MI355X against launches of their own, timed in turn, us a pass: with pooling and product (four 32 x 32 images, ten classes) 46.1 -> 37.5; softmax
// and copy alone are worth no more than two runs of one side differ by, 1 to 4 %: ResNet-50 eight images 519 -> 510, one 324 -> 330, MobileNetV2 five 283 -> 285.
// The pooled head reads its weights once per sample through one compute unit, so it is for small ones: up to 16384 weights, 256 channels and 256
// classes (a hundred kilobytes would take longer than the two launches saved).
#include <algorithm>

#include "classify_out.hpp"

namespace strait {

// POOL: from the feature map; V4: classes a multiple of four, moved 16 bytes at a time.
template <bool POOL, bool V4>
__global__ void __launch_bounds__(256) classify_out_kernel(const ClassifyOut p) {
    __shared__ float part[POOL ? 256 * 9 : 1];         // partial sums of the pooling (pitch 9: no conflicts)
    __shared__ __attribute__((aligned(16))) half_t feat[POOL ? 256 : 8];
    __shared__ float lg[POOL ? 256 : 1];
    __shared__ ClassifyReduce<4> red;
    if (p.hp) __builtin_amdgcn_s_setprio(3);
    const int tid = threadIdx.x, row = blockIdx.x, n = p.n;
    const size_t base = (size_t)row * n;

    if constexpr (POOL) {
        const int C8 = p.C >> 3;
        // a dot product is shared by 8 lanes, each of every 8th chunk of 8 features: the first chunk is requested before the pooling
        const int sub = tid & 7, cls0 = tid >> 3;
        half8 w0 = half8(0);
        if (cls0 < n && sub < C8) w0 = *(const half8*)(p.w + (size_t)cls0 * p.ldw + sub * 8);
        int g2 = 1;                                    // threads beside each other take a pixel's chunks, groups of threads the pixels
        while (g2 < C8) g2 *= 2;
        const int g = tid & (g2 - 1), q = tid / g2, nq = 256 / g2;
        float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        if (g < C8) {
            const half_t* src = p.x + ((size_t)row * p.HW) * p.C + g * 8;
#pragma unroll 4
            for (int k = q; k < p.HW; k += nq) {
                const half8 v = *(const half8*)(src + (size_t)k * p.C);
#pragma unroll
                for (int j = 0; j < 8; ++j) acc[j] += (float)v[j];
            }
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) part[tid * 9 + j] = acc[j];
        __syncthreads();
        if (tid < p.C) {                               // one feature each, its parts added in order, rounded once to fp16
            float s = 0.f;
            for (int k = 0; k < nq; ++k) s += part[(k * g2 + (tid >> 3)) * 9 + (tid & 7)];
            feat[tid] = (half_t)(s * (1.f / (float)p.HW));
        }
        __syncthreads();
        for (int cls = cls0; cls < n; cls += 32) {
            float s = 0.f;
            for (int c = sub; c < C8; c += 8) {
                const half8 wv = cls == cls0 && c == sub ? w0 : *(const half8*)(p.w + (size_t)cls * p.ldw + c * 8);
                const half8 f = *(const half8*)(feat + c * 8);
#pragma unroll
                for (int j = 0; j < 8; ++j) s += (float)wv[j] * (float)f[j];
            }
            s += __shfl_xor(s, 1, 8);
            s += __shfl_xor(s, 2, 8);
            s += __shfl_xor(s, 4, 8);
            if (sub == 0) lg[cls] = s + (p.bias ? p.bias[cls] : 0.f);
        }
        __syncthreads();
    }

    // ---- this thread's classes: 4 tid + k, or tid + 256 k
    float v[4];
    int at[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) at[k] = V4 ? 4 * tid + k : tid + 256 * k;
    if constexpr (POOL) {
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = at[k] < n ? lg[at[k]] : -INFINITY;
    } else if constexpr (V4) {
        float4 t = make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
        if (at[0] < n) t = *(const float4*)(p.logits + base + at[0]);
        v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
    } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = at[k] < n ? p.logits[base + at[k]] : -INFINITY;
    }

    classify_end<4, V4, POOL>(p, row, v, at, red);
}

// (Up to 1024 rows, four workgroups on each of 256 compute units: beyond, a row's own writes to the host hold the next one up.  Kernels and copy in us, launches of
// their own / one.  Ten classes on 16 x 16 images with pooling and product: 600 rows 42.7 / 32.0, 1000 50.3 / 40.3, 2000 70.0 / 69.5, 2500 80.8 / 82.1; MobileNetV2,
// without: 300 rows 259.7 / 256.3, 700 324.3 / 323.7, 1000 357.4 / 357.4, 1500 406.1 / 412.7.)
bool classify_out_takes(long long rows, int n) { return rows > 0 && rows <= 1024 && n > 0 && n <= 1024 && (size_t)rows * (8 * (size_t)n + 4) <= out_chunk_bytes(1); }
bool classify_out_pools(int HW, int C, int n) { return HW > 0 && C > 0 && C % 8 == 0 && C <= 256 && n > 0 && n <= 256 && C * n <= 16384; }

int launch_classify_out(const ClassifyOut& p, hipStream_t stream) {
    if (!p.logits || !p.probs || !p.top1 || !p.host || !p.ctl || !p.counter || !classify_out_takes(p.rows, p.n) ||
        (p.x && (!p.w || !classify_out_pools(p.HW, p.C, p.n) || p.ldw < p.C || p.ldw % 8 != 0))) {
        set_error("classify out: invalid shape"); return -5;
    }
    if ((reinterpret_cast<uintptr_t>(p.logits) | reinterpret_cast<uintptr_t>(p.host) | reinterpret_cast<uintptr_t>(p.x) | reinterpret_cast<uintptr_t>(p.w) |
         (p.n % 4 == 0 ? reinterpret_cast<uintptr_t>(p.probs) : 0)) & 15) {
        set_error("classify out: 16-byte aligned buffers required"); return -1;
    }
    const dim3 grid((unsigned)p.rows), block(256);
    if (p.x) {
        if (p.n % 4 == 0) hipLaunchKernelGGL((classify_out_kernel<true, true>), grid, block, 0, stream, p);
        else hipLaunchKernelGGL((classify_out_kernel<true, false>), grid, block, 0, stream, p);
    } else if (p.n % 4 == 0) hipLaunchKernelGGL((classify_out_kernel<false, true>), grid, block, 0, stream, p);
    else hipLaunchKernelGGL((classify_out_kernel<false, false>), grid, block, 0, stream, p);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) { set_error("classify out launch: %s", hipGetErrorString(e)); return -2; }
    return 0;
}

}  // namespace strait
