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

#include "kernels.hpp"

namespace strait {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef unsigned uintx4 __attribute__((ext_vector_type(4)));

// Through the caches, acknowledged when it is there.  Not for host memory alone: the host may give the instance to another stream once it has seen the
// flag, before this kernel has ended and its plain stores are written back (see copy_out_kernel in elementwise.hip), and the next
// batch's logits may lie where this one's probabilities do.
__device__ __forceinline__ void out_store(char* p, float4 v) {
    const uintx4 r = __builtin_bit_cast(uintx4, v);
    asm volatile("global_store_dwordx4 %0, %1, off sc0 sc1\n\ts_nop 1" ::"v"(p), "v"(r) : "memory");   // (s_nop: see store_through in elementwise.hip)
}
__device__ __forceinline__ void out_store(char* p, float v) { __hip_atomic_store((float*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM); }

// POOL: from the feature map; V4: classes a multiple of four, moved 16 bytes at a time.
template <bool POOL, bool V4>
__global__ void __launch_bounds__(256) classify_out_kernel(const ClassifyOut p) {
    __shared__ float part[POOL ? 256 * 9 : 1];         // partial sums of the pooling (pitch 9: no conflicts)
    __shared__ __attribute__((aligned(16))) half_t feat[POOL ? 256 : 8];
    __shared__ float lg[POOL ? 256 : 1];
    __shared__ float red_max[4], red_sum[4];
    __shared__ int red_idx[4];
    if (p.hp) __builtin_amdgcn_s_setprio(3);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, row = blockIdx.x, n = p.n;
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

    // ---- largest logit, lowest index on ties
    float mx = -INFINITY;
    int mi = 0x7fffffff;
#pragma unroll
    for (int k = 0; k < 4; ++k)
        if (v[k] > mx) { mx = v[k]; mi = at[k]; }
    auto take = [&](float om, int oi) { if (om > mx || (om == mx && oi < mi)) { mx = om; mi = oi; } };
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const float om = __shfl_xor(mx, o, 64);
        const int oi = __shfl_xor(mi, o, 64);
        take(om, oi);
    }
    if (lane == 0) { red_max[wave] = mx; red_idx[wave] = mi; }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < 4; ++w) take(red_max[w], red_idx[w]);
    float e[4], sum = 0.f;
#pragma unroll
    for (int k = 0; k < 4; ++k) { e[k] = __expf(v[k] - mx); sum += e[k]; }    // exp(-inf) = 0 past the row's end
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
    if (lane == 0) red_sum[wave] = sum;
    __syncthreads();
    const float inv = 1.f / (red_sum[0] + red_sum[1] + red_sum[2] + red_sum[3]);

    // The computation's end, for STAMP_K1: that of the row whose result is the last to arrive.  (Counting the rows that got here as well would be exact to less than
    // the difference between two rows' ways to the host, and every row would wait for a second counter.)
    const uint64_t computed = wall_clock64();

    // ---- out: logits, probabilities and index, as they lie in the device's copy
    char* const host_logits = p.host + base * 4;
    char* const host_probs = p.host + ((size_t)p.rows * n + base) * 4;
    if constexpr (V4) {
        if (at[0] < n) {
            const float4 l = make_float4(v[0], v[1], v[2], v[3]), r = make_float4(e[0] * inv, e[1] * inv, e[2] * inv, e[3] * inv);
            out_store(host_logits + at[0] * 4, l);
            out_store(host_probs + at[0] * 4, r);
            if (POOL) out_store((char*)(p.logits + base + at[0]), l);
            out_store((char*)(p.probs + base + at[0]), r);
        }
    } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (at[k] >= n) continue;
            out_store(host_logits + at[k] * 4, v[k]);
            out_store(host_probs + at[k] * 4, e[k] * inv);
            if (POOL) out_store((char*)(p.logits + base + at[k]), v[k]);
            out_store((char*)(p.probs + base + at[k]), e[k] * inv);
        }
    }
    if (tid == 0) {
        __hip_atomic_store((int32_t*)(p.host + (size_t)p.rows * n * 8) + row, mi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        __hip_atomic_store(p.top1 + row, mi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    // each wavefront waits for its own stores to be acknowledged before the workgroup counts its row (see copy_out_kernel in elementwise.hip,
    // also for the order of the last stores)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    // Counted in groups of 32 rows, each on a line of its own, and then group by group: a single counter takes 10 ns a row (1000 rows 7 us).
    if (tid == 0) {
        const unsigned group = (unsigned)row >> 5, groups = ((unsigned)p.rows + 31) >> 5, mine = group + 1 == groups ? (unsigned)p.rows - 32 * group : 32u;
        unsigned* const count = p.counter + 32 * (group + 1);
        bool last = atomicAdd(count, 1u) == mine - 1;
        if (last) {
            __hip_atomic_store(count, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (groups > 1) {
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // the zero is there before this group counts
                last = atomicAdd(p.counter, 1u) == groups - 1;
                if (last) __hip_atomic_store(p.counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        if (last) {
            __hip_atomic_store(&p.ctl->stamp[STAMP_K1], computed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            __hip_atomic_store(&p.ctl->stamp[STAMP_DONE], (uint64_t)wall_clock64(), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __hip_atomic_store(&p.ctl->flag[0], p.seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
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
