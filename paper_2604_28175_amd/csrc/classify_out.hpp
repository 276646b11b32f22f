// The end of a classifier's sample: softmax, top-1 and the result's way to the host (classify_out.hip says why), for the kernels that end with it.
#pragma once
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

template <int NW> struct ClassifyReduce { float max[NW], sum[NW]; int idx[NW]; };

// One workgroup of NW wavefronts, one sample; v: this thread's logits (-inf past the row's end), at: their classes.  V4: classes a multiple of four, a thread's
// beside each other, moved 16 bytes at a time.  LOGITS: the device's copy of the logits is to be written too.
template <int NW, bool V4, bool LOGITS>
__device__ __forceinline__ void classify_end(const ClassifyOut& p, int row, const float (&v)[4], const int (&at)[4], ClassifyReduce<NW>& red) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, n = p.n;
    const size_t base = (size_t)row * n;
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
    if (lane == 0) { red.max[wave] = mx; red.idx[wave] = mi; }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < NW; ++w) take(red.max[w], red.idx[w]);
    float e[4], sum = 0.f;
#pragma unroll
    for (int k = 0; k < 4; ++k) { e[k] = __expf(v[k] - mx); sum += e[k]; }    // exp(-inf) = 0 past the row's end
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
    if (lane == 0) red.sum[wave] = sum;
    __syncthreads();
    float total = red.sum[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) total += red.sum[w];
    const float inv = 1.f / total;

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
            if (LOGITS) out_store((char*)(p.logits + base + at[0]), l);
            out_store((char*)(p.probs + base + at[0]), r);
        }
    } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (at[k] >= n) continue;
            out_store(host_logits + at[k] * 4, v[k]);
            out_store(host_probs + at[k] * 4, e[k] * inv);
            if (LOGITS) out_store((char*)(p.logits + base + at[k]), v[k]);
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

}  // namespace strait
