// Bandwidth-bound kernels of the served models for gfx950: input packing, depthwise 3x3
// convolution, pooling, softmax + top-1, LayerNorm, argmax.  (Paper Section 3.2 step (2): the
// kernel sequence of a batch; these are its non-GEMM members.)
//
// None of these is a contraction worth MFMA: each reads its operands once from HBM/L2 and
// writes its result once, so the design rule is 16-byte accesses that are contiguous across
// the lanes of a wavefront (the channel axis of NHWC), fp32 arithmetic in registers, and
// enough workgroups (>> 256) to cover the chip.
#include <algorithm>

#include "kernels.hpp"

namespace strait {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half4 __attribute__((ext_vector_type(4)));

#define STRAIT_CHECK_LAUNCH(what)                                                   \
    do {                                                                            \
        hipError_t e_ = hipGetLastError();                                          \
        if (e_ != hipSuccess) { set_error(what ": %s", hipGetErrorString(e_)); return -2; } \
    } while (0)

__device__ __forceinline__ float act_f(float v, int act) {
    if (act == ACT_RELU) return fmaxf(v, 0.f);
    if (act == ACT_RELU6) return fminf(fmaxf(v, 0.f), 6.f);
    return v;
}

// ------------------------------------------------------------------------------------------
// fill
__global__ void fill_zero_kernel(uint4* p, size_t n16) {
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t step = (size_t)gridDim.x * blockDim.x;
    for (; i < n16; i += step) p[i] = make_uint4(0, 0, 0, 0);
}
int launch_fill_zero(void* p, size_t bytes, hipStream_t stream) {
    if (bytes == 0) return 0;
    if ((reinterpret_cast<uintptr_t>(p) & 15) || (bytes & 15)) { set_error("fill: 16-byte alignment required"); return -1; }
    const size_t n16 = bytes / 16;
    unsigned blocks = (unsigned)((n16 + 255) / 256 > 4096 ? 4096 : (n16 + 255) / 256);
    hipLaunchKernelGGL(fill_zero_kernel, dim3(blocks), dim3(256), 0, stream, (uint4*)p, n16);
    STRAIT_CHECK_LAUNCH("fill");
    return 0;
}

// ------------------------------------------------------------------------------------------
// Transfers between pinned host memory that the GPU can address and device memory, done by kernels: results on their way out,
// and inputs of up to a few megabytes on their way in.  (A hipMemcpyAsync of such a size, in either direction, now and then
// blocks the submitting thread for milliseconds when other streams are busy; a kernel launch does not.)  They also take the
// timestamps of a batch's record (the device's constant-rate clock, written to the instance's pinned control block) and
// the outgoing one tells the host that the result is there.  An event record costs about 3.6 us between two dependent launches and
// a wait on one 12 us from the last kernel to the waiting thread; the stamps cost nothing and the flag 7 us.
//
// What bounds them is the link, 53 GB/s; what they cost others is the requests they have under way.  A kernel of another stream that begins or ends waits until every
// cache has answered what it was asked, and an answer from host memory takes 1.5 us and the time of all that queues before it.  With 256 workgroups and four loads a
// thread a chain of 2.3 us kernels beside a copy of 2.4 MB took 22 us a kernel, that is, stood still, and the copy 48.5 us; 80 KB under way still fill the link:
//   workgroups of 256, one load a thread    32         24         20         16         12
//   copy us, chain us a kernel              45.1 10.1  45.3 8.1   46.0 7.0   49.1 6.6   63.6 6.4
// and on the way out, four stores a thread  16: 44.7 5.5   8: 45.3 3.7   4: 53.4 2.9.  Where no other stream has a batch 16 do it: with 8 a workgroup's waits, for what it loads
// and behind each part for its stores, leave the link idle (eight sequences' 1.6 MB 34.9 -> 30.2 us, 64 sequences' 12.6 MB 253 -> 229).  128 requests served by two models side by side 4.55 -> 4.25 ms, eight images
// of ResNet-50 alone 485 -> 477 us.
constexpr unsigned COPY_IN_BLOCKS = 20, COPY_OUT_BLOCKS = 16, COPY_OUT_BLOCKS_BESIDE = 8;
__device__ __forceinline__ void copy_range(const uint32_t* __restrict__ src, uint32_t* __restrict__ dst, size_t n4, unsigned block, unsigned blocks) {
    const size_t n16 = n4 >> 2;
    const size_t step = (size_t)blocks * 256;
    for (size_t i = (size_t)block * 256 + threadIdx.x; i < n16; i += step) ((uint4*)dst)[i] = ((const uint4*)src)[i];
    const size_t tail = n16 << 2;
    if (block == 0 && tail + threadIdx.x < n4) dst[tail + threadIdx.x] = src[tail + threadIdx.x];
}

// A piece of an input (and, for token models, the valid lengths behind it): dst <- src, dst2 <- src2, with a stamp at its start and end.
__global__ void __launch_bounds__(256) copy_in_kernel(const uint32_t* __restrict__ src, uint32_t* __restrict__ dst, size_t n4,
                                                      const uint32_t* __restrict__ src2, uint32_t* __restrict__ dst2, unsigned n4b,
                                                      HostControl* ctl, unsigned* counters, int piece) {
    if (blockIdx.x == 0 && threadIdx.x == 0) __hip_atomic_store(&ctl->stamp[STAMP_PIECES + 2 * piece], (uint64_t)wall_clock64(), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    copy_range(src, dst, n4, blockIdx.x, gridDim.x);
    if (blockIdx.x == 0)
        for (unsigned i = threadIdx.x; i < n4b; i += 256) dst2[i] = src2[i];
    __syncthreads();
    if (threadIdx.x == 0 && atomicAdd(&counters[0], 1u) == gridDim.x - 1) {      // the last workgroup to arrive
        __hip_atomic_store(&counters[0], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&ctl->stamp[STAMP_PIECES + 2 * piece + 1], (uint64_t)wall_clock64(), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}
int launch_copy_in(const void* src, void* dst, size_t bytes, const void* src2, void* dst2, size_t bytes2, HostControl* ctl, unsigned* counters,
                   int piece, hipStream_t stream) {
    if (!src || !dst || !ctl || !counters || piece < 0 || piece >= MAX_PIECES || bytes == 0 || (bytes & 3) || (bytes2 & 3) || bytes2 > (1u << 20) || (bytes2 && (!src2 || !dst2)) ||
        ((reinterpret_cast<uintptr_t>(src) | reinterpret_cast<uintptr_t>(dst)) & 15)) {
        set_error("copy in: 16-byte aligned buffers and multiples of 4 bytes required"); return -1;
    }
    const size_t n4 = bytes / 4, n16 = n4 / 4;
    const unsigned blocks = (unsigned)std::min<size_t>(COPY_IN_BLOCKS, std::max<size_t>(1, (n16 + 255) / 256));
    hipLaunchKernelGGL(copy_in_kernel, dim3(blocks), dim3(256), 0, stream, (const uint32_t*)src, (uint32_t*)dst, n4, (const uint32_t*)src2,
                       (uint32_t*)dst2, (unsigned)(bytes2 / 4), ctl, counters, piece);
    STRAIT_CHECK_LAUNCH("copy in");
    return 0;
}

// One timestamp between launches that do not take it themselves.  With src: also dst <- src (n4 words, before the stamp: the valid
// lengths behind an input that a copy engine brings).  With a sequence number: afterwards ctl->k1_seq = seq, which tells the
// host that the kernels before this one are done.
__global__ void __launch_bounds__(256) stamp_kernel(HostControl* ctl, int which, const uint32_t* __restrict__ src, uint32_t* __restrict__ dst, unsigned n4,
                                                    unsigned seq) {
    for (unsigned i = threadIdx.x; i < n4; i += 256) dst[i] = src[i];
    __syncthreads();
    if (threadIdx.x != 0) return;
    __hip_atomic_store(&ctl->stamp[which], (uint64_t)wall_clock64(), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    if (seq) __hip_atomic_store(&ctl->k1_seq, seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
int launch_stamp(HostControl* ctl, int which, hipStream_t stream, const void* src, void* dst, size_t bytes, unsigned seq) {
    if (!ctl || which < 0 || which >= STAMP_COUNT || (bytes & 3) || bytes > (1u << 20) || (bytes && (!src || !dst))) { set_error("stamp: bad argument"); return -1; }
    hipLaunchKernelGGL(stamp_kernel, dim3(1), dim3(bytes ? 256 : 64), 0, stream, ctl, which, (const uint32_t*)src, (uint32_t*)dst, (unsigned)(bytes / 4), seq);
    STRAIT_CHECK_LAUNCH("stamp");
    return 0;
}

// Result, in chunks of out_chunk_bytes, each in OUT_PARTS parts of which a workgroup takes every gridDim.x-th: when the last part of
// chunk c is written, flag[c] becomes `seq`, so that the host can move a chunk on while the next ones are on the link.  Stamps
// STAMP_K1 (first workgroup starts; if `k1_taken`, when the kernels were done, STAMP_D2H0 instead) and STAMP_DONE.  counters[1 + c] count a chunk's parts, counters[0] the
// chunks; both are back at zero, for every stream, before the last flag is set.
// Few workgroups (above).  The stores go through the
// caches (sc0 sc1) and each workgroup waits for its own to be acknowledged before it counts a part: a system-scope fence would
// instead write back the L2s, which hold other batches' data.  A store of 16 bytes still reads its registers for two wait states after it was issued, which
// the compiler does not count for inline assembly: an instruction that reused them right behind it would be stored in their place.
__device__ __forceinline__ void store_through(void* p, uint4 v) {
    typedef unsigned uint4v __attribute__((ext_vector_type(4)));
    const uint4v r = {v.x, v.y, v.z, v.w};
    asm volatile("global_store_dwordx4 %0, %1, off sc0 sc1\n\ts_nop 1" ::"v"(p), "v"(r) : "memory");
}
__global__ void __launch_bounds__(256) copy_out_kernel(const char* __restrict__ src, char* __restrict__ dst, size_t bytes, size_t part_bytes, unsigned parts, unsigned chunks,
                                                       HostControl* ctl, unsigned* counters, unsigned seq, int k1_taken, int hp) {
    if (hp) __builtin_amdgcn_s_setprio(3);
    if (blockIdx.x == 0 && threadIdx.x == 0)
        __hip_atomic_store(&ctl->stamp[k1_taken ? STAMP_D2H0 : STAMP_K1], (uint64_t)wall_clock64(), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    for (unsigned part = blockIdx.x; part < parts; part += gridDim.x) {
        const size_t at = (size_t)part * part_bytes, n = bytes - at < part_bytes ? bytes - at : part_bytes;
        const size_t n16 = n >> 4;
        const uint4* s16 = (const uint4*)(src + at);
        uint4* d16 = (uint4*)(dst + at);
        size_t i = threadIdx.x;
        for (; i + 768 < n16; i += 1024) {
            const uint4 a = s16[i], b = s16[i + 256], c = s16[i + 512], d = s16[i + 768];
            store_through(d16 + i, a); store_through(d16 + i + 256, b); store_through(d16 + i + 512, c); store_through(d16 + i + 768, d);
        }
        for (; i < n16; i += 256) store_through(d16 + i, s16[i]);
        const size_t tail = (n16 << 2) + threadIdx.x;
        if (tail < n >> 2) __hip_atomic_store((uint32_t*)(dst + at) + tail, ((const uint32_t*)(src + at))[tail], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        const unsigned c = part / OUT_PARTS;
        const unsigned mine = parts - c * OUT_PARTS < OUT_PARTS ? parts - c * OUT_PARTS : OUT_PARTS;     // parts of this chunk
        if (threadIdx.x == 0 && atomicAdd(&counters[1 + c], 1u) == mine - 1) {
            __hip_atomic_store(&counters[1 + c], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (atomicAdd(&counters[0], 1u) == chunks - 1) {
                __hip_atomic_store(&counters[0], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(&ctl->stamp[STAMP_DONE], (uint64_t)wall_clock64(), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            }
            // The host may give the instance to another stream as soon as it has seen every flag, before this kernel has ended
            // and its plain stores are written back: the zeros must be where every unit's atomics look before the flag is out.
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __hip_atomic_store(&ctl->flag[c], seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
}
int launch_copy_out(const void* src, void* dst, size_t bytes, HostControl* ctl, unsigned* counters, unsigned seq, bool k1_taken, int hp, bool beside, hipStream_t stream) {
    if (!src || !dst || !ctl || !counters || bytes == 0 || (bytes & 3) ||
        ((reinterpret_cast<uintptr_t>(src) | reinterpret_cast<uintptr_t>(dst)) & 15)) {
        set_error("copy out: 16-byte aligned buffers and a multiple of 4 bytes required"); return -1;
    }
    const size_t chunk = out_chunk_bytes(bytes), part = chunk / OUT_PARTS;
    const unsigned chunks = (unsigned)((bytes + chunk - 1) / chunk);
    const unsigned parts = (unsigned)((bytes + part - 1) / part);
    const unsigned blocks = std::min(parts, beside ? COPY_OUT_BLOCKS_BESIDE : COPY_OUT_BLOCKS);
    hipLaunchKernelGGL(copy_out_kernel, dim3(blocks), dim3(256), 0, stream, (const char*)src, (char*)dst, bytes, part, parts, chunks, ctl, counters, seq,
                       k1_taken ? 1 : 0, hp);
    STRAIT_CHECK_LAUNCH("copy out");
    return 0;
}

// ------------------------------------------------------------------------------------------
// pack: [N][H][W][C] (C <= Cpad, Cpad in {4, 8}) -> zero-bordered [N][Hp][Wp][Cpad].
// One thread per output pixel.
template <int CPAD>
__global__ void __launch_bounds__(256) pack_input_kernel(const half_t* __restrict__ x, int N, int H, int W, int C,
                                                          half_t* __restrict__ y, int Hp, int Wp, int pt, int pl, int hp) {
    if (hp) __builtin_amdgcn_s_setprio(3);
    const long long total = (long long)N * Hp * Wp;
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i >= total) return;
    const int wp = (int)(i % Wp);
    const long long t = i / Wp;
    const int hpix = (int)(t % Hp);
    const int n = (int)(t / Hp);
    const int h = hpix - pt, w = wp - pl;
    _Float16 v[CPAD];
#pragma unroll
    for (int c = 0; c < CPAD; ++c) v[c] = (half_t)0;
    if ((unsigned)h < (unsigned)H && (unsigned)w < (unsigned)W) {
        const half_t* src = x + (((long long)n * H + h) * W + w) * C;
#pragma unroll
        for (int c = 0; c < CPAD; ++c)
            if (c < C) v[c] = src[c];
    }
    half_t* dst = y + i * CPAD;
    if (CPAD == 4) *(half4*)dst = *(half4*)v; else *(half8*)dst = *(half8*)v;
}

int launch_pack_input(const half_t* x, int N, int H, int W, int C, half_t* y, int Hp, int Wp, int Cpad,
                      int pad_top, int pad_left, int hp, hipStream_t stream) {
    if (!x || !y || N <= 0 || H <= 0 || W <= 0 || C <= 0 || C > Cpad || (Cpad != 4 && Cpad != 8) ||
        Hp < H + pad_top || Wp < W + pad_left) { set_error("pack: invalid shape"); return -5; }
    const long long total = (long long)N * Hp * Wp;
    const long long blocks = (total + 255) / 256;
    if (blocks > 0x7fffffffLL) { set_error("pack: grid too large"); return -5; }
    if (Cpad == 4)
        hipLaunchKernelGGL(pack_input_kernel<4>, dim3((unsigned)blocks), dim3(256), 0, stream, x, N, H, W, C, y, Hp, Wp, pad_top, pad_left, hp);
    else
        hipLaunchKernelGGL(pack_input_kernel<8>, dim3((unsigned)blocks), dim3(256), 0, stream, x, N, H, W, C, y, Hp, Wp, pad_top, pad_left, hp);
    STRAIT_CHECK_LAUNCH("pack");
    return 0;
}

// Hardware workgroup id b runs on XCD b mod 8, each XCD with an L2 of its own.  This gives every XCD a contiguous
// range of logical block numbers instead, so that blocks which share input rows (vertically adjacent row tiles of a
// stencil) fetch them through one L2 rather than through several.
__device__ __forceinline__ unsigned xcd_contiguous_block() {
    const unsigned nb = gridDim.x, b = blockIdx.x;
    const unsigned per = nb >> 3, rem = nb & 7, xcd = b & 7, idx = b >> 3;
    return (xcd < rem ? xcd * (per + 1) : rem * (per + 1) + (xcd - rem) * per) + idx;
}

// A thread's place (n, p, q, c8) from its number ((n P + p) Q + q) C8 + c8.  A division is 20 to 40 dependent instructions, one of 64 bits 100, in front of the first
// load of kernels whose threads do a few loads each: numbers below 2^31 are divided by a product and a shift (WIDE: all others).  VGG-19 six images, five poolings
// 2x2: 535.8 -> 534.3 us.
struct Places { unsigned C8, Q, P; Divisor by_c8, by_q, by_p; };
static Places places(long long C8, long long Q, long long P) { return {(unsigned)C8, (unsigned)Q, (unsigned)P, divisor((unsigned)C8), divisor((unsigned)Q), divisor((unsigned)P)}; }
template <bool WIDE>
__device__ __forceinline__ void place(const Places& d, unsigned long long i, unsigned& n, unsigned& p, unsigned& q, unsigned& c8) {
    unsigned long long t, u;
    if (WIDE) { t = i / d.C8; u = t / d.Q; n = (unsigned)(u / d.P); }
    else { t = divide((unsigned)i, d.by_c8); u = divide((unsigned)t, d.by_q); n = divide((unsigned)u, d.by_p); }
    c8 = (unsigned)i - (unsigned)t * d.C8;
    q = (unsigned)t - (unsigned)u * d.Q;
    p = (unsigned)u - n * d.P;
}
#define STRAIT_PLACED(total, KERNEL, ...) \
    do { \
        if ((total) < 0x80000000LL) hipLaunchKernelGGL(KERNEL(false), __VA_ARGS__); \
        else hipLaunchKernelGGL(KERNEL(true), __VA_ARGS__); \
    } while (0)

// ------------------------------------------------------------------------------------------
// depthwise 3x3, pad 1, stride 1 or 2, fused bias + activation.
// A thread owns 8 channels (16 bytes) of TW consecutive output pixels of one output row.  For each
// of the three input rows it loads the (TW-1)*stride+3 input vectors the strip touches once and
// feeds all TW outputs from registers, so a strip of 4 costs 18 (stride 1) or 27 (stride 2) loads
// instead of 36, and the index arithmetic is paid once per strip.  Lanes of a wavefront cover
// consecutive channel groups, i.e. contiguous memory.  fp16 operands, fp32 accumulation.
template <int STRIDE, int TW, bool WIDE>
__global__ void __launch_bounds__(256) dwconv3x3_kernel(const half_t* __restrict__ x, int N, int H, int W, int C,
                                                         const half_t* __restrict__ w, const float* __restrict__ bias,
                                                         int act, half_t* __restrict__ y, int P, int Q, int hp, Places places) {
    if (hp) __builtin_amdgcn_s_setprio(3);
    constexpr int NV = (TW - 1) * STRIDE + 3;
    const unsigned C8 = (unsigned)C >> 3;
    const unsigned QT = (unsigned)(Q + TW - 1) / TW;
    const unsigned long long total = (unsigned long long)N * P * QT * C8;
    const unsigned long long i = (unsigned long long)xcd_contiguous_block() * 256 + threadIdx.x;
    if (i >= total) return;
    unsigned n, pp, qt, c8;
    place<WIDE>(places, i, n, pp, qt, c8);
    const int c = (int)c8 * 8;

    half8 wv[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) wv[k] = *(const half8*)(w + (long long)k * C + c);
    float acc[TW][8];
    {
        float bv[8];
        if (bias) {
            const float4 b0 = *(const float4*)(bias + c), b1 = *(const float4*)(bias + c + 4);
            bv[0] = b0.x; bv[1] = b0.y; bv[2] = b0.z; bv[3] = b0.w; bv[4] = b1.x; bv[5] = b1.y; bv[6] = b1.z; bv[7] = b1.w;
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) bv[j] = 0.f;
        }
#pragma unroll
        for (int tq = 0; tq < TW; ++tq)
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[tq][j] = bv[j];
    }
    const int q0 = (int)qt * TW;
    const int iw0 = q0 * STRIDE - 1;
    const half_t* xin = x + (long long)n * H * W * C + c;
#pragma unroll
    for (int r = 0; r < 3; ++r) {
        const int ih = (int)pp * STRIDE - 1 + r;
        if ((unsigned)ih >= (unsigned)H) continue;
        const half_t* row = xin + (long long)ih * W * C;
        half8 xv[NV];
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            const int iw = iw0 + k;
            if ((unsigned)iw < (unsigned)W) xv[k] = *(const half8*)(row + (long long)iw * C);
            else {
#pragma unroll
                for (int j = 0; j < 8; ++j) xv[k][j] = (half_t)0;
            }
        }
#pragma unroll
        for (int tq = 0; tq < TW; ++tq)
#pragma unroll
            for (int s = 0; s < 3; ++s)
#pragma unroll
                for (int j = 0; j < 8; ++j) acc[tq][j] += (float)xv[tq * STRIDE + s][j] * (float)wv[r * 3 + s][j];
    }
    half_t* yout = y + (((long long)n * P + pp) * Q + q0) * C + c;
#pragma unroll
    for (int tq = 0; tq < TW; ++tq) {
        if (q0 + tq < Q) {
            half8 o;
#pragma unroll
            for (int j = 0; j < 8; ++j) o[j] = (half_t)act_f(acc[tq][j], act);
            *(half8*)(yout + (long long)tq * C) = o;
        }
    }
}


// Stride 1, a column of TH outputs per thread.  Consecutive threads own consecutive 16-byte chunks along an image
// row (pixel-major, then channel group), so every load and store instruction of a wavefront covers one contiguous
// kilobyte whatever the channel count; a thread fetches the left, centre and right vector of each of the TH + 2
// input rows its column touches (the neighbours' copies of the same vectors hit in L1).  The strips of the kernel
// above leave, with few channels, gaps of TW pixels between the lanes of one instruction.  Every output
// accumulates its nine taps in the same order as there, so results are identical.
template <int TH, bool WIDE>
__global__ void __launch_bounds__(256) dwconv3x3_s1_cols_kernel(const half_t* __restrict__ x, int N, int H, int W, int C,
                                                                 const half_t* __restrict__ w, const float* __restrict__ bias,
                                                                 int act, half_t* __restrict__ y, int hp, Places places) {
    if (hp) __builtin_amdgcn_s_setprio(3);
    const unsigned C8 = (unsigned)C >> 3;
    const unsigned PT = (unsigned)(H + TH - 1) / TH;
    const unsigned long long total = (unsigned long long)N * PT * W * C8;
    const unsigned long long i = (unsigned long long)xcd_contiguous_block() * 256 + threadIdx.x;
    if (i >= total) return;
    unsigned n, pt, q, c8;
    place<WIDE>(places, i, n, pt, q, c8);
    const int c = (int)c8 * 8;
    half8 wv[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) wv[k] = *(const half8*)(w + (long long)k * C + c);
    float acc[TH][8];
    {
        float bv[8];
        if (bias) {
            const float4 b0 = *(const float4*)(bias + c), b1 = *(const float4*)(bias + c + 4);
            bv[0] = b0.x; bv[1] = b0.y; bv[2] = b0.z; bv[3] = b0.w; bv[4] = b1.x; bv[5] = b1.y; bv[6] = b1.z; bv[7] = b1.w;
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) bv[j] = 0.f;
        }
#pragma unroll
        for (int o = 0; o < TH; ++o)
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[o][j] = bv[j];
    }
    const int p0 = (int)pt * TH;
    const half_t* xin = x + ((long long)n * H * W + q) * C + c;
    const bool has_l = q > 0, has_r = q + 1 < (unsigned)W;
#pragma unroll
    for (int r = 0; r < TH + 2; ++r) {
        const int ih = p0 - 1 + r;
        if ((unsigned)ih >= (unsigned)H) continue;
        const half_t* row = xin + (long long)ih * W * C;
        half8 xv[3];
#pragma unroll
        for (int j = 0; j < 8; ++j) { xv[0][j] = (half_t)0; xv[2][j] = (half_t)0; }
        if (has_l) xv[0] = *(const half8*)(row - C);
        xv[1] = *(const half8*)row;
        if (has_r) xv[2] = *(const half8*)(row + C);
#pragma unroll
        for (int o = 0; o < TH; ++o) {
            const int fr = r - o;                       // filter row this input row is for output row p0 + o
            if (fr < 0 || fr > 2) continue;
#pragma unroll
            for (int sx = 0; sx < 3; ++sx)
#pragma unroll
                for (int j = 0; j < 8; ++j) acc[o][j] += (float)xv[sx][j] * (float)wv[fr * 3 + sx][j];
        }
    }
#pragma unroll
    for (int o = 0; o < TH; ++o) {
        if (p0 + o >= H) continue;
        half8 ov;
#pragma unroll
        for (int j = 0; j < 8; ++j) ov[j] = (half_t)act_f(acc[o][j], act);
        *(half8*)(y + (((long long)n * H + p0 + o) * W + q) * C + c) = ov;
    }
}

int launch_dwconv3x3(const half_t* x, int N, int H, int W, int C, const half_t* w_rsc, const float* bias,
                     int stride, int act, half_t* y, int hp, hipStream_t stream) {
    if (!x || !w_rsc || !y || N <= 0 || H <= 0 || W <= 0 || C <= 0 || C % 8 != 0 || (stride != 1 && stride != 2)) {
        set_error("dwconv3x3: needs C %% 8 == 0 and stride 1 or 2"); return -5;
    }
    if ((reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(w_rsc) | reinterpret_cast<uintptr_t>(y) |
         reinterpret_cast<uintptr_t>(bias)) & 15) { set_error("dwconv3x3: pointers must be 16-byte aligned"); return -1; }
    const int P = (H + 2 - 3) / stride + 1, Q = (W + 2 - 3) / stride + 1;
    constexpr int TW = 4;
    const long long total = (long long)N * P * ((Q + TW - 1) / TW) * (C / 8);
    const long long blocks = (total + 255) / 256;
    if (blocks > 0x7fffffffLL || (long long)N * P * ((Q + TW - 1) / TW) > 0xffffffffLL) { set_error("dwconv3x3: grid too large"); return -5; }
    constexpr int TH = 4;
    const long long total_cols = (long long)N * ((H + TH - 1) / TH) * W * (C / 8);
    if (stride == 1 && total_cols >= 16384 && (total_cols + 255) / 256 <= 0x7fffffffLL && (long long)N * ((H + TH - 1) / TH) * W <= 0xffffffffLL) {
#define DW_COLS(WIDE) (dwconv3x3_s1_cols_kernel<TH, WIDE>)
        STRAIT_PLACED(total_cols, DW_COLS, dim3((unsigned)((total_cols + 255) / 256)), dim3(256), 0, stream, x, N, H, W, C, w_rsc, bias, act, y, hp,
                      places(C / 8, W, (H + TH - 1) / TH));
    } else if (stride == 1) {
#define DW_ROWS1(WIDE) (dwconv3x3_kernel<1, TW, WIDE>)
        STRAIT_PLACED(total, DW_ROWS1, dim3((unsigned)blocks), dim3(256), 0, stream, x, N, H, W, C, w_rsc, bias, act, y, P, Q, hp, places(C / 8, (Q + TW - 1) / TW, P));
    } else {
#define DW_ROWS2(WIDE) (dwconv3x3_kernel<2, TW, WIDE>)
        STRAIT_PLACED(total, DW_ROWS2, dim3((unsigned)blocks), dim3(256), 0, stream, x, N, H, W, C, w_rsc, bias, act, y, P, Q, hp, places(C / 8, (Q + TW - 1) / TW, P));
    }
    STRAIT_CHECK_LAUNCH("dwconv3x3");
    return 0;
}

// ------------------------------------------------------------------------------------------
// max pooling 3x3 / stride 2 / pad 1.  Thread = 8 channels of one output pixel.
__global__ void __launch_bounds__(256) maxpool3x3s2_kernel(const half_t* __restrict__ x, int N, int H, int W, int C,
                                                            half_t* __restrict__ y, int P, int Q, int hp) {
    if (hp) __builtin_amdgcn_s_setprio(3);
    const int C8 = C >> 3;
    const long long total = (long long)N * P * Q * C8;
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i >= total) return;
    const int c8 = (int)(i % C8);
    long long t = i / C8;
    const int q = (int)(t % Q); t /= Q;
    const int pp = (int)(t % P);
    const int n = (int)(t / P);
    half8 m;
#pragma unroll
    for (int j = 0; j < 8; ++j) m[j] = (half_t)(-65504.f);
    bool any = false;
#pragma unroll
    for (int r = 0; r < 3; ++r) {
        const int ih = pp * 2 - 1 + r;
        if ((unsigned)ih >= (unsigned)H) continue;
#pragma unroll
        for (int s = 0; s < 3; ++s) {
            const int iw = q * 2 - 1 + s;
            if ((unsigned)iw >= (unsigned)W) continue;
            const half8 v = *(const half8*)(x + (((long long)n * H + ih) * W + iw) * C + c8 * 8);
#pragma unroll
            for (int j = 0; j < 8; ++j) m[j] = (!any || v[j] > m[j]) ? v[j] : m[j];
            any = true;
        }
    }
    *(half8*)(y + (((long long)n * P + pp) * Q + q) * C + c8 * 8) = m;
}

int launch_maxpool3x3s2(const half_t* x, int N, int H, int W, int C, half_t* y, int hp, hipStream_t stream) {
    if (!x || !y || N <= 0 || H <= 0 || W <= 0 || C <= 0 || C % 8 != 0) { set_error("maxpool: needs C %% 8 == 0"); return -5; }
    const int P = (H + 2 - 3) / 2 + 1, Q = (W + 2 - 3) / 2 + 1;
    const long long blocks = ((long long)N * P * Q * (C / 8) + 255) / 256;
    if (blocks > 0x7fffffffLL) { set_error("maxpool: grid too large"); return -5; }
    hipLaunchKernelGGL(maxpool3x3s2_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, x, N, H, W, C, y, P, Q, hp);
    STRAIT_CHECK_LAUNCH("maxpool");
    return 0;
}

// ------------------------------------------------------------------------------------------
// max pooling 2x2 / stride 2, no padding (H, W even).  Thread = 8 channels of one output pixel.
template <bool WIDE>
__global__ void __launch_bounds__(256) maxpool2x2s2_kernel(const half_t* __restrict__ x, int N, int H, int W, int C,
                                                            half_t* __restrict__ y, int hp, Places places) {
    if (hp) __builtin_amdgcn_s_setprio(3);
    const int C8 = C >> 3, P = H >> 1, Q = W >> 1;
    const long long total = (long long)N * P * Q * C8;
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i >= total) return;
    unsigned n, pp, q, c8;
    place<WIDE>(places, i, n, pp, q, c8);
    const half_t* src = x + (((long long)n * H + 2 * pp) * W + 2 * q) * C + c8 * 8;
    const half8 a = *(const half8*)src, b = *(const half8*)(src + C);
    const half8 c = *(const half8*)(src + (long long)W * C), d = *(const half8*)(src + (long long)W * C + C);
    const half8 m = __builtin_elementwise_max(__builtin_elementwise_max(a, b), __builtin_elementwise_max(c, d));
    *(half8*)(y + i * 8) = m;                          // (the output's order is the threads')
}

int launch_maxpool2x2s2(const half_t* x, int N, int H, int W, int C, half_t* y, int hp, hipStream_t stream) {
    if (!x || !y || N <= 0 || H <= 0 || W <= 0 || C <= 0 || C % 8 != 0 || H % 2 != 0 || W % 2 != 0) {
        set_error("maxpool 2x2: needs C %% 8 == 0 and even H, W"); return -5;
    }
    const long long total = (long long)N * (H / 2) * (W / 2) * (C / 8), blocks = (total + 255) / 256;
    if (blocks > 0x7fffffffLL) { set_error("maxpool 2x2: grid too large"); return -5; }
#define POOL2X2(WIDE) maxpool2x2s2_kernel<WIDE>
    STRAIT_PLACED(total, POOL2X2, dim3((unsigned)blocks), dim3(256), 0, stream, x, N, H, W, C, y, hp, places(C / 8, W / 2, H / 2));
    STRAIT_CHECK_LAUNCH("maxpool 2x2");
    return 0;
}

// ------------------------------------------------------------------------------------------
// Token assembly of a Vision Transformer: z[n][0] = cls + pos[0], z[n][1 + t] = patch[n][t] + pos[1 + t],
// sums in fp32 rounded once.  patch [N][T][D], cls [D], pos [T + 1][D] fp32, z [N][T + 1][D].
template <bool WIDE>
__global__ void __launch_bounds__(256) vit_tokens_kernel(const half_t* __restrict__ patch, const float* __restrict__ cls,
                                                          const float* __restrict__ pos, int N, int T, int D,
                                                          half_t* __restrict__ z, int hp, Places places) {
    if (hp) __builtin_amdgcn_s_setprio(3);
    const int D8 = D >> 3;
    const long long total = (long long)N * (T + 1) * D8;
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i >= total) return;
    unsigned n, one, tok, d8;
    place<WIDE>(places, i, n, one, tok, d8);
    float v[8];
    if (tok == 0) {
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = cls[d8 * 8 + j];
    } else {
        const half8 h = *(const half8*)(patch + ((long long)n * T + tok - 1) * D + d8 * 8);
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = (float)h[j];
    }
    half8 o;
#pragma unroll
    for (int j = 0; j < 8; ++j) o[j] = (half_t)(v[j] + pos[(long long)tok * D + d8 * 8 + j]);
    *(half8*)(z + i * 8) = o;
}

int launch_vit_tokens(const half_t* patch, const float* cls, const float* pos, int N, int T, int D, half_t* z, int hp,
                      hipStream_t stream) {
    if (!patch || !cls || !pos || !z || N <= 0 || T <= 0 || D <= 0 || D % 8 != 0) { set_error("tokens: needs D %% 8 == 0"); return -5; }
    const long long total = (long long)N * (T + 1) * (D / 8), blocks = (total + 255) / 256;
    if (blocks > 0x7fffffffLL) { set_error("tokens: grid too large"); return -5; }
#define TOKENS(WIDE) vit_tokens_kernel<WIDE>
    STRAIT_PLACED(total, TOKENS, dim3((unsigned)blocks), dim3(256), 0, stream, patch, cls, pos, N, T, D, z, hp, places(D / 8, T + 1, 1));
    STRAIT_CHECK_LAUNCH("tokens");
    return 0;
}

// ------------------------------------------------------------------------------------------
// global average pooling: [N][HW][C] -> [N][C], fp32 sum / HW, rounded once to fp16.
// A workgroup covers 32 channel groups (256 channels) of one image; its 8 wavefront-halves each
// sum every 8th position and the partial sums meet in LDS, so the loads of one image are spread
// over 8 independent chains instead of one serial walk over HW.
__global__ void __launch_bounds__(256) gap_kernel(const half_t* __restrict__ x, int N, int HW, int C,
                                                   half_t* __restrict__ y, int hp) {
    __shared__ float part[8][32][8];
    if (hp) __builtin_amdgcn_s_setprio(3);
    const int C8 = C >> 3;
    const int g = threadIdx.x & 31, part_id = threadIdx.x >> 5;
    const int c8 = blockIdx.x * 32 + g, n = blockIdx.y;
    float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if (c8 < C8) {
        const half_t* src = x + (long long)n * HW * C + c8 * 8;
        for (int k = part_id; k < HW; k += 8) {
            const half8 v = *(const half8*)(src + (long long)k * C);
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[j] += (float)v[j];
        }
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) part[part_id][g][j] = acc[j];
    __syncthreads();
    if (part_id == 0 && c8 < C8) {
        const float inv = 1.f / (float)HW;
        half8 o;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            float s = 0.f;
#pragma unroll
            for (int q = 0; q < 8; ++q) s += part[q][g][j];
            o[j] = (half_t)(s * inv);
        }
        *(half8*)(y + (long long)n * C + c8 * 8) = o;
    }
}

int launch_global_avgpool(const half_t* x, int N, int HW, int C, half_t* y, int hp, hipStream_t stream) {
    if (!x || !y || N <= 0 || HW <= 0 || C <= 0 || C % 8 != 0 || N > 65535) { set_error("avgpool: needs C %% 8 == 0 and N <= 65535"); return -5; }
    hipLaunchKernelGGL(gap_kernel, dim3((unsigned)((C / 8 + 31) / 32), (unsigned)N), dim3(256), 0, stream, x, N, HW, C, y, hp);
    STRAIT_CHECK_LAUNCH("avgpool");
    return 0;
}

// ------------------------------------------------------------------------------------------
// wavefront reductions (64 lanes) through cross-lane shuffles
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    return v;
}
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// softmax + top-1: one wavefront per row of fp32 logits; rows of up to 64 * PER elements are read
// once and kept in registers (PER = 16 covers the 1000-class heads), longer rows are re-read.
template <int PER>
__global__ void __launch_bounds__(256) softmax_top1_kernel(const float* __restrict__ logits, int rows, int n,
                                                            float* __restrict__ probs, int32_t* __restrict__ top1, int hp) {
    if (hp) __builtin_amdgcn_s_setprio(3);
    const int lane = threadIdx.x & 63;
    const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= rows) return;
    const float* src = logits + (long long)row * n;
    float v[PER > 0 ? PER : 1];
    float mx = -INFINITY;
    int mi = 0x7fffffff;
    if (PER > 0) {
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int i = lane + k * 64;
            v[k] = i < n ? src[i] : -INFINITY;
            if (v[k] > mx) { mx = v[k]; mi = i; }           // ascending i: keeps the lowest index on ties
        }
    } else {
        for (int i = lane; i < n; i += 64) {
            const float t = src[i];
            if (t > mx) { mx = t; mi = i; }
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const float ov = __shfl_xor(mx, o, 64);
        const int oi = __shfl_xor(mi, o, 64);
        if (ov > mx || (ov == mx && oi < mi)) { mx = ov; mi = oi; }
    }
    float sum = 0.f;
    if (PER > 0) {
#pragma unroll
        for (int k = 0; k < PER; ++k) { v[k] = __expf(v[k] - mx); sum += v[k]; }    // exp(-inf) = 0 past the row end
    } else {
        for (int i = lane; i < n; i += 64) sum += __expf(src[i] - mx);
    }
    sum = wave_sum(sum);
    const float inv = 1.f / sum;
    float* dst = probs + (long long)row * n;
    if (PER > 0) {
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int i = lane + k * 64;
            if (i < n) dst[i] = v[k] * inv;
        }
    } else {
        for (int i = lane; i < n; i += 64) dst[i] = __expf(src[i] - mx) * inv;
    }
    if (lane == 0) top1[row] = mi;
}

int launch_softmax_top1(const float* logits, int rows, int n, float* probs, int32_t* top1, int hp, hipStream_t stream) {
    if (!logits || !probs || !top1 || rows <= 0 || n <= 0) { set_error("softmax: invalid shape"); return -5; }
    const dim3 grid((rows + 3) / 4), block(256);
    if (n <= 128) hipLaunchKernelGGL(softmax_top1_kernel<2>, grid, block, 0, stream, logits, rows, n, probs, top1, hp);
    else if (n <= 1024) hipLaunchKernelGGL(softmax_top1_kernel<16>, grid, block, 0, stream, logits, rows, n, probs, top1, hp);
    else hipLaunchKernelGGL(softmax_top1_kernel<0>, grid, block, 0, stream, logits, rows, n, probs, top1, hp);
    STRAIT_CHECK_LAUNCH("softmax");
    return 0;
}

// argmax over n fp16 features of selected rows: one wavefront per row.
__global__ void __launch_bounds__(256) argmax_f16_kernel(const half_t* __restrict__ x, int rows, int n, long long row_stride,
                                                          int32_t* __restrict__ top1, int hp) {
    if (hp) __builtin_amdgcn_s_setprio(3);
    const int lane = threadIdx.x & 63;
    const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= rows) return;
    const half_t* src = x + (long long)row * row_stride;
    float mx = -INFINITY;
    int mi = 0x7fffffff;
    for (int i = lane; i < n; i += 64) {
        const float v = (float)src[i];
        if (v > mx) { mx = v; mi = i; }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const float ov = __shfl_xor(mx, o, 64);
        const int oi = __shfl_xor(mi, o, 64);
        if (ov > mx || (ov == mx && oi < mi)) { mx = ov; mi = oi; }
    }
    if (lane == 0) top1[row] = mi;
}

int launch_argmax_f16(const half_t* x, int rows, int n, long long row_stride, int32_t* top1, int hp, hipStream_t stream) {
    if (!x || !top1 || rows <= 0 || n <= 0 || row_stride < n) { set_error("argmax: invalid shape"); return -5; }
    hipLaunchKernelGGL(argmax_f16_kernel, dim3((rows + 3) / 4), dim3(256), 0, stream, x, rows, n, row_stride, top1, hp);
    STRAIT_CHECK_LAUNCH("argmax");
    return 0;
}

// ------------------------------------------------------------------------------------------
// LayerNorm: one wavefront per row, the row held in registers (n <= 8192 -> at most 16 chunks
// of 8 per lane), two-pass mean / variance in fp32.  Rows whose 8-element chunks do not fill 64 lanes evenly but do
// fill 32 (768 features = 96 chunks) go to half a wavefront each: LPR lanes per row.
template <int MAXC, int LPR>
__global__ void __launch_bounds__(256) layernorm_kernel(const half_t* __restrict__ x, const float* __restrict__ gamma,
                                                         const float* __restrict__ beta, int rows, int n, float eps,
                                                         half_t* __restrict__ y, int hp, long long x_row_stride) {
    if (hp) __builtin_amdgcn_s_setprio(3);
    const int lane = threadIdx.x & (LPR - 1);
    const int row = blockIdx.x * (256 / LPR) + threadIdx.x / LPR;
    if (row >= rows) return;                    // whole groups of LPR lanes leave together: the shuffles below stay inside a group
    auto group_sum = [](float t) {
#pragma unroll
        for (int o = LPR / 2; o > 0; o >>= 1) t += __shfl_xor(t, o, 64);
        return t;
    };
    const int nch = n >> 3;
    const half_t* src = x + (long long)row * x_row_stride;
    float v[MAXC][8];
    float s = 0.f;
#pragma unroll
    for (int c = 0; c < MAXC; ++c) {
        const int idx = lane + c * LPR;
        if (idx < nch) {
            const half8 h = *(const half8*)(src + idx * 8);
#pragma unroll
            for (int j = 0; j < 8; ++j) { v[c][j] = (float)h[j]; s += v[c][j]; }
        }
    }
    const float mean = group_sum(s) / (float)n;
    float q = 0.f;
#pragma unroll
    for (int c = 0; c < MAXC; ++c)
        if (lane + c * LPR < nch) {
#pragma unroll
            for (int j = 0; j < 8; ++j) { const float d = v[c][j] - mean; q += d * d; }
        }
    const float rstd = 1.f / sqrtf(group_sum(q) / (float)n + eps);
    half_t* dst = y + (long long)row * n;
#pragma unroll
    for (int c = 0; c < MAXC; ++c) {
        const int idx = lane + c * LPR;
        if (idx < nch) {
            half8 o;
#pragma unroll
            for (int j = 0; j < 8; ++j)
                o[j] = (half_t)((v[c][j] - mean) * rstd * gamma[idx * 8 + j] + beta[idx * 8 + j]);
            *(half8*)(dst + idx * 8) = o;
        }
    }
}

int launch_layernorm(const half_t* x, const float* gamma, const float* beta, int rows, int n, float eps,
                     half_t* y, int hp, hipStream_t stream, long long x_row_stride) {
    if (x_row_stride == 0) x_row_stride = n;
    if (!x || !gamma || !beta || !y || rows <= 0 || n <= 0 || n % 8 != 0 || n > 8192 || x_row_stride < n || x_row_stride % 8 != 0) {
        set_error("layernorm: needs n %% 8 == 0, n <= 8192 and a row stride that is a multiple of 8, at least n"); return -5;
    }
    const dim3 grid((rows + 3) / 4), block(256);
    const int nch = n / 8;
    if (nch <= 128 && nch % 32 == 0 && nch % 64 != 0)
        hipLaunchKernelGGL((layernorm_kernel<4, 32>), dim3((rows + 7) / 8), block, 0, stream, x, gamma, beta, rows, n, eps, y, hp, x_row_stride);
    else if (nch <= 128)
        hipLaunchKernelGGL((layernorm_kernel<2, 64>), grid, block, 0, stream, x, gamma, beta, rows, n, eps, y, hp, x_row_stride);
    else if (nch <= 512)
        hipLaunchKernelGGL((layernorm_kernel<8, 64>), grid, block, 0, stream, x, gamma, beta, rows, n, eps, y, hp, x_row_stride);
    else
        hipLaunchKernelGGL((layernorm_kernel<16, 64>), grid, block, 0, stream, x, gamma, beta, rows, n, eps, y, hp, x_row_stride);
    STRAIT_CHECK_LAUNCH("layernorm");
    return 0;
}

}  // namespace strait
