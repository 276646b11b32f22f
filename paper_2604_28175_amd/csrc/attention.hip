// Fused masked multi-head attention for gfx950: scores, key-padding mask, softmax and the
// product with V in one kernel; the S x S score matrix never leaves registers.
// (Paper Section 3.2 step (2): one member of the encoder workload's kernel sequence.)
//
//   out[b, i, h*64 + :] = softmax_j( q_i . k_j / sqrt(64) ,  j < valid_len[b] ) @ V
//
// A workgroup of 4 wavefronts takes all query rows of one (sequence, head), or one of two halves of them, in blocks of 32
// rows that the wavefronts take in turn; S need not be a multiple of anything: query rows at or beyond S are neither
// read nor written, and key rows at or beyond valid_len arrive in LDS as zeros, so that masked keys can never inject
// non-finite values.
//   - K and V go to LDS as they lie in memory, 128 bytes a row, without passing through registers (buffer_load_dwordx4 ... lds;
//     the buffer ends at row valid_len, and what lies beyond reads as zero).  The 16-byte chunk c of row r sits at
//     c ^ (r & 7) for K, whose operand is 8 rows at one chunk, and at c ^ (bits of r & 7 reversed) for V, whose operand is 4
//     rows at 4 chunks: neither read has a bank conflict;
//   - scores^T = K Q^T with v_mfma_f32_32x32x16_f16 (K rows are the "A" operand), which leaves each lane holding 16 of a
//     block's 32 keys for ONE query: the row maximum and sum need a single exchange with lane ^ 32;
//   - 64 keys at a time with a running maximum: 121 registers whatever the length.  Keeping all scores of 197 keys took 176
//     and left one workgroup of 8 wavefronts per compute unit, which then loaded, computed and stored in turn;
//   - the probabilities, rounded to fp16, are already laid out as the "B" operand of out^T = V^T P^T provided V^T's reduction
//     index is enumerated in the same (permuted) key order: ds_read_b64_tr_b16 transposes 4 keys x 16 features on the way
//     to the registers, two of them per operand;
//   - 32-key blocks and 16-key steps that lie entirely beyond valid_len are skipped.
// Measured (12 heads): 64 x 197 keys 41.5 -> 23.8 us (77 MB moved: 3.2 TB/s; between the vector units' exponentials, about 10 us,
// and the loads, which the three workgroups of a compute unit all issue at the start), 7 x 197 12.4 -> 6.5, 64 x 128 17.1 ->
// 11.4, 8 x 128 7.4 -> 4.8 (a launch and two memory round trips).
#include <type_traits>

#include "kernels.hpp"

namespace strait {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef __fp16 fp16x4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef int intx4 __attribute__((ext_vector_type(4)));
typedef unsigned uintx2 __attribute__((ext_vector_type(2)));
typedef unsigned uintx4 __attribute__((ext_vector_type(4)));

constexpr int ATT_D = 64;
constexpr int ATT_WAVES = 4;
constexpr int ATT_KB = 2;                // blocks of 32 keys per step
constexpr unsigned ATT_ROW = ATT_D * 2;  // bytes of a K or V row in LDS

// One wave-wide transfer of 64 x 16 bytes: lane i's chunk at rsrc.base + voff goes to LDS byte address lds_base + 16 i.
__device__ __forceinline__ void att_dma16(intx4 rsrc, unsigned voff, unsigned lds_base) {
    const unsigned m0v = __builtin_amdgcn_readfirstlane(lds_base);
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(m0v), "v"(voff), "s"(rsrc) : "memory");
}
// The value of this lane and of lane ^ 32: {lanes 0-31's, lanes 32-63's}.
__device__ __forceinline__ float2 both_halves(float v) {
    const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, v), __builtin_bit_cast(unsigned, v), false, false);
    const unsigned lo = r[0], hi = r[1];
    return {__builtin_bit_cast(float, lo), __builtin_bit_cast(float, hi)};
}

__global__ void __launch_bounds__(64 * ATT_WAVES, 4) attention_kernel(const half_t* __restrict__ qkv, const int32_t* __restrict__ valid_len, int S, int heads,
                                                                      int seq_heads, int blocks_per_wg, half_t* __restrict__ out, int hp, Divisor by_heads) {
    extern __shared__ __attribute__((aligned(16))) char att_lds[];      // K rows, then V rows, valid_len rounded up to 16 of each
    if (hp) __builtin_amdgcn_s_setprio(3);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, lh = lane >> 5;
    // (at most two parts; the two divisions took 80 dependent instructions in front of the first load)
    const int part = (int)blockIdx.x >= seq_heads ? 1 : 0, sh = blockIdx.x - part * seq_heads;
    const int b = divide(sh, by_heads), h = sh - b * heads;
    const int nq = (S + 31) >> 5;
    const int qb0 = part * blocks_per_wg, qb1 = qb0 + blocks_per_wg < nq ? qb0 + blocks_per_wg : nq;
    const int hidden = heads * ATT_D, pitch = 3 * hidden;
    const half_t* seq = qkv + (long long)b * S * pitch;
    int L = valid_len[b];
    L = L < 0 ? 0 : (L > S ? S : L);

    // ---- stage K and V: pieces of 8 rows, a lane brings chunk (lane & 7) of row lane >> 3, swizzled
    const unsigned pieces = (unsigned)(L + 15) / 16 * 2;
    const unsigned lds0 = (unsigned)(uintptr_t)att_lds, lds_v = lds0 + pieces * 8 * ATT_ROW;
    if (qb0 * 32 < L) {
        // raw buffer of the rows below L among the 8 rows of a piece: a descriptor per piece, whose offsets fit 32 bits whatever the length
        auto rows8 = [&](unsigned p) -> intx4 {
            const unsigned long long a = (unsigned long long)(seq + (long long)p * 8 * pitch);
            const int left = L - (int)p * 8;
            return {__builtin_amdgcn_readfirstlane((int)(unsigned)a), __builtin_amdgcn_readfirstlane((int)((unsigned)(a >> 32) & 0xffffu)),
                    __builtin_amdgcn_readfirstlane((left < 0 ? 0 : left < 8 ? left : 8) * pitch * 2), 0x00020000};
        };
        const unsigned r = lane >> 3, c = lane & 7, rev = ((r & 1) << 2) | (r & 2) | (r >> 2);
        const unsigned row = r * (unsigned)pitch * 2u + (unsigned)h * ATT_ROW;
        const unsigned koff = row + (unsigned)hidden * 2u + ((c ^ r) << 4), voff = row + (unsigned)hidden * 4u + ((c ^ rev) << 4);
        for (unsigned p = wave; p < pieces; p += ATT_WAVES) att_dma16(rows8(p), koff, lds0 + p * 8 * ATT_ROW);
        for (unsigned p = wave; p < pieces; p += ATT_WAVES) att_dma16(rows8(p), voff, lds_v + p * 8 * ATT_ROW);
    }
    half8 qf[4];
    auto load_q = [&](int qb) {
        if (qb >= qb1 || qb * 32 >= L) return;
        const int q = qb * 32 + l32 < S ? qb * 32 + l32 : S - 1;        // a ragged last block reads a row that exists
        const half_t* qrow = seq + (long long)q * pitch + h * ATT_D;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) qf[ks] = *(const half8*)(qrow + ks * 16 + lh * 8);
    };
    load_q(qb0 + wave);
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");

    const char* krow = att_lds + l32 * ATT_ROW;
    unsigned kchunk[4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) kchunk[ks] = (unsigned)(((ks * 2 + lh) ^ (l32 & 7)) << 4);
    // V: lane i of a group of 16 names keys 4 lh + (i >> 2), features 16 ((lane >> 4) & 1) + 4 (i & 3) .. + 3 of a 16-key step and a
    // 32-feature half, and receives the step's keys 4 lh .. 4 lh + 3 of feature 16 ((lane >> 4) & 1) + i
    const unsigned i16 = lane & 15, vr = lh * 4 + (i16 >> 2), vrev = ((vr & 1) << 2) | (vr & 2) | (vr >> 2);
    const unsigned vbase = lds_v + vr * ATT_ROW + (i16 & 1) * 8, vchunk = (((lane >> 4) & 1) * 2 + ((i16 & 3) >> 1)) ^ vrev;
    const unsigned vaddr[2] = {vbase + (vchunk << 4), vbase + ((vchunk ^ 4) << 4)};
    auto vread = [](unsigned a) { return __builtin_amdgcn_ds_read_tr16_b64_v4f16((__attribute__((address_space(3))) fp16x4*)(uintptr_t)a); };

    for (int qb = qb0 + wave; qb < qb1; qb += ATT_WAVES) {
        const int q0 = qb * 32;
        const bool row_ok = q0 + l32 < S;       // a ragged last block: rows at or beyond S are not written
        half_t* orow = out + ((long long)b * S + q0 + l32) * hidden + h * ATT_D;
        if (q0 >= L) {                          // whole query block is padding: defined output, no work
            if (row_ok) {
#pragma unroll
                for (int i = 0; i < 4; ++i) *(uintx4*)(orow + 16 * i + 8 * lh) = uintx4{0, 0, 0, 0};
            }
            continue;
        }
        if (qb != qb0 + wave) load_q(qb);
        const float c = 0.125f * 1.44269504088896340736f;       // 1/sqrt(64), and log2(e): the probabilities are powers of two
        floatx16 o[2];
#pragma unroll
        for (int v = 0; v < 16; ++v) o[0][v] = o[1][v] = 0.f;
        float mx = -INFINITY, sum = 0.f;        // running maximum of the row, and this lane's part of the sum
        auto step = [&](int k0, auto masked) __attribute__((always_inline)) {
            constexpr bool MASK = decltype(masked)::value;
            floatx16 sc[ATT_KB];                // lane holds query q0 + l32 against keys k0 + kb*32 + 8g + 4*lh + j  (v = 4g + j)
            float m = mx;
#pragma unroll
            for (int kb = 0; kb < ATT_KB; ++kb) {
#pragma unroll
                for (int v = 0; v < 16; ++v) sc[kb][v] = 0.f;
                if (!MASK || k0 + kb * 32 < L) {
#pragma unroll
                    for (int ks = 0; ks < 4; ++ks)
                        sc[kb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(*(const half8*)(krow + (k0 + kb * 32) * ATT_ROW + kchunk[ks]), qf[ks], sc[kb], 0, 0, 0);
                }
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    if (MASK && k0 + kb * 32 + 8 * (v >> 2) + 4 * lh + (v & 3) >= L) sc[kb][v] = -INFINITY;
                    m = fmaxf(m, sc[kb][v]);
                }
            }
            const float2 mm = both_halves(m);
            m = fmaxf(mm.x, mm.y);
            const float mc = m > -INFINITY ? m * c : 0.f;     // nothing but -inf so far: probabilities of 0, as if these keys were masked
            if (k0 > 0) {
                const float alpha = __builtin_amdgcn_exp2f(__builtin_fmaf(mx, c, -mc));
                sum *= alpha;
#pragma unroll
                for (int v = 0; v < 16; ++v) { o[0][v] *= alpha; o[1][v] *= alpha; }
            }
            mx = m;
#pragma unroll
            for (int st = 0; st < 2 * ATT_KB; ++st) {
                if (MASK && k0 + st * 16 >= L) continue;
                half8 pf;
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const float pv = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[st >> 1][(st & 1) * 8 + j], c, -mc));
                    sum += pv;
                    pf[j] = (half_t)pv;
                }
#pragma unroll
                for (int db = 0; db < 2; ++db) {
                    const unsigned a = vaddr[db] + (unsigned)(k0 + st * 16) * ATT_ROW;
                    const fp16x4 lo = vread(a), hi = vread(a + 8 * ATT_ROW);
                    half8 vf;
#pragma unroll
                    for (int j = 0; j < 4; ++j) { vf[j] = (half_t)lo[j]; vf[4 + j] = (half_t)hi[j]; }
                    o[db] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vf, pf, o[db], 0, 0, 0);
                }
            }
        };
        int k0 = 0;
        for (; k0 + 32 * ATT_KB <= L; k0 += 32 * ATT_KB) step(k0, std::false_type{});
        if (k0 < L) step(k0, std::true_type{});
        const float2 ss = both_halves(sum);
        const float inv = 1.f / (ss.x + ss.y);
        // lane holds out[q0+l32][db*32 + 8g + 4*lh + j]; after the exchange with lane ^ 32, 8 features of one g
#pragma unroll
        for (int db = 0; db < 2; ++db)
#pragma unroll
            for (int g = 0; g < 4; g += 2) {
                half4 e, f;
#pragma unroll
                for (int j = 0; j < 4; ++j) { e[j] = (half_t)(o[db][4 * g + j] * inv); f[j] = (half_t)(o[db][4 * g + 4 + j] * inv); }
                const uintx2 eu = __builtin_bit_cast(uintx2, e), fu = __builtin_bit_cast(uintx2, f);
                const auto x = __builtin_amdgcn_permlane32_swap(eu[0], fu[0], false, false);
                const auto y = __builtin_amdgcn_permlane32_swap(eu[1], fu[1], false, false);
                if (row_ok) *(uintx4*)(orow + db * 32 + 8 * (g + lh)) = uintx4{x[0], y[0], x[1], y[1]};
            }
    }
}

int launch_attention(const half_t* qkv, const int32_t* valid_len, int B, int S, int heads, half_t* out, int hp,
                     hipStream_t stream) {
    if (!qkv || !valid_len || !out || B <= 0 || heads <= 0) { set_error("attention: invalid arguments"); return -1; }
    if (S <= 0 || S > 256) { set_error("attention: sequence length %d must be in 1..256", S); return -5; }
    if ((long long)B * heads > 0x3fffffffLL || 8LL * heads * (3 * ATT_D * 2) > 0x7fffffffLL) { set_error("attention: grid or row too large"); return -5; }
    // More than 4 query blocks: two workgroups with one block per wavefront each as long as all of them are on the chip at once (3 of
    // 197 keys per compute unit): 32 x 12 heads 12.7 us against 15.4 with two blocks per wavefront.  Beyond that K and V are better read
    // once (64 x 12: 25.4 against 23.8).
    const int seq_heads = B * heads, nq = (S + 31) / 32;
    const int parts = nq > ATT_WAVES && 2LL * seq_heads <= 768 ? 2 : 1;
    const size_t lds = (size_t)((S + 15) / 16 * 16) * 2 * ATT_ROW;      // at most 64 KB
    hipLaunchKernelGGL(attention_kernel, dim3((unsigned)(seq_heads * parts)), dim3(64 * ATT_WAVES), lds, stream, qkv, valid_len, S, heads, seq_heads,
                       (nq + parts - 1) / parts, out, hp, divisor(heads));
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) { set_error("attention launch: %s", hipGetErrorString(e)); return -2; }
    return 0;
}

}  // namespace strait
