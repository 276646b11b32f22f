// Dense products with a LayerNorm folded in, for the token sequences of the encoder and the Vision Transformer (paper Section 3.2 step (2)).
//
// A LayerNorm of its own reads and writes the whole activation (25 MB for 64 sequences of 128 tokens) and is a launch in a chain of dependent ones;
// at a server's batch sizes the launch is all of its time (5 us of it at 1024 rows, 7.5 at 8192, 10 to 12 at 12608).  conv_dma.hpp (LN) says how the
// products before and after it take its work over.  What that costs them, us a launch, each kernel by itself, plain -> folded into the input (to 2304
// and, with GELU, to 3072 channels) or with statistics and a normalised residual (from 768 and from 3072): 1024 rows 9.3 -> 10.2, 11.8 -> 12.4, 6.3 -> 7.2,
// 12.9 -> 13.8; 8192 rows 40 -> 42.8, 55 -> 59, 17.2 -> 19.7, 45 -> 49.  Encoder batch 8 836 -> 730 us, ViT batch 7 1001 -> 918; 2 x batch 64
// 5257 -> 5105, ViT batch 64 3769 -> 3612 (1 % of each the GELU).
#include <algorithm>

#include "conv_dma.hpp"

namespace strait {

// LDS of a workgroup on a tile; parts: the groups of 64 channels that a row's statistics come in
template <int BM, int BN, int STAGES, int KG>
constexpr unsigned ln_tile_lds(int ln, int parts) {
    constexpr unsigned ring = KG * STAGES * (BM + BN) * 64 * 2, ctile = BM * (BN + 8) * 2, ftile = f32_stage_rows<BM, BN>() * (BN + 4) * 4;
    const unsigned park = ln == LN_IN ? ctile : ftile;
    return (ring > park ? ring : park) + 1024 + (ln == LN_IN ? ln_lds_bytes<BM, LN_IN>(parts) : ln == LN_RES ? ln_lds_bytes<BM, LN_RES>(parts) : 0u);
}

template <int BM, int BN, int WGM, int WGN, int STAGES, int KG = 1>
static int launch_ln_tile(const ConvParams& p, hipStream_t stream) {
    constexpr int BK = 64;
    const long long tiles_m = (p.M + BM - 1) / BM;
    const int tiles_n = (p.Cout + BN - 1) / BN;
    const long long tiles = tiles_m * tiles_n;
    if (tiles <= 0 || tiles > 0x7fffffffLL) { set_error("gemm with LayerNorm: bad grid (%lld tiles)", tiles); return -5; }
    constexpr int most = BN == 256 ? LN_MAX_PARTS_256 : LN_MAX_PARTS;
    static_assert(ln_tile_lds<BM, BN, STAGES, KG>(LN_IN, most) <= 160 * 1024 && ln_tile_lds<BM, BN, STAGES, KG>(LN_RES, most) <= 160 * 1024, "LDS limit");
    const unsigned in = ln_tile_lds<BM, BN, STAGES, KG>(LN_IN, p.Kg / 64), res = ln_tile_lds<BM, BN, STAGES, KG>(LN_RES, p.Cout / 64), out = ln_tile_lds<BM, BN, STAGES, KG>(LN_OUT, 0);
    ConvParams q = p;
    set_tile_order(q, tiles_m, tiles_n, BM, BN, BK, KG);
    // (160 KB are asked for once, for all widths of a LayerNorm)
#define STRAIT_GO(lds, ...) launch_with_lds<conv_igemm_dma_kernel<__VA_ARGS__>>(q, dim3((unsigned)tiles), dim3(64 * WGM * WGN * KG), lds, 160 * 1024, stream)
    int rc;
    if (!p.stats_out) {
        if (p.act == ACT_GELU) {
            if constexpr (KG == 1) rc = STRAIT_GO(in, BM, BN, BK, WGM, WGN, MODE_1X1, STAGES, true, RES_LATE, false, 1, LN_IN);
            else { set_error("gemm with LayerNorm: no GELU on this tile"); return -5; }
        } else rc = STRAIT_GO(in, BM, BN, BK, WGM, WGN, MODE_1X1, STAGES, false, RES_LATE, false, KG, LN_IN);
    } else if (p.ln_stats) {
        rc = STRAIT_GO(res, BM, BN, BK, WGM, WGN, MODE_1X1, STAGES, false, RES_F32, false, KG, LN_RES);
    } else {
        rc = STRAIT_GO(out, BM, BN, BK, WGM, WGN, MODE_1X1, STAGES, false, RES_F32, false, KG, LN_OUT);
    }
#undef STRAIT_GO
    if (rc) return rc;
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) { set_error("gemm with LayerNorm launch: %s", hipGetErrorString(e)); return -2; }
    return 0;
}

bool gemm_ln_supported(long long M, long long N, long long K, int width) {
    return M > 0 && N > 0 && K > 0 && width > 0 && width % 64 == 0 && width / 64 <= LN_MAX_PARTS && N % 64 == 0 && K % 64 == 0 && M * K * 2 <= 0x7fffffffLL &&
           N * K * 2 <= 0x7fffffffLL && M * width / 8 <= 0x7fffffffLL;
}

// Whole passes of three encoder layers, folded against LayerNorm launches of their own.  Above 768 channels the statistics leave no room for the largest tiles and for
// pairs of 128 x 128: 832 to 1024 channels 0.88 to 0.97 of the time at 512 to 2048 rows, 0.94 to 0.98 at 3072, at 4096 0.96 with 832 and 0.98 to 1.03 above, 0.98 to
// 1.07 at 5000 to 6400, 1.05 to 1.09 at 16384; up to 768 channels 0.84 to 1.00 everywhere.  Up to 64 rows the products go to kernels that take no LayerNorm in, and a row of whole
// chunks for 64 lanes is the LayerNorm kernel's fastest form: 512 channels 1.02 to 1.06, 1024 0.98 to 1.02; others 0.89 to 1.02.
bool gemm_ln_pays(long long rows, int width) {
    return rows <= 64 ? width % 512 != 0 : width <= 64 * LN_MAX_PARTS_256 || rows <= (width <= 832 ? 4096 : 3072);
}

int launch_gemm_ln(const ConvParams& params, hipStream_t stream) {
    ConvParams p = params;
    const bool in = p.ln_stats && p.ln_csum, res = p.ln_stats && p.ln_g && p.ln_b;
    if (!gemm_ln_supported(p.M, p.Cout, p.Kg, in ? p.Kg : p.Cout) || p.out_f32 || p.ldy != p.Cout || p.sW != p.Kg || (p.y_sliced && p.stats_out) ||
        (p.stats_out ? !p.res || p.act != ACT_NONE || in || (p.ln_stats && !res) : !in || p.res || (p.act != ACT_NONE && p.act != ACT_GELU))) {
        set_error("gemm with LayerNorm: unsupported combination (%d x %d x %d)", p.M, p.Cout, p.Kg); return -5;
    }
    if ((reinterpret_cast<uintptr_t>(p.ln_stats) | reinterpret_cast<uintptr_t>(p.stats_out)) & 15) { set_error("gemm with LayerNorm: statistics must be 16-byte aligned"); return -1; }
    p.ln_inv_n = 1.f / (float)(in ? p.Kg : p.Cout);
    const int id = choose_gemm_ln(p);
    if (id < 0) return id;
    p.x_slice = p.x_sliced ? (unsigned)p.M * 128u : 128u;
    if (p.x_sliced) p.sW = 64;
    switch (id) {
        case T256x256: return launch_ln_tile<256, 256, 2, 4, 2>(p, stream);
        case T256x192: return launch_ln_tile<256, 192, 4, 2, 2>(p, stream);
        case T192x128: return launch_ln_tile<192, 128, 2, 4, 3>(p, stream);
        case T128x256: return launch_ln_tile<128, 256, 2, 4, 3>(p, stream);
        case T128x128: return launch_ln_tile<128, 128, 4, 2, 4>(p, stream);
        case T128x128_2: return launch_ln_tile<128, 128, 2, 2, 2>(p, stream);
        case T96x128: return launch_ln_tile<96, 128, 1, 4, 4>(p, stream);
        case T64x128: return launch_ln_tile<64, 128, 2, 2, 3>(p, stream);
        case T128x64: return launch_ln_tile<128, 64, 4, 2, 5>(p, stream);
        case T64x64: return launch_ln_tile<64, 64, 2, 2, 3>(p, stream);
        case T32x64: return launch_ln_tile<32, 64, 1, 2, 4>(p, stream);
        case T64x64_g2: return launch_ln_tile<64, 64, 2, 2, 3, 2>(p, stream);
        case T32x64_g4: return launch_ln_tile<32, 64, 1, 2, 3, 4>(p, stream);
        default: set_error("gemm with LayerNorm: no such tile"); return -5;
    }
}

bool gemm_ln_two_fit(int id, const ConvParams& p) {
    const int ln = !p.stats_out ? LN_IN : p.ln_stats ? LN_RES : LN_OUT, parts = (ln == LN_IN ? p.Kg : p.Cout) / 64;
    switch (id) {
        case T128x128_2: return 2 * ln_tile_lds<128, 128, 2, 1>(ln, parts) <= 160 * 1024;
        case T64x128: return 2 * ln_tile_lds<64, 128, 3, 1>(ln, parts) <= 160 * 1024;
        case T64x64: return 2 * ln_tile_lds<64, 64, 3, 1>(ln, parts) <= 160 * 1024;
        case T32x64: return 2 * ln_tile_lds<32, 64, 4, 1>(ln, parts) <= 160 * 1024;
        default: return false;
    }
}

// One wavefront per row of w.  `bad` becomes 1 where a row of w gamma has lost more to its rounding than fp16 takes from ordinary numbers, 2^-11 of each: a
// row that mostly lies below fp16's normal range (6e-5), or a product beyond its largest number.
__global__ void __launch_bounds__(256) fold_layernorm_kernel(const half_t* __restrict__ w, const float* __restrict__ b, const float* __restrict__ gamma,
                                                             const float* __restrict__ beta, int N, int K, half_t* __restrict__ w_out,
                                                             float* __restrict__ csum, float* __restrict__ b_out, int* __restrict__ bad) {
    const int n = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (n >= N) return;
    float s = 0.f, t = 0.f, lost = 0.f, all = 0.f;
    for (int k = lane; k < K; k += 64) {
        const float v = (float)w[(long long)n * K + k];
        const float vg = v * gamma[k];
        const half_t h = (half_t)vg;
        const float d = ((float)h - vg) * 2048.f;
        w_out[(long long)n * K + k] = h;
        s += (float)h;
        t += v * beta[k];
        lost += d * d;
        all += vg * vg;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        s += __shfl_xor(s, o, 64); t += __shfl_xor(t, o, 64);
        lost += __shfl_xor(lost, o, 64); all += __shfl_xor(all, o, 64);
    }
    if (lane == 0) {
        csum[n] = s; b_out[n] = b[n] + t;
        if (bad && !(lost <= all)) *bad = 1;           // (also where one of them is not a number)
    }
}

int launch_fold_layernorm(const half_t* w, const float* b, const float* gamma, const float* beta, int N, int K, half_t* w_out, float* csum, float* b_out,
                          int* bad, hipStream_t stream) {
    if (!w || !b || !gamma || !beta || !w_out || !csum || !b_out || N <= 0 || K <= 0) { set_error("fold_layernorm: invalid arguments"); return -1; }
    hipLaunchKernelGGL(fold_layernorm_kernel, dim3((N + 3) / 4), dim3(256), 0, stream, w, b, gamma, beta, N, K, w_out, csum, b_out, bad);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) { set_error("fold_layernorm launch: %s", hipGetErrorString(e)); return -2; }
    return 0;
}

}  // namespace strait
