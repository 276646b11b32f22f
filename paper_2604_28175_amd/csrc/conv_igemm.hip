// Implicit-GEMM convolution / GEMM on fp16 MFMA for gfx950 (CDNA4), NHWC activations.
//
// Computes the convolution layers (and, with R = S = 1, the linear layers) of a served batch's
// kernel sequence (paper Section 3.2, step (2)):
//     y[m, k] = act(bias[k] + sum_{r,s,c} x[n, p*stride+r-pad, q*stride+s-pad, c] * w[k, r, s, c] (+ res[m, k]))
// with m = (n, p, q) running over output pixels.
//
// Mapping to the machine
//   - a workgroup of 4 wavefronts (2 x 2) owns a BM-pixel x BN-channel output tile and walks the
//     reduction (r, s, c) in slices of BK = 32;
//   - each slice of the gathered input ("X", BM x 32) and of the weights ("W", BN x 32) is staged
//     in LDS with an 80-byte row pitch, which makes the 16-byte MFMA operand reads conflict free;
//     the next slice is fetched from global memory into registers while the current one feeds
//     v_mfma_f32_32x32x16_f16, and two LDS buffers alternate so one barrier per slice suffices;
//   - the weights are the MFMA "A" operand (rows = channels) and the pixels the "B" operand
//     (columns), so a lane ends up holding 4 consecutive channels of one pixel per accumulator
//     quad: the epilogue adds the bias, rounds to fp16, parks the tile in LDS as [pixel][channel]
//     and writes it out (adding the residual, applying the activation) as 16-byte row segments;
//   - workgroup ids are re-ordered so that tiles sharing an input slice run on the same XCD
//     (consecutive hardware ids are dealt round-robin over the 8 XCDs, each with its own L2).
#include <algorithm>
#include <atomic>
#include <cmath>
#include <type_traits>

#include "conv_dma.hpp"

namespace strait {


template <int BM, int BN, int MODE, bool STAGED>
__global__ void __launch_bounds__(256) conv_igemm_kernel(const ConvParams p) {
    constexpr int BK = 32, LDK = BK + 8;
    constexpr int TM = BM / 2, TN = BN / 2;          // wave tile
    constexpr int TMB = TM / 32, TNB = TN / 32;      // 32x32 MFMA blocks per wave tile
    constexpr int XC = BM * 4 / 256, WC = BN * 4 / 256;   // 16-byte chunks per thread per slice
    constexpr int LDC = BN + 8;
    static_assert(XC >= 1 && WC >= 1, "tile too small for 256 threads");
    static_assert(2 * (BM + BN) * LDK >= BM * LDC, "epilogue tile must fit in the pipeline buffers");

    __shared__ __attribute__((aligned(16))) half_t smem[2 * (BM + BN) * LDK];
    half_t* Xs = smem;                       // [2][BM][LDK]
    half_t* Ws = smem + 2 * BM * LDK;        // [2][BN][LDK]

    if (p.hp) __builtin_amdgcn_s_setprio(3);

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int wm0 = (wave & 1) * TM, wn0 = (wave >> 1) * TN;
    const int l32 = lane & 31, lh = lane >> 5;

    // XCD-aware tile order: hardware workgroup id b runs on XCD b % 8.
    const int tiles_n = (p.Cout + BN - 1) / BN;
    int logical;
    {
        const int nb = gridDim.x, b = blockIdx.x;
        const int per = nb >> 3, rem = nb & 7, xcd = b & 7, idx = b >> 3;
        logical = (xcd < rem ? xcd * (per + 1) : rem * (per + 1) + (xcd - rem) * per) + idx;
    }
    const int m0 = (logical / tiles_n) * BM;
    const int n0 = (logical % tiles_n) * BN;

    // ---- per-thread gather state ------------------------------------------------------
    const int ch = tid & 3;                  // which 8-element chunk of the 32-wide slice
    long long xbase[XC];
    int ih0[XC], iw0[XC];
    bool mval[XC];
#pragma unroll
    for (int i = 0; i < XC; ++i) {
        const int row = (tid >> 2) + i * 64;
        const int m = m0 + row;
        mval[i] = m < p.M;
        const int mm = mval[i] ? m : 0;
        if (MODE == MODE_1X1 && p.stride_h == 1) {
            xbase[i] = (long long)mm * p.sW;     // dense [M][C] matrix (sW == row pitch)
            ih0[i] = iw0[i] = 0;
        } else {
            const int n = mm / p.PQ, rem = mm - n * p.PQ;
            const int pp = rem / p.Q, qq = rem - pp * p.Q;
            ih0[i] = pp * p.stride_h - p.pad_h;
            iw0[i] = qq * p.stride_w - p.pad_w;
            xbase[i] = (long long)n * p.sN + (long long)ih0[i] * p.sH + (long long)iw0[i] * p.sW;
        }
    }
    int k0 = ch * 8;                         // this thread's k index within the reduction
    int r = 0, s = 0, c0 = k0;               // MODE_GATHER8: (r, s, c0) of k0
    if (MODE == MODE_GATHER8) {
        while (c0 >= p.C) { c0 -= p.C; if (++s == p.S) { s = 0; ++r; } }
    }
    bool wval[WC];
    const half_t* wptr[WC];
#pragma unroll
    for (int i = 0; i < WC; ++i) {
        const int row = (tid >> 2) + i * 64;
        wval[i] = (n0 + row) < p.Cout;
        wptr[i] = p.w + (long long)(wval[i] ? n0 + row : 0) * p.ldw + ch * 8;
    }

    const int nk = (p.Kg + BK - 1) / BK;
    uint4 xr[XC], wr[WC];

    auto fetch = [&](int kt) {
        const bool kval = k0 < p.Kg;
#pragma unroll
        for (int i = 0; i < WC; ++i) {
            // weight rows are zero padded up to ldw (a multiple of 8), so a chunk that starts
            // below ldw is entirely readable
            wr[i] = (wval[i] && (kt * BK + ch * 8) < p.ldw) ? *(const uint4*)(wptr[i] + kt * BK) : make_uint4(0, 0, 0, 0);
        }
        if (MODE == MODE_1X1) {
#pragma unroll
            for (int i = 0; i < XC; ++i)
                xr[i] = (mval[i] && kval) ? *(const uint4*)(p.x + xbase[i] + k0) : make_uint4(0, 0, 0, 0);
        } else if (MODE == MODE_GATHER8) {
            const int koff = r * p.sH + s * p.sW + c0;
#pragma unroll
            for (int i = 0; i < XC; ++i) {
                const bool ok = mval[i] && kval && (unsigned)(ih0[i] + r) < (unsigned)p.H &&
                                (unsigned)(iw0[i] + s) < (unsigned)p.W;
                xr[i] = ok ? *(const uint4*)(p.x + xbase[i] + koff) : make_uint4(0, 0, 0, 0);
            }
        } else {
#pragma unroll
            for (int i = 0; i < XC; ++i) {
                half8 v;
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const int k = k0 + j;
                    const int rs = k / p.C, c = k - rs * p.C;
                    const int rr = rs / p.S, ss = rs - rr * p.S;
                    const bool ok = mval[i] && k < p.Kg && (unsigned)(ih0[i] + rr) < (unsigned)p.H &&
                                    (unsigned)(iw0[i] + ss) < (unsigned)p.W;
                    v[j] = ok ? p.x[xbase[i] + (long long)rr * p.sH + (long long)ss * p.sW + c] : (half_t)0;
                }
                xr[i] = *(uint4*)&v;
            }
        }
        // advance to the next slice
        k0 += BK;
        if (MODE == MODE_GATHER8) {
            c0 += BK;
            while (c0 >= p.C) { c0 -= p.C; if (++s == p.S) { s = 0; ++r; } }
        }
    };
    auto stash = [&](int buf) {
#pragma unroll
        for (int i = 0; i < XC; ++i)
            *(uint4*)(Xs + (buf * BM + (tid >> 2) + i * 64) * LDK + ch * 8) = xr[i];
#pragma unroll
        for (int i = 0; i < WC; ++i)
            *(uint4*)(Ws + (buf * BN + (tid >> 2) + i * 64) * LDK + ch * 8) = wr[i];
    };

    floatx16 acc[TNB][TMB];
#pragma unroll
    for (int a = 0; a < TNB; ++a)
#pragma unroll
        for (int b = 0; b < TMB; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.f;

    fetch(0);
    stash(0);
    __syncthreads();

    for (int kt = 0; kt < nk; ++kt) {
        const int buf = kt & 1;
        if (kt + 1 < nk) fetch(kt + 1);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            half8 wf[TNB], xf[TMB];
#pragma unroll
            for (int a = 0; a < TNB; ++a)
                wf[a] = *(const half8*)(Ws + (buf * BN + wn0 + a * 32 + l32) * LDK + ks * 16 + lh * 8);
#pragma unroll
            for (int b = 0; b < TMB; ++b)
                xf[b] = *(const half8*)(Xs + (buf * BM + wm0 + b * 32 + l32) * LDK + ks * 16 + lh * 8);
#pragma unroll
            for (int a = 0; a < TNB; ++a)
#pragma unroll
                for (int b = 0; b < TMB; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(wf[a], xf[b], acc[a][b], 0, 0, 0);
        }
        if (kt + 1 < nk) stash(buf ^ 1);
        __syncthreads();
    }

    // ---- epilogue ---------------------------------------------------------------------
    // lane holds, for accumulator (a, b) and quad g: pixel wm0 + b*32 + l32,
    // channels wn0 + a*32 + 8g + 4*lh + {0,1,2,3}
    if (STAGED) {
        half_t* Cs = smem;                   // [BM][LDC]; all waves are past the last barrier
        const bool fuse_act = (p.res == nullptr);
#pragma unroll
        for (int a = 0; a < TNB; ++a)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int cl = wn0 + a * 32 + 8 * g + 4 * lh;
                float bv[4];
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    bv[j] = (p.bias && (n0 + cl + j) < p.Cout) ? p.bias[n0 + cl + j] : 0.f;
#pragma unroll
                for (int b = 0; b < TMB; ++b) {
                    half4 h;
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        float v = acc[a][b][4 * g + j] + bv[j];
                        if (fuse_act) v = apply_act(v, p.act);
                        h[j] = (half_t)v;
                    }
                    *(half4*)(Cs + (wm0 + b * 32 + l32) * LDC + cl) = h;
                }
            }
        __syncthreads();
        constexpr int CPR = BN / 8;          // 16-byte chunks per tile row
#pragma unroll
        for (int i = 0; i < BM * CPR / 256; ++i) {
            const int id = tid + i * 256;
            const int row = id / CPR, c8 = id - row * CPR;
            const int m = m0 + row, n = n0 + c8 * 8;
            if (m < p.M && n < p.Cout) {
                half8 v = *(const half8*)(Cs + row * LDC + c8 * 8);
                if (!fuse_act) {
                    const half8 rv = *(const half8*)(p.res + (long long)m * p.ldy + n);
#pragma unroll
                    for (int j = 0; j < 8; ++j) v[j] = (half_t)apply_act((float)v[j] + (float)rv[j], p.act);
                }
                *(half8*)((half_t*)p.y + (long long)m * p.ldy + n) = v;
            }
        }
    } else {
#pragma unroll
        for (int a = 0; a < TNB; ++a)
#pragma unroll
            for (int b = 0; b < TMB; ++b) {
                const int m = m0 + wm0 + b * 32 + l32;
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int n = n0 + wn0 + a * 32 + 8 * (v >> 2) + 4 * lh + (v & 3);
                    if (m < p.M && n < p.Cout) {
                        float val = acc[a][b][v] + (p.bias ? p.bias[n] : 0.f);
                        if (p.res) val += (float)p.res[(long long)m * p.ldy + n];
                        val = apply_act(val, p.act);
                        if (p.out_f32) ((float*)p.y)[(long long)m * p.ldy + n] = val;
                        else ((half_t*)p.y)[(long long)m * p.ldy + n] = (half_t)val;
                    }
                }
            }
    }
}


// Second pass of a split-K launch: y = act(sum_z slab_z + bias (+ res)), 8 channels per thread,
// slabs summed in a fixed order so that results do not depend on scheduling.
__global__ void __launch_bounds__(256) splitk_finish_kernel(const ConvParams p) {
    if (p.hp) __builtin_amdgcn_s_setprio(3);
    const int c8n = p.Cout >> 3;
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i >= (long long)p.M * c8n) return;
    const int m = (int)(i / c8n), n = (int)(i - (long long)m * c8n) * 8;
    float v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = p.bias ? p.bias[n + j] : 0.f;
    const long long slab = (long long)p.M * p.Cout;
    const float* src = p.ws + (long long)m * p.Cout + n;
    // The slabs are fetched several at a time and added in slab order: one load per trip of a loop whose length the
    // compiler does not know costs a trip to L2 per slab (a 32-way split: 11 us for this kernel against 4).
    auto add_slabs = [&](int z0, auto nconst) {
        constexpr int NB = decltype(nconst)::value;
        float4 lo[NB], hi[NB];
#pragma unroll
        for (int u = 0; u < NB; ++u) { lo[u] = *(const float4*)(src + (z0 + u) * slab); hi[u] = *(const float4*)(src + (z0 + u) * slab + 4); }
#pragma unroll
        for (int u = 0; u < NB; ++u) { v[0] += lo[u].x; v[1] += lo[u].y; v[2] += lo[u].z; v[3] += lo[u].w; v[4] += hi[u].x; v[5] += hi[u].y; v[6] += hi[u].z; v[7] += hi[u].w; }
    };
    int z = 0;
    for (; z + 8 <= p.ksplit; z += 8) add_slabs(z, std::integral_constant<int, 8>());
    if (z + 4 <= p.ksplit) { add_slabs(z, std::integral_constant<int, 4>()); z += 4; }
    if (z + 2 <= p.ksplit) { add_slabs(z, std::integral_constant<int, 2>()); z += 2; }
    if (z < p.ksplit) add_slabs(z, std::integral_constant<int, 1>());
    if (p.res) {
        const half8 r = *(const half8*)(p.res + (long long)m * p.ldy + n);
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] += (float)r[j];
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = apply_act(v[j], p.act);
    if (p.out_f32) {
        float* dst = (float*)p.y + (long long)m * p.ldy + n;
        *(float4*)dst = make_float4(v[0], v[1], v[2], v[3]);
        *(float4*)(dst + 4) = make_float4(v[4], v[5], v[6], v[7]);
    } else {
        half8 o;
#pragma unroll
        for (int j = 0; j < 8; ++j) o[j] = (half_t)v[j];
        *(half8*)((half_t*)p.y + (long long)m * p.ldy + n) = o;
    }
}

// ------------------------------------------------------------------------------------------
// 3x3, stride 1, padding 1, from an input patch held in LDS.
//
// conv_igemm_dma_kernel (conv_dma.hpp) fetches every input pixel nine times, once per filter tap; on the wide early layers that
// traffic between L2 and LDS, not the MFMAs, sets the pace.  Here pixels are numbered in a bordered space: every
// image row is preceded by one border slot and every image by one border row, v = (n (H+1) + y) (W+1) + x for
// output (n, y, x), and the slot with number u holds input pixel (u's row - 1, u's column - 1) or, in the border,
// zero.  A row's right border is the next row's left border and an image's bottom border row the next image's top
// one, so one slot per row and one row per image suffice.  Tap (r, s) of output v then reads slot
// v + r (W+1) + s: one offset per tap for the whole tile.  A workgroup owns BM consecutive v (the one in W+1 with
// x = W and the one row in H+1 with y = H are computed and never stored) and BN output channels.  Per
// 32-channel slice of the input it holds the BM + 2 (W+1) + 2 slots its taps touch (64 bytes each; border slots
// arrive as zeros from out-of-range transfers) and feeds all nine taps' MFMAs from them; only the weights, one
// 32-channel slice of one tap at a time, stream through a three-stage ring.  The patch of the next slice arrives
// in a second buffer during the first seven tap steps of the current one.  Per tap step every wave issues a
// fixed number of transfers, so the in-order load counter tells when a given stage has landed.  LDS rows of 64
// bytes are swizzled as there (16-byte chunk c of row i sits at c ^ ((i >> 2) & 3)), which keeps
// the operand reads conflict free for any run of consecutive rows, i.e. for every tap offset.
template <int BM, int BN, int WGM, int WGN, int NPW, int NBS>
__global__ void __launch_bounds__(64 * WGM * WGN, WGM * WGN / 2) conv3x3_patch_kernel(const ConvParams p) {
    constexpr int NW = WGM * WGN, NT = 64 * NW;
    static_assert((NW == 4 || NW == 8) && BM % (32 * WGM) == 0 && BN % (32 * WGN) == 0 && BN % (16 * NW) == 0, "unsupported tile");
    constexpr int TM = BM / WGM, TN = BN / WGN, TMB = TM / 32, TNB = TN / 32;
    constexpr int WI = BN / (NW * 16);                 // weight transfers per wave per tap step
    constexpr int PRE = NBS - 1;                       // weight stages in flight ahead of the one in use
    constexpr int AS = (NPW + 8 - PRE) / (9 - PRE);    // patch transfers per wave per tap step (steps 0..8-PRE)
    static_assert(NBS >= 3 && NBS <= 8, "ring depth");
    constexpr int PATCH = NPW * NW * 1024;             // bytes of one patch buffer: NPW * 64 pixels
    constexpr int WSTAGE = BN * 64;                    // bytes of one weight stage
    constexpr int RING = 2 * PATCH + NBS * WSTAGE;
    constexpr int LDC = BN + 8;
    constexpr int CT = BM * LDC * 2;
    constexpr unsigned BIAS_LDS = RING > CT ? RING : CT;
    static_assert(BIAS_LDS + 1024 <= 160 * 1024, "LDS limit");

    extern __shared__ __attribute__((aligned(1024))) half_t smem[];
    const unsigned lds0 = (unsigned)(uintptr_t)smem;
    if (p.hp) __builtin_amdgcn_s_setprio(3);

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm0 = (wave % WGM) * TM, wn0 = (wave / WGM) * TN;
    const int l32 = lane & 31, lh = lane >> 5;

    const int tile = xcd_range(p.order.tiles, blockIdx.x), tm = divide(tile, p.order.by_cw);
    const int m0 = tm * BM, n0 = (tile - tm * p.order.cw) * BN;

    // rows wider than 64 pixels are cut into strips, each numbered as an image of its own with a border slot on
    // either side that holds the neighbouring strip's pixel (zero only at the true edges), so those are not shared
    const int SW = p.strip_w, NS = p.strips, Wp = SW + (NS == 1 ? 1 : 2), NI = divide(p.M, p.by_pq) * NS;   // borders shared between neighbours
    const intx4 xrsrc = make_rsrc(p.x, (unsigned)(p.x_elems * 2));
    const intx4 wrsrc = make_rsrc(p.w, (unsigned)((long long)p.Cout * p.ldw * 2));

    // ---- per-lane source offsets: patch pixel (16 per transfer, 4 chunks each), weight row ----------
    unsigned aoff[NPW];
#pragma unroll
    for (int j = 0; j < NPW; ++j) {
        const int pp = (j * NW + wave) * 16 + (lane >> 2);
        int img, yp, xp;
        bordered_place(p, m0 + pp, Wp, img, yp, xp);
        const int n = divide(img, p.by_strips), st = img - n * NS;
        const int xr = st * SW + xp - 1;
        const int lc = (lane & 3) ^ ((pp >> 2) & 3);
        const bool inside = img < NI && yp >= 1 && yp <= p.H && xr >= 0 && xr < p.W;
        aoff[j] = inside ? (unsigned)(((long long)n * p.sN + (long long)(yp - 1) * p.sH + (long long)xr * p.sW + lc * 8) * 2) : OOB_OFFSET;
    }
    unsigned woff[WI];
#pragma unroll
    for (int j = 0; j < WI; ++j) {
        const int row = (j * NW + wave) * 16 + (lane >> 2);
        const int lc = (lane & 3) ^ ((row >> 2) & 3);
        woff[j] = n0 + row < p.Cout ? (unsigned)(((long long)(n0 + row) * p.ldw + lc * 8) * 2) : OOB_OFFSET;
    }
    const int ncs = p.C >> 5;
    auto issue_w = [&](int stage, int tap, int cs) {
        const bool live = cs < ncs;
        const unsigned soff = live ? (unsigned)(tap * p.C + cs * 32) * 2u : 0u;
#pragma unroll
        for (int j = 0; j < WI; ++j)
            dma16(wrsrc, live ? woff[j] : OOB_OFFSET, soff, lds0 + (unsigned)(2 * PATCH + stage * WSTAGE + (j * NW + wave) * 1024));
    };
    auto issue_a = [&](int buf, int j, int cs) {
        const bool live = cs < ncs;
        dma16(xrsrc, live ? aoff[j] : OOB_OFFSET, live ? (unsigned)cs * 64u : 0u, lds0 + (unsigned)(buf * PATCH + (j * NW + wave) * 1024));
    };

    floatx16 acc[TNB][TMB];
#pragma unroll
    for (int a = 0; a < TNB; ++a)
#pragma unroll
        for (int b = 0; b < TMB; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.f;

    static_assert(BN <= 256, "bias row: one transfer carries 256 floats");
    if (wave == 0) {
        const intx4 brsrc = make_rsrc(p.bias, p.bias ? (unsigned)p.Cout * 4u : 0u);
        const int c = n0 + lane * 4;
        dma16(brsrc, (p.bias && lane * 4 < BN && c + 3 < p.Cout) ? (unsigned)c * 4u : OOB_OFFSET, 0u, lds0 + BIAS_LDS);
    }
#pragma unroll
    for (int j = 0; j < NPW; ++j) issue_a(0, j, 0);
#pragma unroll
    for (int t = 0; t < PRE; ++t) issue_w(t, t, 0);    // PRE < 9: all in the first slice
    int rd = 0, wr = PRE;                              // ring stage in use, stage being filled

    const unsigned wrow = (unsigned)((lh ^ ((l32 >> 2) & 3)) << 4);   // chunk lh of weight row l32 (+ multiples of 32 rows)
    for (int cs = 0; cs < ncs; ++cs) {
        const char* Pa = (const char*)smem + (cs & 1) * PATCH;
        const int nbuf = (cs + 1) & 1;
        int wp_l = Wp;                                 // opaque per iteration: keeps the nine taps' operand addresses from being
        asm volatile("" : "+s"(wp_l));                 // hoisted out of the loop, where they would cost eighteen registers
#define STRAIT_TAP_STEP(T)                                                                                              \
        {                                                                                                               \
            wait_loads_then_barrier<patch_wait(NPW, AS, WI, PRE, T)>();                                                  \
            const char* Ws = (const char*)smem + 2 * PATCH + rd * WSTAGE;                                               \
            const int tapoff = (T / 3) * wp_l + (T % 3);                                                                 \
            unsigned a0[TMB];                                                                                           \
            _Pragma("unroll") for (int b = 0; b < TMB; ++b) {                                                           \
                const unsigned pp = (unsigned)(wm0 + b * 32 + l32 + tapoff);                                            \
                a0[b] = pp * 64u + (((lh ^ (pp >> 2)) & 3u) << 4);                                                      \
            }                                                                                                           \
            half8 wf[2][TNB], xf[2][TMB];                                                                               \
            _Pragma("unroll") for (int a = 0; a < TNB; ++a) wf[0][a] = *(const half8*)(Ws + (wn0 + a * 32 + l32) * 64 + wrow); \
            _Pragma("unroll") for (int b = 0; b < TMB; ++b) xf[0][b] = *(const half8*)(Pa + a0[b]);                     \
            issue_w(wr, (T + PRE) % 9, cs + (T + PRE) / 9);                                                             \
            rd = rd + 1 == NBS ? 0 : rd + 1;                                                                            \
            wr = wr + 1 == NBS ? 0 : wr + 1;                                                                            \
            _Pragma("unroll") for (int j = T * AS; j < (T + 1) * AS && j < NPW; ++j) issue_a(nbuf, j, cs + 1);          \
            _Pragma("unroll") for (int a = 0; a < TNB; ++a) wf[1][a] = *(const half8*)(Ws + (((wn0 + a * 32 + l32) * 64 + wrow) ^ 32u)); \
            _Pragma("unroll") for (int b = 0; b < TMB; ++b) xf[1][b] = *(const half8*)(Pa + (a0[b] ^ 32u));             \
            __builtin_amdgcn_sched_barrier(0);                                                                          \
            _Pragma("unroll") for (int ks = 0; ks < 2; ++ks)                                                            \
                _Pragma("unroll") for (int a = 0; a < TNB; ++a)                                                         \
                    _Pragma("unroll") for (int b = 0; b < TMB; ++b)                                                     \
                        acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(wf[ks][a], xf[ks][b], acc[a][b], 0, 0, 0);   \
            __builtin_amdgcn_sched_barrier(0);                                                                          \
        }
        STRAIT_TAP_STEP(0) STRAIT_TAP_STEP(1) STRAIT_TAP_STEP(2) STRAIT_TAP_STEP(3) STRAIT_TAP_STEP(4)
        STRAIT_TAP_STEP(5) STRAIT_TAP_STEP(6) STRAIT_TAP_STEP(7) STRAIT_TAP_STEP(8)
#undef STRAIT_TAP_STEP
    }
    wait_loads_then_barrier<0>();                      // trailing (empty) transfers have landed; LDS is free

    // ---- epilogue: bias, clamp, tile parked in LDS as [pixel][channel], 16-byte row segments out ----
    half_t* Cs = smem;
    const half_t lo = (p.act == ACT_RELU || p.act == ACT_RELU6) ? (half_t)0.f : (half_t)-INFINITY;
    const half_t hi = p.act == ACT_RELU6 ? (half_t)6.f : (half_t)INFINITY;
    const half4 lo4 = {lo, lo, lo, lo}, hi4 = {hi, hi, hi, hi};
    const float* bias_s = (const float*)((const char*)smem + BIAS_LDS);
#pragma unroll
    for (int a = 0; a < TNB; ++a)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int cn = wn0 + a * 32 + 8 * g + 4 * lh;
            const float4 b4 = *(const float4*)(bias_s + cn);
            const float bv[4] = {b4.x, b4.y, b4.z, b4.w};
#pragma unroll
            for (int b = 0; b < TMB; ++b) {
                half4 h;
#pragma unroll
                for (int j = 0; j < 4; ++j) h[j] = (half_t)(acc[a][b][4 * g + j] + bv[j]);
                h = __builtin_elementwise_min(__builtin_elementwise_max(h, lo4), hi4);
                *(half4*)(Cs + (wm0 + b * 32 + l32) * LDC + cn) = h;
            }
        }
    __syncthreads();
    constexpr int CPR = BN / 8, NCH = BM * CPR / NT;
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
        const int id = tid + i * NT;
        const int row = id / CPR, c8 = id - row * CPR;
        int img, yy, xx;
        bordered_place(p, m0 + row, Wp, img, yy, xx);
        const int n = divide(img, p.by_strips), st = img - n * NS;
        if (img < NI && yy < p.H && xx < SW) {
            const half8 v = *(const half8*)(Cs + row * LDC + c8 * 8);
            *(half8*)((half_t*)p.y + ((long long)(n * p.H + yy) * p.W + st * SW + xx) * p.ldy + n0 + c8 * 8) = v;
        }
    }
}

// The same computation for layers whose tiles are short (one to four input slices: the eighteen tap steps of a
// 64-channel layer take about as long as setting a tile up and putting it away).  Half as many workgroups as the
// compute units hold at a time are launched, and each walks over every gridDim.x-th tile: the next tile's first patch
// and first weights arrive during the last slice of the current one, in the buffers that slice no longer reads, and the
// finished tile leaves straight from the accumulators (8 bytes per lane and store), so that no LDS is tied up and no
// barrier separates two tiles.  All output channels in one tile (Cout == BN): weight offsets and the bias row stay put.
// Stores count in the same counter as the transfers.  The waits of the tap steps are not adjusted for them: a wait
// that allows the n newest requests in flight then also waits for stores issued before those, which costs the first
// steps of a tile a little time (counting them in was worth 1 us in 50) and never lets a transfer be read early.
template <int BM, int BN, int WGM, int WGN, int NPW, int NBS>
__global__ void __launch_bounds__(64 * WGM * WGN, WGM * WGN / 2) conv3x3_patch_walk_kernel(const ConvParams p, const int tiles) {
    constexpr int NW = WGM * WGN;
    static_assert((NW == 4 || NW == 8) && BM % (32 * WGM) == 0 && BN % (32 * WGN) == 0 && BN % (16 * NW) == 0, "unsupported tile");
    constexpr int TM = BM / WGM, TN = BN / WGN, TMB = TM / 32, TNB = TN / 32;
    constexpr int WI = BN / (NW * 16);
    constexpr int PRE = NBS - 1;
    constexpr int AS = (NPW + 8 - PRE) / (9 - PRE);
    static_assert(NBS >= 3 && NBS <= 8, "ring depth");
    constexpr int PATCH = NPW * NW * 1024;
    constexpr int WSTAGE = BN * 64;
    constexpr int RING = 2 * PATCH + NBS * WSTAGE;
    static_assert(RING + 1024 <= 160 * 1024 && BN <= 256, "LDS limit; one transfer carries the bias row");

    extern __shared__ __attribute__((aligned(1024))) half_t smem[];
    const unsigned lds0 = (unsigned)(uintptr_t)smem;
    if (p.hp) __builtin_amdgcn_s_setprio(3);

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm0 = (wave % WGM) * TM, wn0 = (wave / WGM) * TN;
    const int l32 = lane & 31, lh = lane >> 5;

    const int SW = p.strip_w, NS = p.strips, Wp = SW + (NS == 1 ? 1 : 2), NI = divide(p.M, p.by_pq) * NS;
    const intx4 xrsrc = make_rsrc(p.x, (unsigned)(p.x_elems * 2));
    const intx4 wrsrc = make_rsrc(p.w, (unsigned)((long long)p.Cout * p.ldw * 2));

    // virtual workgroup v -> tile: the hardware deals consecutive workgroups to the eight XCDs in turn, and gridDim.x is a
    // multiple of eight, so v mod 8 is this workgroup's XCD for every v it takes; each XCD gets a contiguous range of tiles
    auto tile_m0 = [&](int v) __attribute__((always_inline)) -> int {
        const int per = tiles >> 3, rem = tiles & 7, xcd = v & 7, idx = v >> 3;
        return ((xcd < rem ? xcd * (per + 1) : rem * (per + 1) + (xcd - rem) * per) + idx) * BM;
    };
    auto patch_offsets = [&](int m0, bool live, unsigned (&ao)[NPW]) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < NPW; ++j) {
            const int pp = (j * NW + wave) * 16 + (lane >> 2);
            int img, yp, xp;
            bordered_place(p, m0 + pp, Wp, img, yp, xp);
            const int n = divide(img, p.by_strips), st = img - n * NS;
            const int xr = st * SW + xp - 1;
            const int lc = (lane & 3) ^ ((pp >> 2) & 3);
            const bool inside = live && img < NI && yp >= 1 && yp <= p.H && xr >= 0 && xr < p.W;
            ao[j] = inside ? (unsigned)(((long long)n * p.sN + (long long)(yp - 1) * p.sH + (long long)xr * p.sW + lc * 8) * 2) : OOB_OFFSET;
        }
    };
    unsigned woff[WI];
#pragma unroll
    for (int j = 0; j < WI; ++j) {
        const int row = (j * NW + wave) * 16 + (lane >> 2);
        const int lc = (lane & 3) ^ ((row >> 2) & 3);
        woff[j] = row < p.Cout ? (unsigned)(((long long)row * p.ldw + lc * 8) * 2) : OOB_OFFSET;
    }
    const int ncs = p.C >> 5;
    auto issue_w = [&](int stage, int tap, int cs, bool live) __attribute__((always_inline)) {
        const unsigned soff = live ? (unsigned)(tap * p.C + cs * 32) * 2u : 0u;
#pragma unroll
        for (int j = 0; j < WI; ++j)
            dma16(wrsrc, live ? woff[j] : OOB_OFFSET, soff, lds0 + (unsigned)(2 * PATCH + stage * WSTAGE + (j * NW + wave) * 1024));
    };

    floatx16 acc[TNB][TMB];
#pragma unroll
    for (int a = 0; a < TNB; ++a)
#pragma unroll
        for (int b = 0; b < TMB; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.f;

    if (wave == 0) {                                   // the oldest transfer: every later wait covers it
        const intx4 brsrc = make_rsrc(p.bias, p.bias ? (unsigned)p.Cout * 4u : 0u);
        const int c = lane * 4;
        dma16(brsrc, (p.bias && c < BN && c + 3 < p.Cout) ? (unsigned)c * 4u : OOB_OFFSET, 0u, lds0 + RING);
    }
    const int G = (int)gridDim.x;
    int vb = (int)blockIdx.x;
    int m0 = tile_m0(vb);
    unsigned aoff[NPW], anext[NPW];
    patch_offsets(m0, true, aoff);
#pragma unroll
    for (int j = 0; j < NPW; ++j) dma16(xrsrc, aoff[j], 0u, lds0 + (unsigned)((j * NW + wave) * 1024));
#pragma unroll
    for (int t = 0; t < PRE; ++t) issue_w(t, t, 0, true);
    int rd = 0, wr = PRE, par = 0;

    const half_t lo = (p.act == ACT_RELU || p.act == ACT_RELU6) ? (half_t)0.f : (half_t)-INFINITY;
    const half_t hi = p.act == ACT_RELU6 ? (half_t)6.f : (half_t)INFINITY;
    const half4 lo4 = {lo, lo, lo, lo}, hi4 = {hi, hi, hi, hi};
    const float* bias_s = (const float*)((const char*)smem + RING);
    const unsigned wrow = (unsigned)((lh ^ ((l32 >> 2) & 3)) << 4);

    for (;;) {
        const int vnext = vb + G;
        const bool has_next = vnext < tiles;
        const int m0n = has_next ? tile_m0(vnext) : 0;
        patch_offsets(m0n, has_next, anext);
        for (int cs = 0; cs < ncs; ++cs) {
            const bool wrap = cs + 1 == ncs;           // the slice after this one is the next tile's first
            const int csn = wrap ? 0 : cs + 1;
            const bool nlive = !wrap || has_next;
            unsigned asrc[NPW];
#pragma unroll
            for (int j = 0; j < NPW; ++j) asrc[j] = wrap ? anext[j] : aoff[j];
            const char* Pa = (const char*)smem + par * PATCH;
            const unsigned nbuf = lds0 + (unsigned)((par ^ 1) * PATCH);
            int wp_l = Wp;
            asm volatile("" : "+s"(wp_l));
#define STRAIT_WALK_STEP(T)                                                                                             \
            {                                                                                                           \
                wait_loads_then_barrier<patch_wait(NPW, AS, WI, PRE, T)>();                                              \
                const char* Ws = (const char*)smem + 2 * PATCH + rd * WSTAGE;                                           \
                const int tapoff = (T / 3) * wp_l + (T % 3);                                                             \
                unsigned a0[TMB];                                                                                       \
                _Pragma("unroll") for (int b = 0; b < TMB; ++b) {                                                       \
                    const unsigned pp = (unsigned)(wm0 + b * 32 + l32 + tapoff);                                        \
                    a0[b] = pp * 64u + (((lh ^ (pp >> 2)) & 3u) << 4);                                                  \
                }                                                                                                       \
                half8 wf[2][TNB], xf[2][TMB];                                                                           \
                _Pragma("unroll") for (int a = 0; a < TNB; ++a) wf[0][a] = *(const half8*)(Ws + (wn0 + a * 32 + l32) * 64 + wrow); \
                _Pragma("unroll") for (int b = 0; b < TMB; ++b) xf[0][b] = *(const half8*)(Pa + a0[b]);                 \
                if (T + PRE < 9) issue_w(wr, T + PRE, cs, true); else issue_w(wr, T + PRE - 9, csn, nlive);             \
                rd = rd + 1 == NBS ? 0 : rd + 1;                                                                        \
                wr = wr + 1 == NBS ? 0 : wr + 1;                                                                        \
                _Pragma("unroll") for (int j = T * AS; j < (T + 1) * AS && j < NPW; ++j)                                \
                    dma16(xrsrc, asrc[j], (unsigned)csn * 64u, nbuf + (unsigned)((j * NW + wave) * 1024));             \
                _Pragma("unroll") for (int a = 0; a < TNB; ++a) wf[1][a] = *(const half8*)(Ws + (((wn0 + a * 32 + l32) * 64 + wrow) ^ 32u)); \
                _Pragma("unroll") for (int b = 0; b < TMB; ++b) xf[1][b] = *(const half8*)(Pa + (a0[b] ^ 32u));         \
                __builtin_amdgcn_sched_barrier(0);                                                                      \
                _Pragma("unroll") for (int ks = 0; ks < 2; ++ks)                                                        \
                    _Pragma("unroll") for (int a = 0; a < TNB; ++a)                                                     \
                        _Pragma("unroll") for (int b = 0; b < TMB; ++b)                                                 \
                            acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(wf[ks][a], xf[ks][b], acc[a][b], 0, 0, 0); \
                __builtin_amdgcn_sched_barrier(0);                                                                      \
            }
            STRAIT_WALK_STEP(0) STRAIT_WALK_STEP(1) STRAIT_WALK_STEP(2) STRAIT_WALK_STEP(3) STRAIT_WALK_STEP(4)
            STRAIT_WALK_STEP(5) STRAIT_WALK_STEP(6) STRAIT_WALK_STEP(7) STRAIT_WALK_STEP(8)
#undef STRAIT_WALK_STEP
            par ^= 1;
        }
        // ---- the tile leaves from the registers: lane (l32, lh) holds channels 8 g + 4 lh + (0..3) of pixel l32 per 32 x 32 block
        long long ybase[TMB];                          // this lane's pixel in y, in elements; -1: a border slot, nothing to store
#pragma unroll
        for (int b = 0; b < TMB; ++b) {
            int img, yy, xx;
            bordered_place(p, m0 + wm0 + b * 32 + l32, Wp, img, yy, xx);
            const int n = divide(img, p.by_strips), st = img - n * NS;
            ybase[b] = (img < NI && yy < p.H && xx < SW) ? ((long long)(n * p.H + yy) * p.W + st * SW + xx) * p.ldy : -1;
        }
#pragma unroll
        for (int a = 0; a < TNB; ++a)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int cn = wn0 + a * 32 + 8 * g + 4 * lh;
                const float4 b4 = *(const float4*)(bias_s + cn);
                const float bv[4] = {b4.x, b4.y, b4.z, b4.w};
#pragma unroll
                for (int b = 0; b < TMB; ++b) {
                    half4 h;
#pragma unroll
                    for (int j = 0; j < 4; ++j) { h[j] = (half_t)(acc[a][b][4 * g + j] + bv[j]); acc[a][b][4 * g + j] = 0.f; }
                    h = __builtin_elementwise_min(__builtin_elementwise_max(h, lo4), hi4);
                    if (ybase[b] >= 0) *(half4*)((half_t*)p.y + ybase[b] + cn) = h;
                }
            }
        if (!has_next) break;
        vb = vnext;
        m0 = m0n;
#pragma unroll
        for (int j = 0; j < NPW; ++j) aoff[j] = anext[j];
    }
    wait_loads_then_barrier<0>();                      // trailing (empty) transfers have landed
}

template <int BM, int BN, int WGM, int WGN, int NPW, int NBS>
static int launch_patch_walk(const ConvParams& p, long long mv, hipStream_t stream) {
    constexpr int NW = WGM * WGN;
    const long long tiles = (mv + BM - 1) / BM;
    if (p.Cout != BN || tiles < 512 || tiles > 0x7fffffffLL) { set_error("conv: bad grid (%lld tiles)", tiles); return -5; }
    constexpr unsigned lds = 2 * NPW * NW * 1024 + NBS * BN * 64 + 1024;
    static_assert(2 * (lds + 1024) <= 160 * 1024, "two workgroups per compute unit");
    auto kernel = conv3x3_patch_walk_kernel<BM, BN, WGM, WGN, NPW, NBS>;
    static std::atomic<bool> configured{false};
    if (!configured.load(std::memory_order_acquire) && lds > 48 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) { set_error("conv: cannot reserve %u bytes of LDS: %s", lds, hipGetErrorString(e)); return -2; }
    }
    configured.store(true, std::memory_order_release);
    hipLaunchKernelGGL(kernel, dim3(512), dim3(64 * NW), lds, stream, p, (int)tiles);   // two workgroups on each of 256 compute units
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) { set_error("conv launch: %s", hipGetErrorString(e)); return -2; }
    return 0;
}

template <int BM, int BN, int WGM, int WGN, int NPW, int NBS>
static int launch_patch_tile(const ConvParams& p, long long mv, hipStream_t stream) {
    constexpr int NW = WGM * WGN;
    const long long tiles = ((mv + BM - 1) / BM) * (p.Cout / BN);
    if (tiles <= 0 || tiles > 0x7fffffffLL) { set_error("conv: bad grid (%lld tiles)", tiles); return -5; }
    constexpr unsigned ring = 2 * NPW * NW * 1024 + NBS * BN * 64, ctile = BM * (BN + 8) * 2;
    constexpr unsigned lds = (ring > ctile ? ring : ctile) + 1024;
    auto kernel = conv3x3_patch_kernel<BM, BN, WGM, WGN, NPW, NBS>;
    static std::atomic<bool> configured{false};
    if (!configured.load(std::memory_order_acquire) && lds > 48 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) { set_error("conv: cannot reserve %u bytes of LDS: %s", lds, hipGetErrorString(e)); return -2; }
    }
    configured.store(true, std::memory_order_release);
    ConvParams q = p;
    q.order.tiles = (int)tiles; q.order.cw = p.Cout / BN; q.order.by_cw = divisor(q.order.cw);        // (pixel tile by pixel tile)
    hipLaunchKernelGGL(kernel, dim3((unsigned)tiles), dim3(64 * NW), lds, stream, q);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) { set_error("conv launch: %s", hipGetErrorString(e)); return -2; }
    return 0;
}

// ------------------------------------------------------------------------------------------
// Which kernel and tile a layer gets.
//
// Every candidate's time is estimated from the layer's sizes, in microseconds:
//     c0 + c1 R + c2 R nk + c3 R nk [gathered taps] + c4 R [GELU] + c5 MB + c6 max(0, MB - 250)
// with nk the slices of the reduction a workgroup walks through, MB the megabytes of input, weights, residual and output
// (c6: what does not stay in the 256 MB memory-side cache), and R the rounds of tiles a compute unit works off: the tiles
// per unit rounded up where one workgroup fills a unit; where two fit, a pair of tiles counts 1 and an odd one 0.6, since
// alone it gets more than half of the unit.  c0 holds the launch, c1 a tile's start, epilogue and stores, c2 a slice's
// operand traffic and MFMAs.  The coefficients are non-negative least-squares fits (relative error) to measured times, 826
// layer shapes on MI355X: the served networks' layers at batch 1 to 128 and image sides 160 to 256, token products of 32
// to 16384 rows; mean error 5 to 9 %, and the estimated best is on average within 2 % of the measured best candidate.
// The patch kernel's rows and the gathered 256 x 128 x 32 tile's c3 are fits to 240 more 3x3 layers (14 to 224 pixels wide, 32 to 512
// channels in, 40 to 4500 tiles; mean error 3 to 12 %); the choice is then on average 2 % off the best there, before 7 % and up
// to 1.7 times: 16 x 112 x 112, 64 -> 128 53 -> 41 us; 118 x 40 x 40 at stride 2, 160 -> 512 132 -> 83 us.
// The rows of the kernel through registers are fits to 230 layers with fp32 or odd outputs (mean error 17 to 20 %).
// The rows are older than the GELU of activation.hpp and than the operands read ahead on the 96 x 128 and 8-wavefront 128 x 128 tiles: c4 is about a
// quarter too high on tiles that fill a unit, and those two tiles are up to 7 % faster than estimated.
// Against the thresholds used before (and with the pipelined loop): ResNet-50's layers 7 % faster on the sum over batch 1
// to 128 (22 % at batch 1, 5 % at 128), an encoder layer's products 8 to 19 % from 1000 rows on and 20 to 32 % below.
struct TileInfo { int bm, bn, bk, kg; bool shared; float c[7]; };   // shared: two or more workgroups fit a compute unit
static const TileInfo tile_info[T_ESTIMATED] = {
    {256, 256, 64, 1, false, {2.047f, 4.619f, 1.152f, 0.199f, 10.088f, 0.100f, 0.086f}},
    {256, 192, 64, 1, false, {1.482f, 4.048f, 0.952f, 0.175f, 7.991f, 0.100f, 0.108f}},
    {192, 128, 64, 1, false, {0.722f, 3.601f, 0.550f, 0.134f, 3.747f, 0.080f, 0.051f}},
    {128, 256, 64, 1, false, {1.311f, 3.417f, 0.627f, 0.099f, 5.877f, 0.102f, 0.047f}},
    {128, 128, 64, 1, false, {1.037f, 2.932f, 0.404f, 0.085f, 2.509f, 0.076f, 0.048f}},
    {128, 128, 64, 1, true, {2.649f, 2.689f, 0.759f, 0.240f, 3.708f, 0.084f, 0.113f}},
    {96, 128, 64, 1, false, {0.949f, 3.098f, 0.360f, 0.089f, 1.597f, 0.060f, 0.082f}},
    {64, 128, 64, 1, true, {2.205f, 2.481f, 0.490f, 0.086f, 2.066f, 0.050f, 0.144f}},
    {256, 128, 32, 1, true, {2.271f, 3.506f, 0.583f, 0.110f, 10.612f, 0.106f, 0.085f}},
    {128, 64, 32, 1, true, {2.823f, 0.742f, 0.358f, 0.056f, 2.304f, 0.069f, 0.143f}},
    {128, 64, 32, 1, true, {2.525f, 1.151f, 0.308f, 0.071f, 2.345f, 0.070f, 0.103f}},
    {64, 64, 64, 1, true, {2.454f, 1.311f, 0.339f, 0.075f, 0.715f, 0.031f, 0.200f}},
    {64, 64, 32, 1, true, {2.583f, 0.806f, 0.228f, 0.027f, 1.154f, 0.026f, 0.122f}},
    {32, 64, 64, 1, true, {2.712f, 0.950f, 0.272f, 0.069f, 0.342f, 0.032f, 1.280f}},
    {64, 64, 64, 2, false, {1.059f, 2.700f, 0.289f, 0.126f, 0.f, 0.065f, 0.f}},
    {32, 64, 64, 4, false, {1.316f, 2.420f, 0.391f, 0.174f, 0.f, 0.085f, 0.f}},
    {128, 64, 64, 1, false, {1.100f, 2.750f, 0.253f, 0.085f, 0.800f, 0.050f, 0.144f}},
    {16, 16, 64, 4, true, {2.610f, 0.434f, 0.394f, 0.113f, 0.f, 0.f, 0.f}},
    {16, 32, 64, 4, true, {2.783f, 0.392f, 0.603f, 0.126f, 0.f, 0.f, 0.f}},
    {256, 128, 32, 1, true, {1.258f, 4.155f, 0.580f, 0.f, 0.f, 0.163f, 0.069f}},
    {128, 128, 32, 1, true, {2.342f, 2.491f, 0.376f, 0.f, 0.f, 0.129f, 0.142f}},
    {256, 64, 32, 1, true, {2.515f, 4.531f, 0.328f, 0.f, 0.f, 0.057f, 0.052f}},
    {128, 128, 32, 1, true, {0.f, 13.979f, 0.756f, 0.205f, 0.f, 0.230f, 0.f}},
    {128, 64, 32, 1, true, {1.775f, 6.853f, 0.583f, 0.123f, 0.f, 0.218f, 0.f}},
    {64, 64, 32, 1, true, {3.299f, 3.197f, 0.383f, 0.f, 0.f, 0.147f, 0.f}},
};

static const char* const tile_name[T_COUNT] = {
    "256x256x64", "256x192x64", "192x128x64", "128x256x64", "128x128x64, 8 wavefronts", "128x128x64", "96x128x64", "64x128x64", "256x128x32", "128x64x32, 2 slices",
    "128x64x32, 3 slices", "64x64x64", "64x64x32", "32x64x64", "64x64x64, 2 groups", "32x64x64, 4 groups", "128x64x64", "small outputs 16x16", "small outputs 16x32",
    "patch 256x128", "patch 128x128", "patch 256x64", "through registers 128x128", "through registers 128x64", "through registers 64x64",
    "slabs 64x64x64", "slabs 64x64x32", "small 3x3 32x16", "small 3x3 64x16", "small 3x3 64x32", "small 3x3 128x32", "mid 3x3 96x128", "mid 3x3 192x128"};

// The patch kernel's view of a layer: strips and bordered pixels (mv); -1 = not a layer of its.
static int patch_geometry(const ConvParams& p, int* strip_w, int* slots, long long* mv) {
    int sw = p.W;
    while (sw > 64 && sw % 2 == 0) sw /= 2;
    if (sw > 128) return -1;
    const int wp = sw + (p.W == sw ? 1 : 2);
    *strip_w = sw;
    *slots = wp;
    *mv = (long long)(p.M / p.PQ) * (p.W / sw) * (p.H + 1) * wp;
    return *mv >= (1LL << 24) - 4096 ? -1 : 0;         // slots in whole rows of tiles: far below 2^31
}
static int patch_transfers(int bm, int nw, int slots) { return ((bm + 2 * slots + 2 + 15) / 16 + nw - 1) / nw; }
// Whether the patch kernel's tile `id` takes the layer; *mv as above.
static bool patch_takes(const ConvParams& p, TileId id, long long* mv) {
    int sw, wp;
    if (patch_geometry(p, &sw, &wp, mv)) return false;
    if (id == T_PATCH256x128) return p.Cout % 128 == 0 && patch_transfers(256, 8, wp) <= 4;
    if (id == T_PATCH128x128) return p.Cout % 128 == 0 && patch_transfers(128, 4, wp) <= 6;
    return id == T_PATCH256x64 && p.Cout % 64 == 0 && p.Cout % 128 != 0 && patch_transfers(256, 4, wp) <= 8;
}
static int launch_conv3x3_patch(const ConvParams& params, TileId id, hipStream_t stream) {
    ConvParams p = params;
    int wp;
    long long mv;
    if (!patch_takes(p, id, &mv) || patch_geometry(p, &p.strip_w, &wp, &mv)) { set_error("conv: not a layer of the patch kernel"); return -5; }
    p.strips = p.W / p.strip_w;
    p.by_pq = divisor(p.PQ); p.by_strips = divisor(p.strips); p.by_row = divisor(wp); p.by_image = divisor((p.H + 1LL) * wp);
    if (id == T_PATCH256x128) {
        if (patch_transfers(256, 8, wp) <= 3) return launch_patch_tile<256, 128, 4, 2, 3, 3>(p, mv, stream);
        return launch_patch_tile<256, 128, 4, 2, 4, 3>(p, mv, stream);
    }
    if (id == T_PATCH128x128) {
        if (patch_transfers(128, 4, wp) <= 4) return launch_patch_tile<128, 128, 2, 2, 4, 3>(p, mv, stream);
        return launch_patch_tile<128, 128, 2, 2, 6, 3>(p, mv, stream);
    }
    // 64 channels in and out and tiles enough for two per workgroup: workgroups that walk over tiles
    const bool walk = p.Cout == 64 && p.C <= 128 && (mv + 255) / 256 >= 1024;
    if (patch_transfers(256, 4, wp) <= 6) return walk ? launch_patch_walk<256, 64, 4, 1, 6, 3>(p, mv, stream) : launch_patch_tile<256, 64, 4, 1, 6, 3>(p, mv, stream);
    return walk ? launch_patch_walk<256, 64, 4, 1, 8, 3>(p, mv, stream) : launch_patch_tile<256, 64, 4, 1, 8, 3>(p, mv, stream);
}

// Tile columns of a group (TileOrder): the contiguous range of about tiles / 8 tiles that an XCD gets should
// touch as few operand rows as possible, cw * BN weight rows and (range / cw) * BM input rows.
static int pick_tile_cw(long long tiles_m, int tiles_n, int bm, int bn) {
    const double per = std::max(1.0, (double)(tiles_m * tiles_n) / 8.0);
    int best = 1;
    double best_rows = 1e30;
    for (int c = 1; c <= tiles_n; ++c) {
        const double rows = c * (double)bn + std::min((double)tiles_m, std::ceil(per / c)) * bm;
        if (rows < best_rows) { best_rows = rows; best = c; }
    }
    return best;
}

void set_tile_order(ConvParams& p, long long tiles_m, int tiles_n, int bm, int bn, int bk, int parts) {
    TileOrder& o = p.order;
    o.cw = pick_tile_cw(tiles_m, tiles_n, bm, bn);
    o.tiles = (int)(tiles_m * tiles_n);
    o.group = (int)(tiles_m * o.cw);
    o.full = tiles_n / o.cw;
    o.last = tiles_n - o.full * o.cw;
    o.by_tiles = divisor(o.tiles); o.by_group = divisor(o.group); o.by_cw = divisor(o.cw); o.by_last = divisor(o.last);
    p.by_pq = divisor(p.PQ); p.by_q = divisor(p.Q); p.by_c = divisor(p.C); p.by_s = divisor(p.S);
    p.by_row = divisor(p.W + 1LL); p.by_image = divisor((p.H + 1LL) * (p.W + 1LL));
    p.kchunk = ((p.Kg + bk - 1) / bk + parts - 1) / parts;
}

// One launch of conv_igemm_dma_kernel on a BM x BN tile.  KG > 1: the reduction split over KG groups of wavefronts inside the
// workgroup; p.ksplit > 1 (KG == 1 only): over ksplit workgroups per tile, with a second launch that adds their slabs.
template <int BM, int BN, int BK, int WGM, int WGN, int STAGES, int KG = 1>
static int launch_dma_tile(const ConvParams& p, int mode, hipStream_t stream) {
    const long long tiles_m = (p.M + BM - 1) / BM;
    const int tiles_n = (p.Cout + BN - 1) / BN;
    const long long tiles = tiles_m * tiles_n * p.ksplit;
    if (tiles <= 0 || tiles > 0x7fffffffLL) { set_error("conv: bad grid (%lld tiles)", tiles); return -5; }
    constexpr unsigned ring = KG * STAGES * (BM + BN) * BK * 2, ctile = BM * (BN + 8) * 2;
    constexpr unsigned lds = (ring > ctile ? ring : ctile) + 1024;    // the epilogue parks the output tile in the ring's LDS; + the tile's bias row
    static_assert(lds <= 160 * 1024, "LDS limit");
    dim3 grid((unsigned)tiles), block(64 * WGM * WGN * KG);
    ConvParams q = p;
    set_tile_order(q, tiles_m, tiles_n, BM, BN, BK, KG > 1 ? KG : p.ksplit);
#define STRAIT_GO(...) launch_with_lds<conv_igemm_dma_kernel<__VA_ARGS__>>(q, grid, block, lds, lds, stream)
    auto after = [&]() -> int {                        // the second launch of a split reduction
        if (p.ksplit > 1) {
            const long long n8 = (long long)p.M * (p.Cout / 8);
            hipLaunchKernelGGL(splitk_finish_kernel, dim3((unsigned)((n8 + 255) / 256)), dim3(256), 0, stream, q);
        }
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) { set_error("conv launch: %s", hipGetErrorString(e)); return -2; }
        return 0;
    };
    int rc;
    if (p.res_f32 && p.ksplit == 1) {
        if constexpr (BM <= 64 && BN == 64) {
            if (mode == MODE_1X1) rc = STRAIT_GO(BM, BN, BK, WGM, WGN, MODE_1X1, STAGES, false, RES_WIDE, false, KG);
            else rc = STRAIT_GO(BM, BN, BK, WGM, WGN, MODE_GATHER8, STAGES, false, RES_WIDE, false, KG);
        } else { set_error("conv: this tile does not add a residual in fp32"); return -5; }
    } else if constexpr (KG > 1) {
        if (mode == MODE_1X1 && p.res) rc = STRAIT_GO(BM, BN, BK, WGM, WGN, MODE_1X1, STAGES, false, RES_EARLY, false, KG);
        else if (mode == MODE_1X1) rc = STRAIT_GO(BM, BN, BK, WGM, WGN, MODE_1X1, STAGES, false, RES_LATE, false, KG);
        else rc = STRAIT_GO(BM, BN, BK, WGM, WGN, MODE_GATHER8, STAGES, false, RES_LATE, false, KG);
    } else {
        if constexpr (BM == 128 && BN == 128 && dma_deep<BM, BN, BK, WGM, WGN>()) {
            if (p.Kg < 512 && p.act != ACT_GELU && !p.x2) {
                if (mode == MODE_1X1 && p.res && p.ksplit == 1) rc = STRAIT_GO(BM, BN, BK, WGM, WGN, MODE_1X1, STAGES, false, RES_EARLY, false, 1, LN_NONE, false);
                else if (mode == MODE_1X1) rc = STRAIT_GO(BM, BN, BK, WGM, WGN, MODE_1X1, STAGES, false, RES_LATE, false, 1, LN_NONE, false);
                else rc = STRAIT_GO(BM, BN, BK, WGM, WGN, MODE_GATHER8, STAGES, false, RES_LATE, false, 1, LN_NONE, false);
                return rc ? rc : after();
            }
        }
        if (mode == MODE_1X1 && p.act == ACT_GELU) rc = STRAIT_GO(BM, BN, BK, WGM, WGN, MODE_1X1, STAGES, true, RES_LATE);
        else if (mode == MODE_1X1 && p.x2) rc = STRAIT_GO(BM, BN, BK, WGM, WGN, MODE_1X1, STAGES, false, RES_LATE, true);
        else if (mode == MODE_1X1 && p.res && p.ksplit == 1) rc = STRAIT_GO(BM, BN, BK, WGM, WGN, MODE_1X1, STAGES, false, RES_EARLY);
        else if (mode == MODE_1X1) rc = STRAIT_GO(BM, BN, BK, WGM, WGN, MODE_1X1, STAGES, false, RES_LATE);
        else rc = STRAIT_GO(BM, BN, BK, WGM, WGN, MODE_GATHER8, STAGES, false, RES_LATE);
    }
#undef STRAIT_GO
    return rc ? rc : after();
}

template <int BM, int BN>
static int launch_tile(const ConvParams& p, int mode, bool staged, hipStream_t stream) {
    const long long tiles = (long long)((p.M + BM - 1) / BM) * ((p.Cout + BN - 1) / BN);
    if (tiles <= 0 || tiles > 0x7fffffffLL) { set_error("conv: bad grid (%lld tiles)", tiles); return -5; }
    dim3 grid((unsigned)tiles), block(256);
#define STRAIT_LAUNCH(MODE, ST) hipLaunchKernelGGL((conv_igemm_kernel<BM, BN, MODE, ST>), grid, block, 0, stream, p)
    if (mode == MODE_1X1) { if (staged) STRAIT_LAUNCH(MODE_1X1, true); else STRAIT_LAUNCH(MODE_1X1, false); }
    else if (mode == MODE_GATHER8) { if (staged) STRAIT_LAUNCH(MODE_GATHER8, true); else STRAIT_LAUNCH(MODE_GATHER8, false); }
    else { if (staged) STRAIT_LAUNCH(MODE_SCALAR, true); else STRAIT_LAUNCH(MODE_SCALAR, false); }
#undef STRAIT_LAUNCH
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) { set_error("conv launch: %s", hipGetErrorString(e)); return -2; }
    return 0;
}

static float estimate_us(const ConvParams& p, TileId id, long long pixels, bool gather, bool staged, double mb) {
    const TileInfo& t = tile_info[id];
    const long long tiles = (pixels + t.bm - 1) / t.bm * ((p.Cout + t.bn - 1) / t.bn);
    const long long per_cu = (tiles + 255) / 256;
    const double nk = std::ceil((double)p.Kg / (t.bk * t.kg));
    double r;
    if (id == T_SK16 || id == T_SK32) r = staged ? std::max(1.0, tiles / 256.0) : (double)per_cu;     // (the better fit in each case)
    else if (!t.shared) r = (double)per_cu;
    else r = per_cu > 8 ? tiles / 512.0 : per_cu / 2 + (per_cu % 2 ? 0.6 : 0.0);
    return (float)(t.c[0] + r * (t.c[1] + nk * (t.c[2] + (gather ? t.c[3] : 0.f)) + (p.act == ACT_GELU ? t.c[4] : 0.f)) + t.c[5] * mb +
                   t.c[6] * std::max(0.0, mb - 250.0));
}

// The small 3x3 kernel's tiles (conv3x3_small.hip), T_SMALL32x16 on: their time is the launch, a round of tiles, a slice of 64 channels, its patch (in
// transfers of 32 slots) and the operands' megabytes.  Fits to 152 to 188 layers each (1 to 32 images of 5 to 64 pixels, 64 to 512 channels; mean error 1.5 %,
// largest 6.5 %; the choice among them was the best of them every time).
struct SmallTile { int bm, bn; float c[5]; };
static const SmallTile small_tile[4] = {{32, 16, {1.428f, 2.552f, 0.236f, 0.0627f, 0.021f}}, {64, 16, {1.494f, 2.644f, 0.550f, 0.0211f, 0.f}},
                                        {64, 32, {1.348f, 2.764f, 0.605f, 0.0712f, 0.f}}, {128, 32, {1.259f, 2.766f, 0.913f, 0.0644f, 0.116f}}};
static float small_us(const ConvParams& p, const SmallTile& t, double mb) {
    const long long mv = (long long)(p.M / p.PQ) * (p.H + 1) * (p.W + 1);
    const double r = std::ceil((double)((mv + t.bm - 1) / t.bm * (p.Cout / t.bn)) / 256.0), nk = p.C / 64;
    return (float)(t.c[0] + r * (t.c[1] + nk * (t.c[2] + t.c[3] * ((t.bm + 2 * (p.W + 1) + 2 + 31) / 32))) + t.c[4] * mb);
}

// The mid-size 3x3 kernel's (conv3x3_mid.hip): the launch, a round of tiles, a tap of 64 channels, the operands' megabytes.
// Fits to 80 layers (3 to 32 images of 14 to 64 pixels, 64 to 512 channels): at most 11 % off, and that where half of the units are idle and they are too high.
struct MidTile { int bm; float c[4]; };
static const MidTile mid_tile[2] = {{96, {2.4f, 4.4f, 0.29f, 0.04f}}, {192, {1.2f, 6.9f, 0.54f, 0.03f}}};
static float mid_us(const ConvParams& p, const MidTile& t, double mb) {
    const long long mv = (long long)(p.M / p.PQ) * (p.H + 1) * (p.W + 1);
    const double r = std::ceil((double)((mv + t.bm - 1) / t.bm * (p.Cout / 128)) / 256.0);
    return (float)(t.c[0] + r * (t.c[1] + 9 * (p.C / 64) * t.c[2]) + t.c[3] * mb);
}

static int launch_tile_id(const ConvParams& p, TileId id, int mode, bool staged, hipStream_t stream) {
    switch (id) {
        case T256x256: return launch_dma_tile<256, 256, 64, 2, 4, 2>(p, mode, stream);
        case T256x192: return launch_dma_tile<256, 192, 64, 4, 2, 2>(p, mode, stream);
        case T192x128: return launch_dma_tile<192, 128, 64, 2, 4, 3>(p, mode, stream);
        case T128x256: return launch_dma_tile<128, 256, 64, 2, 4, 3>(p, mode, stream);
        case T128x128: return launch_dma_tile<128, 128, 64, 4, 2, 4>(p, mode, stream);
        case T128x128_2: return launch_dma_tile<128, 128, 64, 2, 2, 2>(p, mode, stream);
        case T96x128: return launch_dma_tile<96, 128, 64, 1, 4, 4>(p, mode, stream);
        case T64x128: return launch_dma_tile<64, 128, 64, 2, 2, 3>(p, mode, stream);
        case T256x128s: return launch_dma_tile<256, 128, 32, 4, 2, 3>(p, mode, stream);
        case T128x64_2: return launch_dma_tile<128, 64, 32, 2, 2, 2>(p, mode, stream);
        case T128x64_3: return launch_dma_tile<128, 64, 32, 2, 2, 3>(p, mode, stream);
        case T64x64: return launch_dma_tile<64, 64, 64, 2, 2, 3>(p, mode, stream);
        case T64x64s: return launch_dma_tile<64, 64, 32, 2, 2, 3>(p, mode, stream);
        case T32x64: return launch_dma_tile<32, 64, 64, 1, 2, 4>(p, mode, stream);
        case T64x64_g2: return launch_dma_tile<64, 64, 64, 2, 2, 3, 2>(p, mode, stream);
        case T32x64_g4: return launch_dma_tile<32, 64, 64, 1, 2, 3, 4>(p, mode, stream);
        case T128x64: return launch_dma_tile<128, 64, 64, 4, 2, 5>(p, mode, stream);
        case T_SK16: return launch_conv_skinny(p, 16, mode == MODE_GATHER8, stream);
        case T_SK32: return launch_conv_skinny(p, 32, mode == MODE_GATHER8, stream);
        case T_SLABS64: return launch_dma_tile<64, 64, 64, 2, 2, 3>(p, mode, stream);
        case T_SLABS64s: return launch_dma_tile<64, 64, 32, 2, 2, 3>(p, mode, stream);
        case T_REG128x128: return launch_tile<128, 128>(p, mode, staged, stream);
        case T_REG128x64: return launch_tile<128, 64>(p, mode, staged, stream);
        case T_REG64x64: return launch_tile<64, 64>(p, mode, staged, stream);
        case T_SMALL32x16: case T_SMALL64x16: case T_SMALL64x32: case T_SMALL128x32:
            return launch_conv3x3_small(p, small_tile[id - T_SMALL32x16].bm, small_tile[id - T_SMALL32x16].bn, stream);
        case T_MID96x128: case T_MID192x128: return launch_conv3x3_mid(p, mid_tile[id - T_MID96x128].bm, stream);
        default: return launch_conv3x3_patch(p, id, stream);
    }
}

// Up to 128 tiles of 64 x 64, split over up to 32 workgroups each that leave fp32 slabs, which a second launch adds: the number of parts
// (at least four 64-wide slices each, slabs of at most `limit` bytes) with the smallest estimate, which *us receives; 1 = no split.
// The estimate is a fit like the table's, to 200 layers of 8 to 4096 channels and reductions of 512 to 32768, each in 2 to 48 parts
// (mean error 7 %; its number of parts is on average within 5 % of the best): the two launches, a round of workgroups, a slice,
// the slabs' bytes, the finishing launch's chain of slabs, the operands' bytes; and no faster than 6.2 TB/s of operands.
static int slab_split(const ConvParams& p, size_t limit, bool gather, float* us) {
    int best = 1;
    *us = 1e30f;
    const long long t = (long long)((p.M + 63) / 64) * ((p.Cout + 63) / 64);
    if (t > 128 || p.x2 || p.Cout % 8 != 0 || p.ldy % 8 != 0) return 1;
    const double slab_mb = (double)p.M * p.Cout * 4e-6, operand_mb = ((double)p.x_elems + (double)p.Cout * p.Kg) * 2e-6;
    for (int ks : {2, 3, 4, 6, 8, 12, 16, 24, 32}) {
        const double nk = std::ceil(p.Kg / 64.0 / ks), r = std::max(1.0, (double)(t * ks) / 512.0);
        if (nk < 4 || (size_t)ks * p.M * p.Cout * 4 > limit) break;
        const float e = (float)std::max(2.0 + operand_mb / 6.2, 5.093 + r * (0.586 + nk * (gather ? 0.287 : 0.181)) + 0.651 * ks * slab_mb + 0.111 * ks + 0.064 * operand_mb);
        if (e < *us) { *us = e; best = ks; }
    }
    return best;
}

// Checks a layer, fills in what the launchers derive and chooses its kernel: >= 0 a TileId, < 0 an error.
static int choose_conv(ConvParams& p, int* mode_out, bool* staged_out) {
    if (!p.x || !p.w || !p.y || p.M <= 0 || p.Cout <= 0 || p.Kg <= 0 || p.C <= 0 || p.R <= 0 || p.S <= 0 ||
        p.Q <= 0 || p.PQ <= 0 || p.stride_h <= 0 || p.stride_w <= 0) {
        set_error("conv: invalid parameters"); return -1;
    }
    if (p.x2) {
        // a second source: both parts whole 64-wide slices, the first part a dense pointwise input, no residual
        if (p.R != 1 || p.S != 1 || p.stride_h != 1 || p.stride_w != 1 || p.pad_h || p.pad_w || p.res || p.out_f32 || p.act == ACT_GELU ||
            p.C % 64 != 0 || p.K2 <= 0 || p.K2 % 64 != 0 || p.Kg != p.C + p.K2 || p.sW != p.C || p.stride2 <= 0 ||
            p.sW2 % 8 != 0 || p.sH2 % 8 != 0 || p.sN2 % 8 != 0 || p.Cout % 8 != 0 || p.ldy % 8 != 0 ||
            (reinterpret_cast<uintptr_t>(p.x2) & 15)) {
            set_error("conv: unsupported use of a second source"); return -5;
        }
        // the furthest element any output pixel reads from it
        p.x2_elems = (long long)(p.M / p.PQ - 1) * p.sN2 + (long long)((p.PQ / p.Q - 1) * p.stride2) * p.sH2 +
                     (long long)((p.Q - 1) * p.stride2) * p.sW2 + p.K2;
        if (p.x2_elems * 2 > 0x7fffffffLL) { set_error("conv: second source too large"); return -5; }
    } else if (p.Kg != p.R * p.S * p.C) { set_error("conv: Kg != R*S*C"); return -5; }
    if (p.ldw % 8 != 0 || p.ldw < p.Kg) { set_error("conv: weight pitch %d must be a multiple of 8 and >= %d", p.ldw, p.Kg); return -5; }
    if (p.ldy < p.Cout) { set_error("conv: ldy < Cout"); return -5; }
    if ((reinterpret_cast<uintptr_t>(p.x) | reinterpret_cast<uintptr_t>(p.w) | reinterpret_cast<uintptr_t>(p.y) |
         reinterpret_cast<uintptr_t>(p.res)) & 15) { set_error("conv: pointers must be 16-byte aligned"); return -1; }
    const bool vec_ok = (p.C % 8 == 0) && (p.sW % 8 == 0) && (p.sH % 8 == 0) && (p.sN % 8 == 0);
    int& mode = *mode_out;
    if (vec_ok && p.R == 1 && p.S == 1 && p.pad_h == 0 && p.pad_w == 0) mode = MODE_1X1;
    else if (vec_ok) mode = MODE_GATHER8;
    else mode = MODE_SCALAR;
    const bool staged = *staged_out = !p.out_f32 && (p.Cout % 8 == 0) && (p.ldy % 8 == 0);
    auto tiles = [&](int bm, int bn) { return (long long)((p.M + bm - 1) / bm) * ((p.Cout + bn - 1) / bn); };
    const bool dense = mode == MODE_1X1 && p.stride_h == 1;
    p.x_elems = dense ? (long long)p.M * p.sW : (long long)(p.M / p.PQ) * p.sN;
    const long long lead = (long long)p.pad_h * p.sH + (long long)p.pad_w * p.sW;
    const bool small = (p.x_elems + lead) * 2 <= 0x7fffffffLL && (long long)p.Cout * p.ldw * 2 <= 0x7fffffffLL;
    auto through_registers = [&]() {
        if (p.Cout > 64 && tiles(128, 128) >= 512) return T_REG128x128;
        return tiles(128, 64) >= 512 ? T_REG128x64 : T_REG64x64;
    };
    p.ksplit = 1;
    // Up to 128 tiles of 64 x 64 the residual's pass through LDS is little beside a reduction of more than 1024 (128 x 768 x 3072: 8.6 us, 8.5 without); larger
    // layers, which their stores bound, add it to the rounded product.
    p.res_f32 = p.res && p.Kg > 1024 && tiles(64, 64) <= 128;
    // (GELU after a residual add is left to the first kernel: the LDS-direct one applies GELU before the staging)
    const bool regular = (mode == MODE_1X1 && !(p.act == ACT_GELU && p.res)) || (mode == MODE_GATHER8 && p.C % 32 == 0 && p.R * p.S <= 32 && p.act != ACT_GELU);
    if (regular && small) {
        const bool whole64 = p.Kg % 64 == 0 && p.C % 64 == 0;                 // slices of 64 never straddle a tap or the end
        const bool gather = mode == MODE_GATHER8;
        const double mb = ((double)p.x_elems * 2 + (double)p.Cout * p.Kg * 2 + (double)p.M * p.Cout * ((p.out_f32 ? 4 : 2) + (p.res ? 2 : 0))) * 1e-6;
        TileId best = T_COUNT;
        float best_us = 1e30f;
        auto consider = [&](TileId id, long long pixels) {
            const float us = estimate_us(p, id, pixels, gather, staged, mb);
            if (us < best_us) { best_us = us; best = id; }
        };
        if (staged) {
            for (int i = 0; i < T_DMA; ++i) {
                const TileInfo& t = tile_info[i];
                if (t.bk == 64 && gather && p.C % 64 != 0) continue;
                if (p.res_f32 && (t.bm > 64 || t.bn > 64)) continue;                        // (the larger ones leave most compute units idle)
                if (t.kg > 1 && (p.Kg < 512 || p.x2 || p.act == ACT_GELU)) continue;        // too short to split
                if (i == T256x128s && p.Kg >= 512 && !(gather && p.C % 64 != 0)) continue;  // a tile for streaming layers, and for channels in halves of a slice
                if (i == T128x64 && (p.Kg < 512 || p.Cout < 128)) continue;                 // fitted on reductions worth its ring
                if (t.bm < 128 && mb > 250 && !p.res_f32) continue;                                       // estimates are not good for so many small tiles
                consider((TileId)i, p.M);
            }
            if (gather && p.R == 3 && p.S == 3 && p.stride_h == 1 && p.stride_w == 1 && p.pad_h == 1 && p.pad_w == 1 && !p.res &&
                p.W >= 14 && p.Q == p.W && p.PQ == p.H * p.W) {
                for (int i = T_PATCH256x128; i <= T_PATCH256x64; ++i) {
                    long long mv;
                    if (patch_takes(p, (TileId)i, &mv)) consider((TileId)i, mv);
                }
            }
            if (gather && p.R == 3 && p.S == 3 && p.stride_h == 1 && p.stride_w == 1 && p.pad_h == 1 && p.pad_w == 1 && !p.res &&
                p.Q == p.W && p.PQ == p.H * p.W) {
                for (int i = 0; i < 4; ++i) {
                    if (!conv3x3_small_takes(p, small_tile[i].bm, small_tile[i].bn)) continue;
                    const float us = small_us(p, small_tile[i], mb);
                    if (us < best_us) { best_us = us; best = (TileId)(T_SMALL32x16 + i); }
                }
                for (int i = 0; i < 2; ++i) {
                    if (!conv3x3_mid_takes(p, mid_tile[i].bm)) continue;
                    const float us = mid_us(p, mid_tile[i], mb);
                    if (us < best_us) { best_us = us; best = (TileId)(T_MID96x128 + i); }
                }
            }
        } else {
            // fp32 outputs, and counts of channels that are no whole chunks: the register-staged kernel on the tile that fills the chip,
            // against the small-output kernel further down.  With fp32 outputs 16384 x 768 x 4096 takes 168 us here and 1034 there, 2221 x
            // 1000 x 768 22 and 47, 9 x 1000 x 2048, a classifier, 23 and 5.5.  230 layers: the choice is on average
            // 2.6 % off the better of the two.
            consider(through_registers(), p.M);
        }
        // short reductions to whole fp16 chunks stay with the kernels that read operands through LDS
        if (whole64 && (!staged || p.Kg >= 192) && tiles(16, 16) <= 0x7fffffffLL && mb <= 250) {
            consider(T_SK16, p.M);
            consider(T_SK32, p.M);
        }
        // A split reduction for few outputs, where the kernels above leave compute units idle behind a long chain; fp16 outputs of at most
        // 4608 had none that gained.  385 x 1024 x 8192 with fp32 outputs: 20 us against 87 with small outputs; 399 x 768 x 8192: 19
        // against 65; 13 x 1000 x 25088 in fp16: 16 against 41.  A fifth is asked of it against kernels that share the
        // reduction out themselves: with that none of the 200 layers measured is slower for it.
        if ((!staged || p.Kg > 4608) && p.ws && (reinterpret_cast<uintptr_t>(p.ws) & 15) == 0) {
            float us;
            const int ks = slab_split(p, p.ws_bytes, gather, &us);
            if (ks > 1 && us < (best >= T_REG128x128 && best < T_SMALL32x16 ? 1.f : 0.8f) * best_us) {
                p.ksplit = ks;
                return whole64 ? T_SLABS64 : T_SLABS64s;
            }
        }
        if (best != T_COUNT) return best;
    }
    if (p.x2) { set_error("conv: a second source needs the LDS-direct kernels (sizes out of their range)"); return -5; }
    return through_registers();
}

// The same for a dense product with a LayerNorm folded in: the LDS-direct kernel only, on the tiles that gemm_ln.hip instantiates (slices of 64).  The
// estimates are the plain products', whose epilogues are shorter by 0.6 to 1 us a round (gemm_ln.hip); among tiles that they put within a few per
// cent of each other the choice is not better founded than that.
static int gemm_ln_tile(ConvParams& p) {
    int mode = 0;
    bool staged = false;
    const int rc = choose_conv(p, &mode, &staged);     // checks the parameters and fills in what is derived
    if (rc < 0) return rc;
    if (mode != MODE_1X1 || !staged || p.stride_h != 1 || p.x2 || p.Kg % 64 != 0 || p.Cout % 64 != 0) { set_error("gemm with LayerNorm: not a dense product of whole 64-channel groups"); return -5; }
    p.ksplit = 1;
    const double mb = ((double)p.x_elems * 2 + (double)p.Cout * p.Kg * 2 + (double)p.M * p.Cout * (p.res ? 4 : 2)) * 1e-6;
    int best = -5;
    float best_us = 1e30f;
    for (int i = 0; i < T_DMA; ++i) {
        const TileInfo& t = tile_info[i];
        if (p.ln_stats && t.bn == 256 && (p.ln_csum ? p.Kg : p.Cout) > 64 * LN_MAX_PARTS_256) continue;         // (LDS)
        if (t.bk != 64 || (t.kg > 1 && (p.Kg < 512 || p.act == ACT_GELU)) || (t.bm < 128 && mb > 250)) continue;
        if (t.shared && !gemm_ln_two_fit(i, p)) continue;   // (the rows' statistics lie in LDS too: those of more than 768 channels leave no room for a second tile)
        const float us = estimate_us(p, (TileId)i, p.M, false, true, mb);
        if (us < best_us) { best_us = us; best = i; }
    }
    return best;
}

// A part of a batch (ConvParams::whole_M) may take another kernel than the whole one only where both add in the same order, so that a batch's result is the same
// bit for bit whether it is computed in parts or not, which depends on what else the GPU has to do.  The LDS-direct kernel adds up the reduction in steps of 16 on
// all tiles on which one group of wavefronts does; every other kernel, or way of splitting the reduction, has an order of its own.
static bool same_order(int a, const ConvParams& pa, int b, const ConvParams& pb) {
    auto one_group = [](int id) { return id < T_DMA && tile_info[id].kg == 1; };
    return pa.ksplit == pb.ksplit && pa.res_f32 == pb.res_f32 && (a == b || (one_group(a) && one_group(b)));
}

int choose_gemm_ln(ConvParams& p) {
    const int id = gemm_ln_tile(p);
    if (id < 0 || p.whole_M <= p.M) return id;
    ConvParams whole = p;
    whole.M = p.whole_M;
    const int as_whole = gemm_ln_tile(whole);
    return as_whole < 0 || !same_order(id, p, as_whole, whole) ? as_whole : id;
}

int launch_conv(const ConvParams& params, hipStream_t stream) {
    ConvParams p = params;
    int mode = 0;
    bool staged = false;
    int id = choose_conv(p, &mode, &staged);
    if (id >= 0 && p.whole_M > p.M) {                  // (a kernel that takes the whole takes a part)
        ConvParams whole = p;
        whole.M = p.whole_M;
        const int as_whole = choose_conv(whole, &mode, &staged);
        if (as_whole < 0 || !same_order(id, p, as_whole, whole)) {
            id = as_whole;
            p.ksplit = whole.ksplit; p.res_f32 = whole.res_f32;
        }
    }
    return id < 0 ? id : launch_tile_id(p, (TileId)id, mode, staged, stream);
}
size_t conv_workspace_bytes(const ConvParams& params, size_t limit) {
    ConvParams p = params;
    p.ws = (float*)256;                                // any aligned address: nothing is launched
    p.ws_bytes = limit;
    int mode = 0;
    bool staged = false;
    const int id = choose_conv(p, &mode, &staged);
    return id == T_SLABS64 || id == T_SLABS64s ? (size_t)p.ksplit * p.M * p.Cout * 4 : 0;
}
const char* conv_kernel_name(const ConvParams& params) {
    ConvParams p = params;
    int mode = 0;
    bool staged = false;
    const int id = choose_conv(p, &mode, &staged);
    return id < 0 ? nullptr : tile_name[id];
}

}  // namespace strait
