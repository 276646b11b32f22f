// The first two layers of an inverted residual block in one launch for gfx950: a 1x1 convolution that expands Cin
// channels to Chid (+ bias + activation) and the depthwise 3x3 convolution of stride 1 or 2 and padding 1 behind it
// (+ bias + activation).  (Paper Section 3.2 step (2): two members of MobileNetV2's kernel sequence.)
//
// Run as two launches, the expanded tensor, six times the block's input and the largest tensor of the network, is
// written to memory and read back.  Here it exists only tile by tile in LDS: a workgroup (4 wavefronts) takes a tile of
// TP x TQ output positions of one image and
//   A. loads the input pixels under the tile and its one-pixel rim (all Cin channels, zeros outside the image) into
//      LDS once;
//   B. for each group of 32 expanded channels in turn
//      1. computes the group for every pixel of A: blocks of 32 pixels, v_mfma_f32_32x32x16_f16 with the weights as
//         the A operand (this lane's fragments in registers, those of the next group already requested), + bias,
//         activation, fp16, zero for pixels outside the image (the depthwise layer pads the expanded tensor, not the
//         input), into LDS as [pixel][32 channels];
//      2. depthwise: a thread owns 8 channels of a column of TH output positions and adds their nine taps in fp32
//         from LDS, in the order the stand-alone depthwise kernels use, + bias, activation, and stores 16 bytes per
//         position.
// Every arithmetic step is the one the two stand-alone kernels take, in the same order: results are bit-identical.
// The groups of a tile can be shared out over several workgroups (gridDim.y), down to one group each (ONE): such a workgroup
// requests nothing ahead and is done after one pass, which is the whole time of a small batch's launch.  5 images of 14 x 14 with 64
// channels expanded to 384: tiles of 4 rows and one group each, 240 workgroups, 4.7 us; tiles of 14 rows, two groups
// each, 30 workgroups, were 12.7.
#include <algorithm>
#include <atomic>

#include "tiles.hpp"

namespace strait {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef unsigned uintx4 __attribute__((ext_vector_type(4)));

constexpr int EDW_HP = 40;                                // halfs between pixels of the expanded tile: 32 channels + 8

struct ExpandDwParams {
    const half_t* x; int N, H, W, Cin;
    const half_t* w1; int ldw1; const float* b1; int Chid, act1;
    const half_t* wd; const float* bd; int act2;
    half_t* y; int P, Q, tiles_p, tiles_q, groups_per_block, hp;
    Divisor by_tiles_p, by_tiles_q;
    int wide;                          // rows of 59 million elements and more
};

__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// px / IC for 0 <= px < LIMIT, by a 24-bit product (exact: px (IC - 65536 mod IC) stays below 65536)
template <int IC, int LIMIT>
__device__ __forceinline__ int edw_tile_row(int px) {
    constexpr unsigned INV = 65536u / IC + 1;
    static_assert((unsigned)LIMIT * (INV * IC - 65536u) < 65536u && (unsigned)LIMIT * INV < (1u << 24), "exact quotients");
    return (int)(((unsigned)px & 0xffffffu) * INV >> 16);
}
__device__ __forceinline__ float edw_act(float v, int act) {
    if (act == ACT_RELU) return fmaxf(v, 0.f);
    if (act == ACT_RELU6) return fminf(fmaxf(v, 0.f), 6.f);
    return v;
}

// KS: 16-channel steps of the expansion's reduction (Cin rounded up); STRIDE of the depthwise layer; the tile is
// TP x TQ outputs with TP = 256 / (4 TQ) * TH.  ONE: one tile and one group per workgroup.
template <int KS, int STRIDE, int TQ, int TH, bool ONE>
__global__ void __launch_bounds__(256) expand_dw_kernel(const ExpandDwParams p) {
    constexpr int STRIPS = 256 / (4 * TQ), TP = STRIPS * TH;
    constexpr int IR = (TP - 1) * STRIDE + 3, IC = (TQ - 1) * STRIDE + 3;      // input pixels under the tile and its rim
    constexpr int NPX = IR * IC, NPB = (NPX + 31) / 32, ROWS = NPB * 32;
    constexpr int XP = KS * 16 + 8;                                            // halfs between pixels of the input tile
    extern __shared__ __attribute__((aligned(16))) half_t edw_smem[];
    half_t* xs = edw_smem;                                                     // [ROWS][XP]
    half_t* hs = edw_smem + ROWS * XP;                                         // [ROWS][EDW_HP]
    if (p.hp) __builtin_amdgcn_s_setprio(3);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l32 = lane & 31, lh = lane >> 5;

    // A workgroup takes every gridDim.x-th tile.  Virtual workgroup v -> tile: every XCD takes a contiguous range of tiles
    // (neighbouring tiles share rim pixels through one L2); v mod 8 is this workgroup's XCD for every v it takes, because
    // a grid smaller than the number of tiles is a multiple of eight.
    const int ntiles = p.N * p.tiles_p * p.tiles_q;
    auto tile_of = [&](int v, int& n, int& P0, int& Q0) __attribute__((always_inline)) {
        const int tile = xcd_range(ntiles, v), rest = divide(tile, p.by_tiles_q);
        n = divide(rest, p.by_tiles_p);
        Q0 = (tile - rest * p.tiles_q) * TQ; P0 = (rest - n * p.tiles_p) * TP;
    };
    const int groups = (p.Chid + 31) >> 5;
    const int g_begin = (int)blockIdx.y * p.groups_per_block;
    const int g_end = g_begin + p.groups_per_block < groups ? g_begin + p.groups_per_block : groups;

    // Weights and biases come through buffers: channels past the end have an offset beyond them and read as zero.
    constexpr unsigned OOB = 0x80000000u;
    const auto w1r = __builtin_amdgcn_make_buffer_rsrc((void*)p.w1, 0, p.Chid * p.ldw1 * 2, 0x00020000);
    const auto wdr = __builtin_amdgcn_make_buffer_rsrc((void*)p.wd, 0, 9 * p.Chid * 2, 0x00020000);
    const auto b1r = __builtin_amdgcn_make_buffer_rsrc((void*)p.b1, 0, p.b1 ? p.Chid * 4 : 0, 0x00020000);
    const auto bdr = __builtin_amdgcn_make_buffer_rsrc((void*)p.bd, 0, p.bd ? p.Chid * 4 : 0, 0x00020000);
    // fragments of the expansion's weights and its bias for group g: output channel 32 g + l32, input channels 16 ks + 8 lh ..
    auto load_w1 = [&](int g, half8 (&wf)[KS], float (&bv)[4][4]) __attribute__((always_inline)) {
        const int row = 32 * g + l32;
        const unsigned at = row < p.Chid ? (unsigned)(row * p.ldw1 + 8 * lh) * 2u : OOB;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            wf[ks] = __builtin_bit_cast(half8, __builtin_amdgcn_raw_buffer_load_b128(w1r, 16 * ks + 8 * lh < p.Cin ? at + 32u * ks : OOB, 0, 0));
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4) {
            const floatx4 b = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(b1r, (unsigned)(32 * g + 8 * g4 + 4 * lh) * 4u, 0, 0));
#pragma unroll
            for (int e = 0; e < 4; ++e) bv[g4][e] = b[e];
        }
    };
    // the depthwise layer's weights and bias of group g for this thread's 8 channels (c8)
    const int c8 = tid & 3, col = (tid >> 2) % TQ, strip = (tid >> 2) / TQ;
    auto load_wd = [&](int g, half8 (&wv)[9], float (&bdv)[8]) __attribute__((always_inline)) {
        const unsigned cd = (unsigned)(32 * g + 8 * c8), at = (int)cd < p.Chid ? cd * 2u : OOB;
#pragma unroll
        for (int k = 0; k < 9; ++k) wv[k] = __builtin_bit_cast(half8, __builtin_amdgcn_raw_buffer_load_b128(wdr, at, (unsigned)(k * p.Chid) * 2u, 0));
        const floatx4 b0 = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(bdr, cd * 4u, 0, 0));
        const floatx4 b1 = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(bdr, cd * 4u + 16u, 0, 0));
#pragma unroll
        for (int e = 0; e < 4; ++e) { bdv[e] = b0[e]; bdv[4 + e] = b1[e]; }
    };
    // both layers' weights are requested a whole group ahead: a group is short, and a wait for them would be most of it
    half8 wf[KS], wf_next[KS], wv[9], wv_next[9];
    float bv[4][4], bv_next[4][4], bdv[8], bdv_next[8];
    load_w1(g_begin, wf, bv);
    load_wd(g_begin, wv, bdv);

    // ---- A: the input tile: its 16-byte pieces are requested into registers (several before the first is waited for; a piece outside the image has an offset
    // beyond the buffer and reads as zero) and deposited in LDS.  Where a thread holds few enough of them, the next tile's are requested while this
    // tile is computed.  Threads take the same piece of every PSTEP-th pixel, so that nothing but the pixel's row and column is worked out per piece: a division, being
    // inside and a 64-bit address for each took 600 to 1400 instructions in front of the first MFMA, half of a small launch at one wavefront per SIMD, and a third of
    // them are gone (MobileNetV2 five images 281 -> 262 us).
    constexpr int CH = KS * 2;                                                 // 16-byte pieces per pixel, zero-padded
    constexpr int PSTEP = 256 / CH, NIT = (ROWS + PSTEP - 1) / PSTEP;
    constexpr bool AHEAD = NIT <= 12;
    constexpr int BATCH = AHEAD ? NIT : 8;
    const int px0 = tid / CH, ch = tid - px0 * CH;                             // (256 is no multiple of 12 or 20 pieces: the last threads take none)
    const bool takes = px0 < PSTEP, whole = ch * 8 < p.Cin;
    const unsigned row_bytes = (unsigned)(p.W * p.Cin) * 2u, pixel_bytes = (unsigned)p.Cin * 2u;
    uintx4 xv[BATCH];
    auto request_tile = [&](int v, int it0) __attribute__((always_inline)) {
        int n, P0, Q0;
        tile_of(v, n, P0, Q0);
        const int ih0 = P0 * STRIDE - 1, iw0 = Q0 * STRIDE - 1, top = ih0 < 0 ? 0 : ih0;
        // the rows under the tile, from the first that there is
        const int rows = p.H - top < IR ? p.H - top : IR;
        if (__builtin_expect(p.wide, 0)) {                                     // 18 rows that a 32-bit offset does not span
#pragma unroll
            for (int b = 0; b < BATCH; ++b) {
                const int px = px0 + (it0 + b) * PSTEP, ir = edw_tile_row<IC, ROWS + BATCH * PSTEP>(px), ic = px - ir * IC;
                const int ih = ih0 + ir, iw = iw0 + ic;
                xv[b] = uintx4{0, 0, 0, 0};
                if (px < NPX && (unsigned)ih < (unsigned)p.H && (unsigned)iw < (unsigned)p.W && whole)
                    xv[b] = *(const uintx4*)(p.x + (((long long)n * p.H + ih) * p.W + iw) * p.Cin + ch * 8);
            }
            return;
        }
        const auto xr = __builtin_amdgcn_make_buffer_rsrc((void*)(p.x + ((long long)n * p.H + top) * p.W * p.Cin), 0, (int)((unsigned)rows * row_bytes), 0x00020000);
#pragma unroll
        for (int b = 0; b < BATCH; ++b) {
            const int px = px0 + (it0 + b) * PSTEP, ir = edw_tile_row<IC, ROWS + BATCH * PSTEP>(px), ic = px - ir * IC;
            const int ih = ih0 + ir, iw = iw0 + ic;
            const bool ok = px < NPX && ih >= 0 && (unsigned)iw < (unsigned)p.W && whole;      // (rows past the last end the buffer)
            xv[b] = __builtin_amdgcn_raw_buffer_load_b128(xr, ok ? (unsigned)(ih - top) * row_bytes + (unsigned)iw * pixel_bytes + 16u * ch : OOB, 0, 0);
        }
    };
    half_t* const xdst = xs + px0 * XP + ch * 8;
    auto deposit_tile = [&](int it0) __attribute__((always_inline)) {
#pragma unroll
        for (int b = 0; b < BATCH; ++b)
            if (takes && px0 + (it0 + b) * PSTEP < ROWS) *(uintx4*)(xdst + (it0 + b) * PSTEP * XP) = xv[b];
    };
    const half_t lo1 = (p.act1 == ACT_RELU || p.act1 == ACT_RELU6) ? (half_t)0.f : (half_t)-INFINITY;
    const half_t hi1 = p.act1 == ACT_RELU6 ? (half_t)6.f : (half_t)INFINITY;
    const half4 lo4 = {lo1, lo1, lo1, lo1}, hi4 = {hi1, hi1, hi1, hi1};
    const half4 zero4 = {(half_t)0.f, (half_t)0.f, (half_t)0.f, (half_t)0.f};

    if (AHEAD) request_tile((int)blockIdx.x, 0);
    for (int v = (int)blockIdx.x; v < ntiles; v += (int)gridDim.x) {
    int n, P0, Q0;
    tile_of(v, n, P0, Q0);
    const int ih0 = P0 * STRIDE - 1, iw0 = Q0 * STRIDE - 1;
    if (AHEAD) {
        deposit_tile(0);
    } else {
#pragma unroll
        for (int it0 = 0; it0 < NIT; it0 += BATCH) { request_tile(v, it0); deposit_tile(it0); }
    }
    __syncthreads();                                                           // the input tile is in place
    if (AHEAD && v + (int)gridDim.x < ntiles) request_tile(v + (int)gridDim.x, 0);

    for (int g = g_begin; g < g_end; ++g) {
        const int cd = 32 * g + 8 * c8;
        const bool cd_ok = cd < p.Chid;
        // ---- B1: expansion of this group for every pixel of the tile ----------------------------------------------
        for (int blk = wave; blk < NPB; blk += 4) {
            const int px = blk * 32 + l32;
            floatx16 acc;
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[v] = 0.f;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const half8 xf = *(const half8*)(xs + px * XP + 16 * ks + 8 * lh);
                acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(wf[ks], xf, acc, 0, 0, 0);
            }
            const int ir = px / IC, ic = px - ir * IC;
            const bool inside = px < NPX && (unsigned)(ih0 + ir) < (unsigned)p.H && (unsigned)(iw0 + ic) < (unsigned)p.W;
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4) {
                half4 h;
#pragma unroll
                for (int e = 0; e < 4; ++e) h[e] = (half_t)(acc[4 * g4 + e] + bv[g4][e]);
                h = __builtin_elementwise_min(__builtin_elementwise_max(h, lo4), hi4);
                *(half4*)(hs + px * EDW_HP + 8 * g4 + 4 * lh) = inside ? h : zero4;
            }
        }
        const int g_next = g + 1 < g_end ? g + 1 : g_begin;                   // after a tile's last group: the next tile's first
        if (!ONE) {
            load_w1(g_next, wf_next, bv_next);                                // requested while this group goes on
            load_wd(g_next, wv_next, bdv_next);
        }
        lds_barrier();
        // ---- B2: depthwise 3x3 from the expanded tile --------------------------------------------------------------
        {
            float acc[TH][8];
#pragma unroll
            for (int o = 0; o < TH; ++o)
#pragma unroll
                for (int j = 0; j < 8; ++j) acc[o][j] = bdv[j];
            constexpr int RR = (TH - 1) * STRIDE + 3;
#pragma unroll
            for (int rr = 0; rr < RR; ++rr) {
                const int ir = strip * TH * STRIDE + rr;
                if ((unsigned)(ih0 + ir) >= (unsigned)p.H) continue;            // a row of padding adds nothing
                half8 xv[3];
#pragma unroll
                for (int sx = 0; sx < 3; ++sx) xv[sx] = *(const half8*)(hs + (ir * IC + col * STRIDE + sx) * EDW_HP + 8 * c8);
#pragma unroll
                for (int o = 0; o < TH; ++o) {
                    const int fr = rr - o * STRIDE;
                    if (fr < 0 || fr > 2) continue;
#pragma unroll
                    for (int sx = 0; sx < 3; ++sx)
#pragma unroll
                        for (int j = 0; j < 8; ++j) acc[o][j] += (float)xv[sx][j] * (float)wv[fr * 3 + sx][j];
                }
            }
            const int gq = Q0 + col;
#pragma unroll
            for (int o = 0; o < TH; ++o) {
                const int gp = P0 + strip * TH + o;
                if (gp < p.P && gq < p.Q && cd_ok) {
                    half8 ov;
#pragma unroll
                    for (int j = 0; j < 8; ++j) ov[j] = (half_t)edw_act(acc[o][j], p.act2);
                    *(half8*)(p.y + (((long long)n * p.P + gp) * p.Q + gq) * p.Chid + cd) = ov;
                }
            }
        }
        if (ONE) return;
#pragma unroll
        for (int k = 0; k < 9; ++k) wv[k] = wv_next[k];
#pragma unroll
        for (int j = 0; j < 8; ++j) bdv[j] = bdv_next[j];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) wf[ks] = wf_next[ks];
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4)
#pragma unroll
            for (int e = 0; e < 4; ++e) bv[g4][e] = bv_next[g4][e];
        lds_barrier();                                                         // the next group overwrites the expanded tile
    }
    }
}

constexpr unsigned edw_lds_bytes(int ks, int stride, int tq, int th) {
    const int tp = 256 / (4 * tq) * th, ir = (tp - 1) * stride + 3, ic = (tq - 1) * stride + 3, rows = (ir * ic + 31) / 32 * 32;
    return (unsigned)(rows * (ks * 16 + 8 + EDW_HP) * 2);
}

// One way to cut a layer: the tile, and how many groups a workgroup takes.
struct EdwCut {
    int tp, npb, th, lds;                  // output rows, 32-pixel blocks of input, positions per thread, bytes of LDS
    long long tiles;
    int gpb;                               // groups per workgroup (1: the kernel without look-ahead)
    double us;                             // estimate
};
constexpr int edw_pixel_blocks(int stride, int tq, int th) {
    return ((256 / (4 * tq) * th - 1) * stride + 3) * ((tq - 1) * stride + 3) / 32 + ((((256 / (4 * tq) * th - 1) * stride + 3) * ((tq - 1) * stride + 3)) % 32 != 0);
}
constexpr bool edw_ahead(int ks, int stride, int tq, int th) { return (edw_pixel_blocks(stride, tq, th) * 32 + 256 / (2 * ks) - 1) / (256 / (2 * ks)) <= 12; }

// Estimated times, fitted to 15 layers of images of 160, 224 and 256 pixels at 1 to 128 images, every tile and split of them (mean
// error 7 % with one group per workgroup, 18 % with several).  One group: a launch, a pass over the tile, and what the
// workgroups that share a compute unit add, more where LDS does not hold them at once.  Several: every workgroup of a compute unit in turn.
template <int KS, int STRIDE, int TQ, int TH>
static EdwCut edw_cut(const ExpandDwParams& p, bool one) {
    EdwCut c;
    c.th = TH;
    c.tp = 256 / (4 * TQ) * TH;
    c.npb = edw_pixel_blocks(STRIDE, TQ, TH);
    c.lds = (int)edw_lds_bytes(KS, STRIDE, TQ, TH);
    c.tiles = (long long)p.N * ((p.P + c.tp - 1) / c.tp) * ((p.Q + TQ - 1) / TQ);
    const int groups = (p.Chid + 31) / 32, resident = std::min(160 * 1024 / (c.lds + 512), 4);
    c.gpb = 1;
    if (!one) {
        int split = 1;
        while (c.tiles * split < 256 && split * 2 <= groups) split *= 2;
        c.gpb = (groups + split - 1) / split;
        // two full workgroups per compute unit, where they fit and the split comes out even: they hide each other's waits
        const int g2 = (int)((c.tiles * groups + 511) / 512);
        const long long n2 = g2 > 0 && g2 <= groups ? c.tiles * ((groups + g2 - 1) / g2) : 0;
        if (resident >= 2 && n2 >= 448 && n2 <= 512) c.gpb = g2;
    }
    const long long n = c.tiles * ((groups + c.gpb - 1) / c.gpb);
    const double per_cu = (double)((n + 255) / 256);
    if (one) c.us = 3.6 + 0.36 * ((c.npb + 3) / 4) + 0.77 * TH + (per_cu - 1) * (0.044 * c.npb * KS + 0.25 * TH) + 2.2 * (double)((n + 256LL * resident - 1) / (256LL * resident) - 1);
    else c.us = 4.6 + per_cu * (0.10 * c.npb * KS + c.gpb * (0.83 + 0.29 * TH));
    return c;
}

template <int KS, int STRIDE, int TQ, int TH, bool ONE>
static int launch_edw_tile(const ExpandDwParams& q, const EdwCut& c, hipStream_t stream) {
    static_assert(edw_lds_bytes(KS, STRIDE, TQ, TH) <= 160 * 1024, "LDS limit");
    ExpandDwParams p = q;
    p.tiles_p = (p.P + c.tp - 1) / c.tp;
    p.tiles_q = (p.Q + TQ - 1) / TQ;
    p.by_tiles_p = divisor(p.tiles_p); p.by_tiles_q = divisor(p.tiles_q);
    if (c.tiles <= 0 || c.tiles > 0x7fffffffLL) { set_error("expand+depthwise: bad grid (%lld tiles)", c.tiles); return -5; }
    const int groups = (p.Chid + 31) / 32;
    p.groups_per_block = c.gpb;
    const unsigned gy = (unsigned)((groups + c.gpb - 1) / c.gpb);
    auto kernel = expand_dw_kernel<KS, STRIDE, TQ, TH, ONE>;
    static std::atomic<bool> configured{false};
    if (!configured.load(std::memory_order_acquire) && c.lds > 48 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, c.lds);
        if (e != hipSuccess) { set_error("expand+depthwise: cannot reserve %d bytes of LDS: %s", c.lds, hipGetErrorString(e)); return -2; }
    }
    configured.store(true, std::memory_order_release);
    // where the kernel requests a tile's input one tile ahead, two workgroups per compute unit walk over the tiles
    const unsigned gx = (!ONE && edw_ahead(KS, STRIDE, TQ, TH) && c.tiles > 512) ? 512u : (unsigned)c.tiles;
    hipLaunchKernelGGL(kernel, dim3(gx, gy), dim3(256), (unsigned)c.lds, stream, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) { set_error("expand+depthwise launch: %s", hipGetErrorString(e)); return -2; }
    return 0;
}

// The tile TQ x TH with several groups per workgroup, or with one, or one of the two smallest tiles with one: whichever is estimated to
// be the fastest.  With `us`: only its estimate.
template <int KS, int STRIDE, int TQ, int TH>
static int launch_edw_best(const ExpandDwParams& p, hipStream_t stream, double* us) {
    const EdwCut several = edw_cut<KS, STRIDE, TQ, TH>(p, false), one = edw_cut<KS, STRIDE, TQ, TH>(p, true), s8 = edw_cut<KS, STRIDE, 8, 1>(p, true);
    double best = std::min(std::min(several.us, one.us), s8.us);
    if constexpr (edw_lds_bytes(KS, STRIDE, 16, 1) <= 160 * 1024) {
        const EdwCut s16 = edw_cut<KS, STRIDE, 16, 1>(p, true);
        if (us) { *us = std::min(best, s16.us); return 0; }
        if (s16.us < best) return launch_edw_tile<KS, STRIDE, 16, 1, true>(p, s16, stream);
    }
    if (us) { *us = best; return 0; }
    if (best == s8.us) return launch_edw_tile<KS, STRIDE, 8, 1, true>(p, s8, stream);
    if (best == one.us) return launch_edw_tile<KS, STRIDE, TQ, TH, true>(p, one, stream);
    return launch_edw_tile<KS, STRIDE, TQ, TH, false>(p, several, stream);
}

template <int KS>
static int launch_edw_ks(const ExpandDwParams& p, int stride, hipStream_t stream, double* us) {
    // large tile by image width: 32 wide, 16 wide (14 x 14 maps as one tile), 8 wide (7 x 7)
    if (stride == 1) {
        if (p.Q > 16) return launch_edw_best<KS, 1, 32, 4>(p, stream, us);
        if (p.Q > 8) return launch_edw_best<KS, 1, 16, 4>(p, stream, us);
        return launch_edw_best<KS, 1, 8, 1>(p, stream, us);
    }
    // stride 2 puts four input pixels under an output: with many input channels only the smallest tile fits LDS
    // (two workgroups per compute unit matter more than a tile's ratio of rim to area: half the height where the taller tile
    // would take more than half of LDS)
    if constexpr (edw_lds_bytes(KS, 2, 32, 2) <= 80 * 1024) {
        if (p.Q > 16) return launch_edw_best<KS, 2, 32, 2>(p, stream, us);
    } else if constexpr (edw_lds_bytes(KS, 2, 32, 1) <= 160 * 1024) {
        if (p.Q > 16) return launch_edw_best<KS, 2, 32, 1>(p, stream, us);
    }
    if constexpr (edw_lds_bytes(KS, 2, 16, 2) <= 80 * 1024) {
        if (p.Q > 8) return launch_edw_best<KS, 2, 16, 2>(p, stream, us);
    } else if constexpr (edw_lds_bytes(KS, 2, 16, 1) <= 160 * 1024) {
        if (p.Q > 8) return launch_edw_best<KS, 2, 16, 1>(p, stream, us);
    }
    return launch_edw_best<KS, 2, 8, 1>(p, stream, us);
}

static int launch_edw(const ExpandDwParams& p, int stride, hipStream_t stream, double* us) {
    const int ks = (p.Cin + 15) / 16;
    if (ks <= 1) return launch_edw_ks<1>(p, stride, stream, us);
    if (ks <= 2) return launch_edw_ks<2>(p, stride, stream, us);
    if (ks <= 4) return launch_edw_ks<4>(p, stride, stream, us);
    if (ks <= 6) return launch_edw_ks<6>(p, stride, stream, us);
    return launch_edw_ks<10>(p, stride, stream, us);
}

bool expand_dw_supported(int Cin, int Chid, int stride) {
    return Cin >= 8 && Cin % 8 == 0 && Cin <= 160 && Chid >= 8 && Chid % 8 == 0 && (stride == 1 || stride == 2);
}

// One launch or two: the estimate above against that of the 1x1 and the depthwise launch, 8.2 us for the pair and its bytes (the
// expanded tensor written and read, the output written) at 5.6 TB/s, 2.6 TB/s past the 250 MB that stay in the memory-side cache.
// Measured on the served network's nine layers at image sides 160 and 224 and 8 to 128 images, one launch / two in us:
// 224, 16 images: 56x56x24>144 20.8 / 17.8, stride 2 11.6 / 13.3, 28x28x32>192 9.3 / 11.1, 14x14x64>384 7.8 / 10.6, 7x7x160>960 7.6 /
// 10.0; 64 images: 54.5 / 41.2, 31.7 / 32.9, 20.3 / 19.7, 17.8 / 14.5, 27.0 / 14.4; 112x112x16>96 stride 2 18.1 / 24.8 at 16 images,
// 94 / 191 at 128.  Over these 162 the two-launch estimate is 8 % off on average, the choice costs 0.4 % of the sum of the better times
// (always two launches: 17 %).  The one-launch estimate knows nothing of memory's rate, so where two launches take more than
// 25 us only the layer whose expanded tensor dwarfs its input, at stride 2 its output too, is computed in one.
bool expand_dw_pays(int N, int H, int W, int Cin, int Chid, int stride) {
    if (N <= 0 || H <= 0 || W <= 0 || !expand_dw_supported(Cin, Chid, stride)) return false;
    ExpandDwParams p{};
    p.N = N; p.H = H; p.W = W; p.Cin = Cin; p.Chid = Chid;
    p.P = (H - 1) / stride + 1; p.Q = (W - 1) / stride + 1;
    const double mb = 2e-6 * N * Chid * (2.0 * H * W + (double)p.P * p.Q);
    const double two = 8.2 + mb / 5.6 + std::max(0.0, mb - 250) / 9;
    if (two > 25 && !(stride == 2 && Cin <= 16)) return false;
    double one = 0;
    (void)launch_edw(p, stride, nullptr, &one);
    return one < 0.95 * two;
}

int launch_expand_dw(const half_t* x, int N, int H, int W, int Cin, const half_t* w1, int ldw1, const float* b1, int Chid, int act1,
                     const half_t* wd_rsc, const float* bd, int stride, int act2, half_t* y, int hp, hipStream_t stream) {
    if (!x || !w1 || !wd_rsc || !y || N <= 0 || H <= 0 || W <= 0 || !expand_dw_supported(Cin, Chid, stride) || ldw1 < Cin || ldw1 % 8 != 0 ||
        act1 == ACT_GELU || act2 == ACT_GELU) {
        set_error("expand+depthwise: needs 8 to 160 input channels and a number of expanded channels that are multiples of 8, stride 1 or 2");
        return -5;
    }
    if ((reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(w1) | reinterpret_cast<uintptr_t>(wd_rsc) | reinterpret_cast<uintptr_t>(y) |
         reinterpret_cast<uintptr_t>(b1) | reinterpret_cast<uintptr_t>(bd)) & 15) {
        set_error("expand+depthwise: pointers must be 16-byte aligned"); return -1;
    }
    ExpandDwParams p{};
    p.x = x; p.N = N; p.H = H; p.W = W; p.Cin = Cin;
    p.w1 = w1; p.ldw1 = ldw1; p.b1 = b1; p.Chid = Chid; p.act1 = act1;
    p.wd = wd_rsc; p.bd = bd; p.act2 = act2; p.y = y; p.hp = hp;
    p.P = (H - 1) / stride + 1; p.Q = (W - 1) / stride + 1;      // 3x3, padding 1
    p.wide = 18LL * W * Cin * 2 > 0x7fffffffLL;
    return launch_edw(p, stride, stream, nullptr);
}

}  // namespace strait
