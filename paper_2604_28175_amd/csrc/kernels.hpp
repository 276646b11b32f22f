// Internal launcher interface between the runtime and the gfx950 kernels.
// Every launcher validates the operand shapes its kernel and grid assume and returns a
// negative status (see strait.h) instead of launching when they do not hold.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace strait {

typedef _Float16 half_t;

enum Act { ACT_NONE = 0, ACT_RELU = 1, ACT_RELU6 = 2, ACT_GELU = 3 };

// Division by a number that is the same for a whole launch, prepared on the host: n / d = floor(2 n mul / 2^32) >> shift, exact for 0 <= n < 2^31 and
// 1 <= d < 2^31 (shift = ceil(log2 d), mul = floor(2^(31 + shift) / d) + 1: the error, less than 2 n d / 2^(32 + shift) <= n / 2^31 of one, reaches no next
// quotient); by more it is 0.  A division by an unknown number is 30 to 40 instructions that depend on each other, at one wavefront per SIMD 100 ns; a launch of a
// small batch, 4 to 6 us long, began with four to eleven of them.
struct Divisor { unsigned mul, shift; };
inline Divisor divisor(long long d) {
    Divisor r{1u, 0u};
    if (d < 1) return r;
    if (d > 0x7fffffffLL) return {0u, 0u};
    while ((1LL << r.shift) < d) ++r.shift;
    r.mul = (unsigned)((1ULL << (31 + r.shift)) / (unsigned long long)d + 1);
    return r;
}
#ifdef __HIPCC__
__host__ __device__
#endif
inline int divide(int n, Divisor d) { return (int)((unsigned)(((unsigned long long)((unsigned)n << 1) * d.mul) >> 32) >> d.shift); }
// Tiles are numbered down groups of cw tile columns (row-major inside a group), so that the contiguous range an XCD gets covers a rectangle of about equal
// extent in pixels and channels: its L2 then fetches the fewest operand rows.  Of `full` whole groups and one of the `last` columns.
struct TileOrder { int tiles, cw, full, last, group; Divisor by_tiles, by_group, by_cw, by_last; };   // group: tiles of a whole one

// One implicit-GEMM convolution (or plain GEMM) launch.
//   y[m, k] = act(bias[k] + sum_{r,s,c} x[addr(m) + r*sH + s*sW + c] * w[k*ldw + (r*S + s)*C + c] (+ res[m*ldy + k]))
// with m = (n, p, q), addr(m) = n*sN + (p*stride - pad)*sH + (q*stride_w - pad_w)*sW, taps outside
// [0,H) x [0,W) contributing zero.  A plain NHWC convolution has sW = C, sH = W*C, sN = H*W*C;
// the decoupled strides also describe a channel-padded, spatially pre-padded stem input whose
// taps along a row are contiguous ("virtual" 1-wide kernel with C = taps*Cpad).
struct ConvParams {
    const half_t* x;
    const half_t* w;
    const float* bias;       // [Cout] or nullptr
    const half_t* res;       // [M][ldy] or nullptr
    void* y;                 // fp16 (or fp32 when out_f32) [M][ldy]
    int M;                   // N * P * Q
    int PQ, Q;
    int H, W, C, R, S;
    int stride_h, stride_w, pad_h, pad_w;
    long long sN;
    int sH, sW;
    int Kg;                  // R * S * C
    int ldw;                 // weight row pitch in elements (multiple of 8, zero padded past Kg)
    int Cout, ldy;
    int act;
    int out_f32;
    int hp;                  // raise wave priority (high-priority batch)
    long long x_elems;       // extent of x in elements; filled in by launch_conv
    float* ws;               // optional split-K workspace (16-byte aligned) and its size in bytes
    size_t ws_bytes;
    int ksplit;              // filled in by launch_conv
    int res_f32;             // add the residual in fp32, before the rounding; filled in by launch_conv
    int whole_M;             // of rows that are a part of a larger launch's: the number of all of them, whose order of summation they get (0: M)
    TileOrder order;         // filled in by the launcher (set_tile_order), like the divisors and kchunk
    Divisor by_pq, by_q, by_c, by_s, by_row, by_image;   // PQ, Q, C, S; W + 1 and (H + 1)(W + 1), the pixels of a bordered row and image
    int kchunk;              // slices of a part of the reduction
    int strip_w, strips;     // 3x3 patch kernel: width and number of the strips a row is cut into; filled in by the launcher
    Divisor by_strips;
    // Optional second source of a 1x1 convolution with stride 1 (a block-closing convolution that absorbs the block's 1x1
    // projection shortcut): reduction elements [C, C + K2) are x2[n*sN2 + p*stride2*sH2 + q*stride2*sW2 + (k - C)], and
    // w is [Cout][C + K2].  Kg = C + K2; no res.
    const half_t* x2;
    int K2, stride2, sH2, sW2;
    long long sN2;
    long long x2_elems;      // extent of x2 in elements; filled in by launch_conv
    // A LayerNorm folded into the products on its two sides (launch_gemm_ln only).  Statistics of a tensor [M][n], n a multiple of 64: for each
    // row and 64 channels {sum, sum of squares about their own mean}, [M][n / 64]; 16-byte aligned.
    const float2* ln_stats;  // of the input (with ln_csum) or of the residual (with ln_g, ln_b), which is then normalised
    const float* ln_csum;    // [Cout] sums of the rows of w, which holds gamma; bias holds w beta
    const float* ln_g; const float* ln_b;    // [Cout]
    float ln_eps, ln_inv_n;  // (ln_inv_n filled in by launch_gemm_ln)
    float2* stats_out;       // of the output
    // Between two such products a tensor [M][n] may lie in slices of 64 channels, [n / 64][M][64]: what a tile reads of a slice is then one piece of
    // memory and not a row every 2 n bytes.
    int x_sliced, y_sliced;
    unsigned x_slice;        // bytes from one slice of the input to the next; filled in by launch_gemm_ln
};

int launch_conv(const ConvParams& p, hipStream_t stream);
const char* conv_kernel_name(const ConvParams& p);     // of the kernel and tile that launch_conv takes; null where it refuses the layer
// Bytes of workspace (ConvParams::ws), at most `limit`, with which launch_conv splits this layer's reduction into slabs; 0 = it uses none.
size_t conv_workspace_bytes(const ConvParams& p, size_t limit);
// Small outputs with a reduction worth sharing out (conv_skinny.hip): 16 pixels x tn (16 or 32) channels per workgroup.  Called by
// launch_conv with x_elems filled in; C and Kg multiples of 64.
int launch_conv_skinny(const ConvParams& p, int tn, bool gather, hipStream_t stream);
// 3x3 with stride 1 and padding 1 on small images (conv3x3_small.hip), bm bordered pixels x bn channels per workgroup; called by launch_conv with x_elems
// filled in.  No residual; C a multiple of 64.
bool conv3x3_small_takes(const ConvParams& p, int bm, int bn);
int launch_conv3x3_small(const ConvParams& p, int bm, int bn, hipStream_t stream);
// Larger ones, bm (96 or 192) bordered pixels x 128 channels per workgroup (conv3x3_mid.hip); likewise.
bool conv3x3_mid_takes(const ConvParams& p, int bm);
int launch_conv3x3_mid(const ConvParams& p, int bm, hipStream_t stream);
// The order of tiles_m x tiles_n tiles, whose operands are bm input rows and bn weight rows, and the divisors; bk: elements of a slice, parts: of the reduction
void set_tile_order(ConvParams& p, long long tiles_m, int tiles_n, int bm, int bn, int bk, int parts);

// A dense product with a LayerNorm folded in (gemm_ln.hip): of its input (ln_stats, ln_csum; no residual), or its output's statistics for one that
// follows (stats_out; with a residual, normalised where ln_stats, ln_g and ln_b are given).
int launch_gemm_ln(const ConvParams& p, hipStream_t stream);
// whether launch_gemm_ln takes M x N x K products whose normalised width is `width`
bool gemm_ln_supported(long long M, long long N, long long K, int width);
bool gemm_ln_pays(long long rows, int width);          // whether folding is no slower than a LayerNorm launch between the products
// w [N][K], b [N] and the LayerNorm's gamma, beta [K] -> fp16(gamma w), its row sums, b + w beta; *bad, if given, becomes 1 where
// gamma w does not keep fp16's precision (gemm_ln.hip), and is left alone otherwise
int launch_fold_layernorm(const half_t* w, const float* b, const float* gamma, const float* beta, int N, int K, half_t* w_out, float* csum, float* b_out,
                          int* bad, hipStream_t stream);
int choose_gemm_ln(ConvParams& p);                     // >= 0 a tile (conv_dma.hpp: TileId); < 0 an error

// Two chained pointwise convolutions in one launch (pointwise_pair.hip):
//   y[m, 0:N1] = act1(x[m, 0:K1] w3^T + b3 (+ res[m, 0:N1]));   z[m, 0:N2] = act2(y[m, 0:N1] w1^T + b1)
// x [M][K1], w3 [N1][K1], res and y [M][N1], w1 [N2][N1], z [M][N2], all dense fp16; biases fp32 or nullptr.
// z must not share memory with x or res (other workgroups may still be reading them).
// With x2 (a second input [M][K2], for a block whose shortcut is a 1x1 projection of x2) the first product is
// [x | x2] w3^T with w3 [N1][K1 + K2], and there is no res.
struct PairParams {
    const half_t* x; const half_t* w3; const float* b3; const half_t* res; half_t* y;
    const half_t* w1; const float* b1; half_t* z;
    int M, K1, N1, N2, act1, act2, hp;
    const half_t* x2; int K2;
};
bool pointwise_pair_supported(int K1, int N1, int N2);
bool pointwise_pair_proj_supported(int K1, int K2, int N1, int N2);
int launch_pointwise_pair(const PairParams& p, hipStream_t stream);

int launch_pack_input(const half_t* x, int N, int H, int W, int C, half_t* y, int Hp, int Wp, int Cpad,
                      int pad_top, int pad_left, int hp, hipStream_t stream);
// 7x7 stride-2 pad-3 convolution of a 3-channel image to 64 channels + bias + ReLU + 3x3 stride-2 pad-1 max pooling.
// wf: [64][176] fp16, row k = 22 fragments of 8: fragment 3r + j holds halfs 8j..8j+7 of filter row r's 24-half window
// {0, w[k][r][s=0][c=0..2], ..., w[k][r][6][0..2], 0, 0}; the 22nd fragment is zero.  W even.
// w1 [64][64] fp16, b1 [64] fp32 or nullptr, t1 like y: optionally also t1 = relu(y w1^T + b1), the 1x1 convolution behind it
int launch_stem_pool(const half_t* x, const half_t* wf, const float* bias, int N, int H, int W, half_t* y, int hp,
                     hipStream_t stream, const half_t* w1 = nullptr, const float* b1 = nullptr, half_t* t1 = nullptr);
// 3x3 stride-2 pad-1 convolution of a 3-channel image to Kout <= 32 channels + bias + activation (stem3x3.hip).
// wf: [32][48] fp16, row k = 3 filter rows x 16 halfs {0, w[k][r][s=0][c=0..2], w[k][r][1][..], w[k][r][2][..], 0 x 6}; rows
// from Kout on zero.  W even, Kout a multiple of 8.
int launch_stem3x3s2(const half_t* x, const half_t* wf, const float* bias, int N, int H, int W, int Kout, int act, half_t* y, int hp,
                     hipStream_t stream);
// 3x3 stride-1 pad-1 convolution of a 3-channel image to 16, 32 or 64 channels + bias + activation (stem3x3.hip), W even.  wf: [Kout rounded up to 32]
// [2][3][16]: per channel, for even and for odd columns, three filter rows of 9 halfs {w[k][r][s][c]}, at 1 .. 9 and at 0 .. 8; the rest zero.
bool stem3x3s1_supported(int W, int Kout, int act);
bool stem3x3s1_pays(int N, int H, int W);              // whether it is estimated to be no slower than the packing launch and the product
int launch_stem3x3s1(const half_t* x, const half_t* wf, const float* bias, int N, int H, int W, int Kout, int act, half_t* y, int hp,
                     hipStream_t stream);
// The stride-2 stem (32 output channels) with a stride-1 depthwise 3x3 behind it (wd_rsc [3][3][32], + bd, act2) in one launch;
// y [N,P,Q,32].  Bit-identical to launch_stem3x3s2 followed by launch_dwconv3x3.
int launch_stem3x3s2_dw(const half_t* x, const half_t* wf, const float* bias, int act1, const half_t* wd_rsc, const float* bd, int act2,
                        int N, int H, int W, half_t* y, int hp, hipStream_t stream);
// 1x1 convolution Cin -> Chid (+ b1, act1) and the depthwise 3x3 of stride 1 or 2, padding 1, behind it (+ bd, act2) in one
// launch (expand_dw.hip): x [N,H,W,Cin] -> y [N,P,Q,Chid]; w1 [Chid][ldw1], wd_rsc [3][3][Chid].  Bit-identical to the two
// launches.  expand_dw_supported: whether the kernel takes these channel counts and this stride;
// expand_dw_pays: whether it does and is estimated to be faster than the two launches.
bool expand_dw_supported(int Cin, int Chid, int stride);
bool expand_dw_pays(int N, int H, int W, int Cin, int Chid, int stride);
int launch_expand_dw(const half_t* x, int N, int H, int W, int Cin, const half_t* w1, int ldw1, const float* b1, int Chid, int act1,
                     const half_t* wd_rsc, const float* bd, int stride, int act2, half_t* y, int hp, hipStream_t stream);
int launch_dwconv3x3(const half_t* x, int N, int H, int W, int C, const half_t* w_rsc, const float* bias,
                     int stride, int act, half_t* y, int hp, hipStream_t stream);
int launch_maxpool3x3s2(const half_t* x, int N, int H, int W, int C, half_t* y, int hp, hipStream_t stream);
int launch_maxpool2x2s2(const half_t* x, int N, int H, int W, int C, half_t* y, int hp, hipStream_t stream);
int launch_vit_tokens(const half_t* patch, const float* cls, const float* pos, int N, int T, int D, half_t* z, int hp,
                      hipStream_t stream);
int launch_global_avgpool(const half_t* x, int N, int HW, int C, half_t* y, int hp, hipStream_t stream);
int launch_softmax_top1(const float* logits, int rows, int n, float* probs, int32_t* top1, int hp,
                        hipStream_t stream);
// x_row_stride: elements between consecutive input rows (0 = n); the output rows are contiguous.
int launch_layernorm(const half_t* x, const float* gamma, const float* beta, int rows, int n, float eps,
                     half_t* y, int hp, hipStream_t stream, long long x_row_stride = 0);
int launch_attention(const half_t* qkv, const int32_t* valid_len, int B, int S, int heads, half_t* out, int hp,
                     hipStream_t stream);
int launch_argmax_f16(const half_t* x, int rows, int n, long long row_stride, int32_t* top1, int hp,
                      hipStream_t stream);
// Weight preparation on the device (load time): BatchNorm fold + OIHW -> kernel layout.
int launch_fill_zero(void* p, size_t bytes, hipStream_t stream);
// ---- transfers by kernel, with the timestamps and the completion flags of a batch (elementwise.hip)
// STAMP_PIECES + 2 i, + 2 i + 1: start and end of the i-th piece of an input that goes in by kernel; of one that copy engines bring, the
// first pair holds its start and end, STAMP_LAST the start of a last piece that follows another batch's
enum { STAMP_K0 = 0, STAMP_K1 = 1, STAMP_D2H0 = 2, STAMP_DONE = 3, STAMP_LAST = 4, STAMP_PIECES = 8, MAX_PIECES = 32, STAMP_COUNT = STAMP_PIECES + 2 * MAX_PIECES };
constexpr unsigned OUT_PARTS = 8, OUT_MAX_CHUNKS = 4096;
inline size_t out_chunk_bytes(size_t bytes) {          // of a result: 256 KB, doubled while it has more chunks than there are flags (beyond 1 GiB)
    size_t c = 256u << 10;
    while ((bytes + c - 1) / c > OUT_MAX_CHUNKS) c *= 2;
    return c;
}
struct HostControl {                     // in pinned host memory, written by the GPU
    uint64_t stamp[STAMP_COUNT];         // device clock (hipDeviceAttributeWallClockRate)
    uint32_t k1_seq, pad[7];             // sequence number of the last batch whose kernels are done (results that leave on a copy stream)
    uint32_t flag[OUT_MAX_CHUNKS];       // ... of the last batch whose chunk of the result has arrived
};
// counters: one unsigned (copy in), 1 + OUT_MAX_CHUNKS of them (copy out), in device memory, zero before the first launch and after each
int launch_copy_in(const void* src, void* dst, size_t bytes, const void* src2, void* dst2, size_t bytes2, HostControl* ctl, unsigned* counters,
                   int piece, hipStream_t stream);
int launch_stamp(HostControl* ctl, int which, hipStream_t stream, const void* src = nullptr, void* dst = nullptr, size_t bytes = 0, unsigned seq = 0);
// The end of a classifier's batch (classify_out.hip): softmax and top-1 of `rows` samples' logits, and logits, probabilities and indices both to their
// places on the device and to host memory; stamps and flag as launch_copy_out.  With x, a feature map [rows][HW][C], first the logits: its mean over
// the HW positions, rounded to fp16, times w [n][ldw], + bias.  Results of one chunk (classify_out_takes), small heads (classify_out_pools).
struct ClassifyOut {
    const half_t* x; int HW, C;
    const half_t* w; int ldw; const float* bias;
    float* logits; float* probs; int32_t* top1;
    int rows, n;
    char* host; HostControl* ctl; unsigned* counter;   // counter: launch_copy_out's, 33 lines of 32 from the first
    unsigned seq;
    int hp;
};
bool classify_out_takes(long long rows, int n);
bool classify_out_pools(int HW, int C, int n);
int launch_classify_out(const ClassifyOut& p, hipStream_t stream);
// beside: another stream has a batch, whose launches this one's requests hold up
int launch_copy_out(const void* src, void* dst, size_t bytes, HostControl* ctl, unsigned* counters, unsigned seq, bool k1_taken, int hp, bool beside, hipStream_t stream);

void set_error(const char* fmt, ...);

}  // namespace strait
