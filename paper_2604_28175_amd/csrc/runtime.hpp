// Host-side runtime: weight container, BatchNorm fold and re-layout, per-architecture layer
// plans, model instances with pinned staging, dual-priority dispatch and completion records.
#pragma once
#include <hip/hip_runtime.h>

#include <atomic>
#include <condition_variable>
#include <deque>
#include <map>
#include <mutex>
#include <set>
#include <string>
#include <thread>
#include <vector>

#include "../../include/strait.h"
#include "kernels.hpp"

namespace strait {

enum OpKind { OP_CONV = 0, OP_DWCONV = 1, OP_POOL = 2, OP_SOFTMAX = 3, OP_LAYERNORM = 4, OP_ATTENTION = 5, OP_PACK = 6, OP_TOKENS = 7, OP_STEMPOOL = 8, OP_STEM3 = 9 };
enum PoolKind { POOL_MAX3X3S2 = 0, POOL_GLOBAL_AVG = 1, POOL_ARGMAX = 2, POOL_MAX2X2S2 = 3 };

// Where an operand lives.  Slots >= 0 index the instance's activation buffers; the input and
// output slots are the instance's device input / output buffers (output at a byte offset that
// depends on the batch size).
enum { SLOT_NONE = -1, SLOT_INPUT = -2, SLOT_OUT = -3 };

struct OutRef { int kind = 0; };   // 0: start of output buffer, 1: after logits (probs), 2: after logits+probs (top1), 3: after hidden states

struct Op {
    std::string name;
    int kind = OP_CONV;
    int sub = 0;                      // PoolKind for OP_POOL
    int in = SLOT_NONE, out = SLOT_NONE, res = SLOT_NONE;
    int out_ref = 0, out_ref2 = 0;    // which region of the output buffer (when out == SLOT_OUT)
    // geometry per sample
    int H = 1, W = 1, C = 1;          // input
    int P = 1, Q = 1, K = 1;          // output
    int R = 1, S = 1, stride = 1, pad = 0, act = 0;
    int out_f32 = 0;
    // Independent branch: `side` ops run on the instance's side stream, forked off the main stream right
    // before them; the first later op with `join` set waits for the side stream before it is launched.
    int side = 0, join = 0;
    // A block-closing pointwise convolution whose output feeds the pointwise convolution `pair` ops further on (0 = none):
    // at large batches the two run as one launch (pointwise_pair.hip) and the second op is skipped.
    int pair = 0;
    // Such a pair in a block whose shortcut is a 1x1 projection of the block input with the block's own stride 1: the
    // projection can join the closing convolution's reduction (w_proj = [w | projection's w], bias_proj = the two biases
    // added), and the projection's own launch is skipped.  proj_down: on the closing convolution, the index of the
    // projection op; proj_of: on the projection op, the index of the closing convolution (-1 = none).
    int proj_down = -1, proj_of = -1;
    // on the fused stem: the index of the 1x1 convolution (64 -> 64, ReLU) that reads nothing but its output and can run inside it
    int stem_next = -1;
    // on a 1x1 expansion or the 3x3/2 stem: the next op is the depthwise 3x3 that alone reads its output, and both can run as one launch
    bool dw_next = false;
    const half_t* w_proj = nullptr;
    const float* bias_proj = nullptr;
    // A LayerNorm between token-wise products can be folded into them (gemm_ln.hip).  On the LayerNorm: fold_ops, the products concerned (before it;
    // behind it, reading its output; reading it as a residual, or -1), and ln_slot, the instance's statistics buffer it takes.  On those products
    // its index, as ln_out, ln_in, ln_res.  w_ln, bias_ln, csum_ln: the weights of an ln_in product with gamma, beta and the row sums in them.
    int fold_ops[3] = {-1, -1, -1};
    int ln_slot = 0, ln_out = -1, ln_in = -1, ln_res = -1;
    const half_t* w_ln = nullptr;
    const float *bias_ln = nullptr, *csum_ln = nullptr;
    // implicit-GEMM addressing (elements), see ConvParams
    long long sN = 0; int sH = 0, sW = 0, stride_w = 1, pad_h = 0, pad_w = 0, vC = 0, vR = 0, vS = 0, vH = 0, vW = 0;
    int ldw = 0;
    // pack
    int Hp = 0, Wp = 0, Cpad = 0;
    // attention / layernorm
    int seq = 0, heads = 0;
    float eps = 0.f;
    long long in_row_stride = 0;      // LayerNorm: elements between input rows (0 = contiguous)
    const half_t* w = nullptr;        // (OP_PACK: of the stem behind it, where that can read the image itself)
    const float* bias = nullptr;      // conv/gemm bias, LayerNorm gamma, class token (OP_TOKENS)
    const float* beta = nullptr;      // LayerNorm beta, position embeddings (OP_TOKENS)
    strait_layer_info info{};
};

struct Instance {
    void* pinned_in = nullptr;
    void* pinned_in_dev = nullptr;     // the same memory as the GPU addresses it
    void* pinned_out = nullptr;
    void* pinned_out_dev = nullptr;    // the same memory as the GPU addresses it
    void* dev_in = nullptr;
    void* dev_out = nullptr;
    int32_t* dev_valid = nullptr;
    float* splitk_ws = nullptr;        // fp32 slabs of split-K convolutions (small batches)
    bool ln_fold = true;               // whether the batch in flight was begun with LayerNorms folded
    float2* ln_stats[2] = {nullptr, nullptr};   // statistics of the tensors that a folded LayerNorm normalises; consecutive ones alternate
    std::vector<void*> bufs;
    HostControl* ctl = nullptr;        // pinned: timestamps and completion flags of the batch in flight, written by the GPU
    HostControl* ctl_dev = nullptr;    // the same memory as the GPU addresses it
    unsigned* counters = nullptr;      // device: [0] copy in, [1 ..] copy out (see kernels.hpp)
    unsigned seq = 0;                  // sequence number of the batch in flight: what its completion flags will read
    hipEvent_t ev_h2d = nullptr;       // input on the device, where a copy stream brings it
    hipEvent_t ev_seg[2] = {nullptr, nullptr};   // ends of the two plan segments a yielding low-priority batch has in flight
    hipStream_t side = nullptr;        // default priority, non-blocking: carries branches that do not depend on each other
    hipEvent_t ev_fork = nullptr, ev_join = nullptr;
    std::vector<hipEvent_t> layer_ev;
    std::vector<char> layer_skipped;    // by the last timed run: layers that were computed inside another layer's launch
    // Captured kernel sequences, keyed by (batch, wave-priority flag + 2 where the last layers are left to the result's way out); a key is captured on its second
    // use, after one eager pass has set the kernels' attributes outside of any capture.
    std::map<std::pair<int, int>, hipGraphExec_t> graphs;
    std::set<std::pair<int, int>> warmed;
    bool busy = false;
};

constexpr size_t SPLITK_WS_BYTES = 16u << 20;

struct Context;

struct Model {
    Context* ctx = nullptr;
    int id = 0;
    int arch = 0;
    int hyper[8] = {0};
    int max_batch = 0;
    std::vector<Op> ops;
    std::vector<char> cuts;            // [i]: 0, or that a batch can be computed part by part up to layer i, in parts that begin at a multiple of so many samples (plan_parts)
    std::vector<size_t> buf_elems;     // per-sample elements of each activation buffer
    size_t in_elems = 0;               // per-sample fp16 input elements
    int classes = 0;                   // CNN
    int seq = 0, hidden = 0;           // encoder, Vision Transformer
    bool fold_layernorms = true;       // false: no LayerNorm is to be folded, for want of the memory that a second set of weights takes
    int ln_folds = 0;                  // LayerNorms that can be folded into products
    // Weights of products that a folded LayerNorm replaces, on the host until everything that a batch does read has its place (finish_plan): what a
    // batch reads then lies together and in the 256 MB memory-side cache.  (ViT batch 7, products of 3072 inputs: 23.6 us a launch, with
    // 100 MB of such weights in between, against 19.6.)
    struct Cold { size_t op; std::vector<half_t> w; std::vector<float> b; };
    std::vector<Cold> cold;
    void* fold_tmp = nullptr;          // device memory the fold reads them from
    size_t fold_tmp_bytes = 0;
    std::vector<void*> dev_allocs;     // weights
    std::vector<Instance> inst;
    std::mutex mu;
    int in_flight = 0;

    size_t in_bytes(int b) const { return (size_t)b * in_elems * 2; }
    size_t out_bytes(int b) const;
    size_t out_offset(int ref, int b) const;
};

// What the time on the link of one batch's input is found from, besides its stamps.
struct InputTiming {
    bool by_kernel = false;            // every piece has its start and end; else (copy engine) the whole has
    int pieces = 0;
    int64_t handed[MAX_PIECES];        // host time at which each was enqueued
    size_t bytes[MAX_PIECES];
    bool last_timed = false;           // STAMP_LAST is set: another batch's transfers came between these pieces
};

struct Ticket {
    Model* model = nullptr;
    int instance = 0, prio = 0, batch = 0;
    void* host_out = nullptr;
    strait_record rec{};
    std::atomic<bool> done{false};
    int status = 0;
    bool deferred = false;             // kernels not enqueued yet: the stream's worker issues them segment by segment
    bool k0_stamped = false;           // kernel start has a stamp of its own (else it is the end of the input copy)
    unsigned seq = 0;
    InputTiming input;
    int copies = 0;                    // copy streams that bring its input, from `copy` on (Context::copy_outstanding); 2: in parts
    size_t worker = 0;                 // index of its compute stream in Context::workers
    size_t copy = 0;                   // index of its copy stream in Context::copy
    unsigned chunks = 0;               // of its result
    size_t chunk_bytes = 0;
    std::atomic<unsigned> chunk_next{0}, chunk_done{0};   // handed out to a copying thread / copied to the caller's buffer
    std::atomic<bool> chunks_coming{false};               // the copy off the device is enqueued: another thread may lend a hand
    std::atomic<int64_t> t_last{0};    // host time at which the last chunk was seen to be there
    std::atomic<int> copy_status{0};
    int out_first = 0;                 // first op that the launch behind its kernel sequence computes; the number of ops: none
    bool out_pending = false;          // large result: its copy is enqueued when the kernels are seen done
    int hp = 0;                        // wave-priority flag its kernels are launched with
};

struct StreamWorker {
    hipStream_t stream = nullptr;
    std::thread th;
    std::deque<Ticket*> q;
    std::atomic<int> outstanding{0};   // batches submitted to this stream whose result has not arrived
};

struct Context {
    int device = 0;
    std::vector<hipStream_t> hp, lp, copy;
    std::vector<StreamWorker*> workers;     // one per compute stream: hp first, then lp
    // A batch's kernels and result copy are enqueued under their stream's mutex, so that batches submitted from several threads do
    // not interleave there.  Inputs may, piece by piece (an input that is staged by the caller, or small, is one piece): a
    // high-priority input then waits for the rest of a piece, not for the rest of a low-priority batch that its caller is still
    // copying.  A record holds its own batch's time on the link only (InputTiming).
    std::deque<std::mutex> compute_mu, copy_mu;
    std::vector<unsigned> copy_seq;         // per copy stream, under its mutex: transfers enqueued so far
    std::deque<std::atomic<int>> copy_outstanding;   // per copy stream: batches whose input it brings and whose result has not arrived
    std::mutex mu;                          // guards worker queues, ticket completion, counters
    std::condition_variable cv_work, cv_done;
    bool stop = false;
    double ms_per_tick = 1e-5;              // of the device clock the stamps are taken from
    bool wave_priority = true;
    bool use_graphs = false;
    long long proj_min_pixels = 1;          // the same for pairs that absorb a projection shortcut: three launches become one
    long long pair_min_pixels = 40000;      // from this many output pixels on, marked pairs of pointwise convolutions run as one launch (0 = never)
    int lp_yield_layers = 0;                // > 0: low-priority batches are issued in segments of this many layers and yield between them
    std::atomic<int> low_in_parts{0};       // low-priority batches whose input came in parts, over two copy streams, and whose result has not arrived
    std::atomic<int> hp_in_flight{0};       // high-priority batches submitted and not yet complete
    bool branch_streams = true;             // independent branches of a plan go to the instance's side stream
    size_t h2d_kernel_limit = 8u << 20;   // inputs up to this size go in by a copy kernel, larger ones by hipMemcpyAsync
    unsigned n_hp_sub = 0, n_lp_sub = 0, n_copy_sub = 0;
    int n_models = 0, next_model_id = 0;
};

int build_plan(Model& m, const void* blob, size_t bytes);
int finish_plan(Model& m);             // after the instances' buffers
// Enqueues layers first_layer..last_layer (last_layer < 0: up to the end) of the plan for `batch` samples on `stream`.
// read_last: the output of last_layer is going to be read by the caller (a layer folded or laid out for the next one is then computed as it is).
// base, whole_batch: the samples are those from `base` on of a batch of whole_batch whose first layers are computed part by part (layers 0..Parts::layers - 1),
// or, with first_layer > 0, all of it, for which that is done.
int run_plan(Model& m, Instance& in, int batch, hipStream_t stream, int hp, int last_layer, bool timed, int first_layer = 0, bool read_last = false, int base = 0, int whole_batch = 0);
// The parts that a large batch's input comes in, and the number of layers that are computed for each as soon as it is there, while the next one is on the link: as many
// as take no longer than that does, by the estimate of a launch's 4 us and a rate (0.8 PFLOP/s, 4.5 TB/s) for each, fewer than `last`,
// and as can be computed so.  The first part is half as large as the others, the last one what is left; all begin where the kernels can read and write 16 bytes at a time.
struct Parts { int layers = 0, first = 0, each = 0; };     // layers 0: in one piece
Parts plan_parts(const Model& m, int batch, int last);
// The first op of those that enqueue_classify_out computes on the result's way out; the number of ops where it computes none, as in
// the layer-by-layer plan (strait_ctx_set_pair_fusion).  Asked once per batch (Ticket::out_first), so that its sequence, also one in segments or a captured
// one, ends where the launch behind it begins.
int classify_out_first(const Model& m, int batch);
int enqueue_classify_out(Model& m, Instance& in, int batch, int first, hipStream_t stream, int hp, unsigned seq);

}  // namespace strait
