// Host-side objects behind the opaque handles of bild.h, shared by the product entry points (bild_api.hip)
// and the measurement entry points (bench_api.hip).  Not part of the public ABI.
#pragma once
#include <algorithm>
#include <cstring>
#include <array>
#include <map>
#include <mutex>
#include <utility>
#include <vector>

#include "bild_internal.h"

#define HIPC(expr)                                   \
    do {                                             \
        hipError_t e_ = (expr);                      \
        if (e_ != hipSuccess) return BILD_EHIP;      \
    } while (0)

using bild::Ctl;
using bild::StatPart;
using bild::TMat;
using bild::kMaxRows;

struct LayerW {
    const float* ln1 = nullptr;
    TMat wqkv, wo;
    const float* lnc = nullptr;
    TMat cwq, cwkv, cwo;
    const float* ln2 = nullptr;
    TMat win, wout;
};

// Scratch buffers of bild_head_stats between its calls: whoever needs one takes it (calls of several threads take several),
// at most kKept wait here, and they are freed with the model.
struct HeadScratch {
    void* p = nullptr;
    size_t bytes = 0;
    int dev = -1;
    unsigned *done = nullptr, *done_dev = nullptr;  // pinned, a word per row: the number of the last call whose result is there
    unsigned calls = 0;
    void release() {  // (the first waits for whatever is still running)
        (void)hipFree(p);
        if (done) (void)hipHostFree(done);
    }
};
class HeadPool {
    static constexpr int kKept = 4;
    std::mutex mu;
    std::vector<HeadScratch> kept;

public:
    // For a call on stream `st`: what a fresh buffer has to hold is put there on it, in front of the call's kernels.  (A fill on the null stream
    // is not ordered with a stream that does not wait for it.)
    HeadScratch take(size_t bytes, hipStream_t st) {
        HeadScratch b;
        if (hipGetDevice(&b.dev) != hipSuccess) return b;
        {
            std::lock_guard<std::mutex> lock(mu);
            for (size_t i = 0; i < kept.size(); ++i)
                if (kept[i].dev == b.dev && kept[i].bytes >= bytes) {
                    b = kept[i];
                    kept.erase(kept.begin() + i);
                    return b;
                }
        }
        b.bytes = bytes;
        if (hipMalloc(&b.p, bytes) != hipSuccess) b.p = nullptr;
        if (b.p && hipMemsetAsync(b.p, 0, std::min(bytes, (size_t)256), st) != hipSuccess) {  // (the count of workgroups that arrive)
            (void)hipFree(b.p);
            b.p = nullptr;
        }
        void* h = nullptr;
        if (b.p && hipHostMalloc(&h, sizeof(unsigned) * kMaxRows, hipHostMallocMapped) == hipSuccess) {
            void* dp = nullptr;
            if (hipHostGetDevicePointer(&dp, h, 0) == hipSuccess) {
                std::memset(h, 0, sizeof(unsigned) * kMaxRows);
                b.done = (unsigned*)h;
                b.done_dev = (unsigned*)dp;
            } else {
                (void)hipHostFree(h);
            }
        }
        return b;
    }
    void give(const HeadScratch& b) {  // (no kernel uses it any more); the smallest of too many goes
        HeadScratch out = b;
        {
            std::lock_guard<std::mutex> lock(mu);
            kept.push_back(b);
            if (kept.size() <= (size_t)kKept) return;
            size_t least = 0;
            for (size_t i = 1; i < kept.size(); ++i)
                if (kept[i].bytes < kept[least].bytes) least = i;
            out = kept[least];
            kept.erase(kept.begin() + least);
        }
        out.release();
    }
    ~HeadPool() {
        for (HeadScratch& b : kept) b.release();
    }
};

struct bild_model {
    bild_model_config cfg;
    TMat emb, head;
    const float* enc_final = nullptr;
    const float* dec_final = nullptr;
    const float* enc_rel = nullptr;  // relative-position models: [heads][2*rel_max_dist + 1] score biases of the
    const float* dec_rel = nullptr;  // encoder's / decoder's self-attention, shared by all layers of the stack
    std::vector<LayerW> enc, dec;
    TMat cwkv_all;                   // the cross K/V projections of all decoder layers side by side (dec[l].cwkv points into it)
    std::vector<void*> allocs;
    mutable HeadPool head_pool;
    size_t device_bytes = 0;
    int inner() const { return cfg.n_heads * cfg.d_head; }
    int esz() const { return cfg.dtype == BILD_DT_BF16 ? 2 : 4; }
    bool gated() const { return cfg.act != BILD_ACT_RELU; }
    size_t layer_weight_bytes() const {  // weight matrices of one decoder layer
        const size_t d = cfg.d_model, I = inner(), F = cfg.d_ff;
        return (4 * d * I * (cfg.cross_attn ? 2 : 1) + (gated() ? 3 : 2) * d * F) * esz();
    }
};

// A stream that no state owns: the small model's encoder runs on it, beside the large one's on the stream of the state (one
// encode at a time; whoever finds it taken runs both encoders on the stream of its state).  A process has four hardware queues
// unless told otherwise, handed out as streams are made, and requests whose streams share one run strictly one after the other.
// So a new state takes the spare stream as its own and a new spare is made: only a queue that no state wanted is spent on it.
// (A second stream in every state, or one that keeps its early place, had two T5-shaped requests share a queue beside an idle
// state: 2274 tokens/s, passes as kernels of their own; 4060 with this one.)
class SpareStream {
    std::mutex mu;
    hipStream_t stream = nullptr;
    hipEvent_t fork = nullptr, join = nullptr;
    int dev = -1;

public:
    // The stream of a new state: the spare one or a new one.  Null: none can be made.
    hipStream_t take(int device) {
        std::lock_guard<std::mutex> lock(mu);
        hipStream_t st = device == dev ? std::exchange(stream, nullptr) : nullptr;
        if (!st && hipStreamCreate(&st) != hipSuccess) return nullptr;
        return st;
    }
    // Makes sure that there is one (without: the encoders run one after the other).
    void renew(int device) {
        std::lock_guard<std::mutex> lock(mu);
        if (stream) return;
        dev = device;
        if (!fork && hipEventCreateWithFlags(&fork, hipEventDisableTiming) != hipSuccess) fork = nullptr;
        if (!join && hipEventCreateWithFlags(&join, hipEventDisableTiming) != hipSuccess) join = nullptr;
        if (fork && join && hipStreamCreate(&stream) != hipSuccess) stream = nullptr;
    }
    // The work of `first` on the stream `st` of a state and that of `second` on this one, both behind what is on `st`; what
    // follows on `st` waits for both.  False: neither was called.
    template <class First, class Second>
    bool beside(int device, hipStream_t& st, First&& first, Second&& second, int* rc) {
        std::unique_lock<std::mutex> lock(mu, std::try_to_lock);
        if (!lock.owns_lock() || !stream || device != dev || hipEventRecord(fork, st) != hipSuccess) return false;
        *rc = first();
        if (*rc) return true;
        if (hipStreamWaitEvent(stream, fork, 0) != hipSuccess) {
            *rc = BILD_EHIP;
            return true;
        }
        std::swap(st, stream);
        *rc = second();
        std::swap(st, stream);
        // (also behind an error)
        if (hipEventRecord(join, stream) != hipSuccess || hipStreamWaitEvent(st, join, 0) != hipSuccess) *rc = BILD_EHIP;
        return true;
    }
    ~SpareStream() {
        if (fork) (void)hipEventDestroy(fork);
        if (join) (void)hipEventDestroy(join);
        if (stream) (void)hipStreamDestroy(stream);
    }
};

struct bild_pair {
    bild_model* m[2];  // [0] small, [1] large
    bool decoder_only;
    bool small_borrows_encoder;
    int trunk_layers = 0;        // > 0: early-exit pair, m[0] is a view of m[1]'s first trunk_layers decoder layers
    bild_model* view = nullptr;  // that view (owned by the pair; it owns no device memory)
    mutable SpareStream spare;
};

struct ModelState {
    const bild_model* m = nullptr;
    char* kcache = nullptr;  // [L][cap][I]
    char* vcache = nullptr;
    char* ck = nullptr;      // cross [L][max_src][I]
    char* cv = nullptr;
    float *x = nullptr, *q = nullptr, *a = nullptr, *h = nullptr;  // [rows_cap][d], [rows_cap][I], [rows_cap][I], [rows_cap][F]
    int rows_cap = kMaxRows;  // rows one decoder pass may carry (the whole prompt for decoder-only prefill)
    StatPart* part = nullptr;
    int nparts_cap = 0;
    float* zt = nullptr;
    float* dbg = nullptr;     // [32][vocab], only when debugging
    float* att_o = nullptr;   // split-key partials
    float* att_ml = nullptr;
    int max_splits = 1;
    // encoder scratch (models with an encoder)
    float* enc_x = nullptr;   // [max_src][d]
    float* enc_q = nullptr;   // [max_src][I]
    float* enc_a = nullptr;   // [max_src][I]
    float* enc_h = nullptr;   // [max_src][F]
    char* enc_k = nullptr;    // [max_src][I]
    char* enc_v = nullptr;
    int last_rows = 0;        // rows of the last LM-head pass (for debug logits)
    // bf16 models: activations of a pass of a few rows as high / low bf16 planes (see GemmArgs::xb_hi)
    uint16_t* xb = nullptr;   // [2][32][d]   residual stream times the next norm's gain
    uint16_t* ab = nullptr;   // [2][32][I]   attention output
    uint16_t* hb = nullptr;   // [2][32][F]   FFN hidden
    float* ssq = nullptr;     // [d / 16 + 8][32] partial sums of squares beside xb
    float* x2 = nullptr;      // [32][d] second residual-stream buffer (see GemmArgs::x_out)
    float* px = nullptr;      // [kPartSlices][32][d] partial results of a split FFN output projection
    float* pxh = nullptr;     // [kMaxHeadParts][32][d] one partial result per head of attention fused with its output projection
    float* pe = nullptr;      // sinusoidal models: position table [max(cap_len, cap_src)][d] for the embedding
    double2* rope = nullptr;  // rotary models: cos and sin, [max(cap_len, cap_src)][d_head / 2]
    // bf16 models, passes over many rows: the residual stream as tile planes (see TileGemmArgs) and the partial sums of squares
    // beside it; the attention output and the FFN hidden state use the memory of enc_a, enc_h (a, h without an encoder)
    char* xt = nullptr;
    float* ssq_t = nullptr;
    int rows_t = 0;           // rows these hold
    // whole passes in one kernel (pass_kernel.hip)
    int pass_groups = 0;      // workgroups; 0: the shape is not made for it
    int pass_die_groups = 0;  // the same of the form on one die
    bool pass_wide = false;   // the form of pass_wide.hip
    int pass_wide_rows = 0;   // most rows of passes there
    bild::PassLayer* pass_layers = nullptr;  // device
    int pass_die_rows = 0;    // most rows there (the small model's passes with an LM head have one)
    char* pass_turns[bild::kPassRooms] = {};  // what its workgroups hand over, by the rows there is room for
};

// How a pass ran (ROUTE_GAVE_UP: those of the first two that were run again as kernels).
enum Route : int { ROUTE_CHIP = 0, ROUTE_DIE = 1, ROUTE_KERNELS = 2, ROUTE_GAVE_UP = 3 };

struct bild_state {
    const bild_pair* pair = nullptr;
    ModelState ms[2];
    Ctl* ctl = nullptr;   // device
    Ctl* hctl = nullptr;  // pinned host mirror of the control block, written by the policy kernel
    int seq_issued = 0;   // passes with a policy kernel enqueued so far (the device counts them in Ctl::seq)
    Ctl* hctl_dev = nullptr;  // the same buffer as the device sees it
    int* hy = nullptr;        // pinned copy of y on the host: every token the host sets or a pass reports goes into it
    int* hsrc = nullptr;      // pinned copy of src
    float alpha_fb = -1.f, alpha_rb = -1.f;  // thresholds currently in the device control block
    bool use_graphs = true;
    bool one_kernel = true;   // passes of a few rows run as one kernel where there is one for the shape (takes_one_kernel)
    bool one_die = true;      // ... on one die, if it fits
    float* thin_sums = nullptr;  // of the slices of the thin GEMM's projections
    unsigned* thin_arrived = nullptr;
    float* split_part = nullptr;  // of the workgroups that share a head's keys
    unsigned* split_arrived = nullptr;
    int wide_most_rows = 0;   // > 0: passes of wide models in one kernel have up to so many rows, where there is a kernel for them (else see wide_rows)
    int thin_min_rows = 0;    // > 0: passes of a bf16 model from so many rows on take the thin GEMM (else see takes_thin)
    unsigned* pass_sync = nullptr;
    bool last_one = false;    // the pass issued last is one kernel
    int pass_pause = 0, pass_fails = 0;  // passes to run as separate kernels before the next attempt; attempts in vain in a row
    int pass_spins = 6000;    // polls of a wait, about 4 ms: kernels of other streams come to an end in that time, the same kernel of another process
                              // does not (64 times as many of the head inside a pass, which waits for all of the layers: pass_head.h)
    int device = 0, cus = 0;
    int depth = 0;            // calls of this state that are on the stack (see Call)
    int64_t routes[4] = {};   // passes with an LM head so far, by Route
    int ksplit_max_d = 2048;      // ... of models up to this wide (7B-shaped small model, 2048 wide: 0.729 -> 0.717 ms per step)
    int ksplit_min_f = 2048;      // FFN widths from which the output projection of a narrow model (d <= 1024) is cut into input slices
    int fuse_max_kv = 32 << 10;   // ... while one head's cached K/V are at most this many bytes
    bool fuse_attn = true;        // single-row passes of narrow models: attention and its output projection in one kernel
    bool fuse_embed = true;       // single-row passes: the first projection gathers its input row from the embedding matrix
    int pre_min_rows = 0;         // > 0 (experiments): row count from which a bf16 pass hands activations on as bf16 planes
    bool gemm_only = false;       // measurement: a pass launches only its weight-streaming GEMMs
    int64_t gemm_count = 0, gemm_bytes = 0;  // tallied while a pass is being issued
    int stage_count = 0;          // kernel launches of the pass issued or replayed last (counted also where a measurement skips the launch)
    struct Captured { hipGraphExec_t exec; int stages; };
    std::map<std::array<int, 7>, Captured> graphs;  // captured passes by (model, rows, lm rows, mode, key bucket, source bucket, options)
    float top_p = 0.f;         // > 0: sampling variant, tokens are drawn from the nucleus
    float* u_dev[2] = {nullptr, nullptr};  // uniform number per sequence position, per model
    bild::DrawWs* draw_ws = nullptr; // workspace of the draw that is spread over the chip
    bool draw_spread = true;   // false (BILD_DRAW_ONE_WG=1, tests): every draw by the single workgroup of the policy kernel
    int accept_mode = 0;       // 1: the review uses the rejection-sampling rule (needs top_p > 0)
    float* u_acc = nullptr;    // uniform number per sequence position for that rule
    float* s_ring = nullptr;   // [kMaxRows][vocab] the small model's logits of the pending drafts
    float4* s_draw = nullptr;  // [max_len + 1] (max, threshold key, nucleus mass) of the small model's row per position
    float* trunk_x = nullptr;  // early-exit pair: [cap_len][d] hidden state after the trunk's last layer, by position
    int* y = nullptr;     // device [max_len + 1]
    int* src = nullptr;   // device [max_src]
    hipStream_t stream = nullptr;
    bool own_stream = false;
    int max_src = 0, max_len = 0, n_max = 0;
    int cap_len = 0, cap_src = 0;  // cache capacities: max_len / max_src rounded up to 32 rows
    // host mirror of the control block (kept exact by reading back after every pass)
    int y_len = 0, draft_start = 0, len[2] = {0, 0}, n_src = 0, n0 = 0;
    bool encoded = false;
    bool debug_logits = false;
    std::vector<void*> allocs;
    std::vector<void*> host_allocs;
    // event bracketing of GEMM launches (measurement only)
    bool prof_on = false;
    int prof_cap = 0, prof_used = 0, prof_dropped = 0;
    std::vector<hipEvent_t> prof_ev;
    struct ProfRec { int model, cls; int64_t bytes; };
    std::vector<ProfRec> prof_rec;
};


namespace bild {
// shared host logic (bild_api.hip)
int dev_alloc(std::vector<void*>& keep, void** p, size_t bytes);
int key_bucket(int nkeys);
int catch_up(bild_state* s, int w, int target);
// A call of the library that runs passes, from its entry to its end (see g_inside, bild_api.hip).
struct Call {
    bild_state* s;
    explicit Call(bild_state* state);
    ~Call();
    Call(const Call&) = delete;
};
int run_pass(bild_state* s, int w, int T, int lm_rows, int mode);
int pass_gave_up(bild_state* s, int w, int T);
int decoder_pass(bild_state* s, int w, int T, int lm_rows, int mode, int key_hint, bool one);
int pick_splits_raw(int d_head, int esz, int max_splits, int nkeys, int heads, int T, bool* defer);
int pick_attn_waves(int dtype, int d_head, int T, int nkeys, int splits);
}  // namespace bild
