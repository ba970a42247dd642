// C ABI of the BiLD library: model upload, per-request state, and the launch
// sequences of the decoder passes.  All numerical work is in kernels.hip; this
// file owns memory and ordering only.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <array>
#include <atomic>
#include <cmath>
#include <cstdlib>
#include <map>
#include <cstdio>
#include <chrono>
#include <cstring>
#include <new>
#include <vector>

#include "bild_state.h"
#include "attn_split.h"
#include "gemm_thin.h"
#include "head.h"

using namespace bild;

namespace bild {
int dev_alloc(std::vector<void*>& keep, void** p, size_t bytes) {
    void* d = nullptr;
    if (bytes == 0) bytes = 16;
    if (hipMalloc(&d, bytes) != hipSuccess) return BILD_ENOMEM;
    keep.push_back(d);
    *p = d;
    return BILD_OK;
}
}  // namespace bild

namespace {

// ---------------------------------------------------------------- helpers

bool config_ok(const bild_model_config& c) {
    if (c.n_dec_layers < 1 || c.n_enc_layers < 0) return false;
    if (c.d_model < 32 || c.d_model % 32 || c.d_ff < 32 || c.d_ff % 32) return false;
    if (c.n_heads < 1 || c.d_head < 8 || c.d_head > 128 || c.d_head % 8) return false;
    if ((c.n_heads * c.d_head) % 32) return false;
    if (c.act < 0 || c.act > 2 || c.pos < 0 || c.pos > 2 || c.dtype < 0 || c.dtype > 1) return false;
    if (c.vocab < 1 || c.bos < 0 || c.bos >= c.vocab) return false;
    if (c.n_enc_layers > 0 && !c.cross_attn) return false;
    if (!(c.norm_eps >= 0.f) || !(c.rope_base > 0.f)) return false;
    if (c.tie_shift < 0) return false;
    if (c.pos == BILD_POS_RELATIVE && (c.rel_max_dist < 1 || c.rel_max_dist > 4096)) return false;
    return true;
}

// what the workgroups of a pass in one kernel hand over: three layers' memory
size_t pass_turns_bytes(const ModelState& M, int room) {
    const bool f32 = M.m->cfg.dtype == BILD_DT_F32;
    const PassPlan p = pass_plan(1 << room, M.m->cfg.d_model, M.m->inner(), M.m->cfg.d_ff, f32, M.pass_wide);
    PassHead h = {};
    if (room != 0 || M.pass_die_groups == 0) return 3 * (size_t)p.layer;
    pass_head_plan(h, p, M.m->cfg.d_model, f32, 256);  // (on one die: of 256 compute units)
    return (size_t)h.at + 2 * (size_t)h.bytes;
}

// captured passes carry some of the state's settings by value: where one changes they are captured anew
void drop_graphs(bild_state* s) {
    (void)hipStreamSynchronize(s->stream);
    for (auto& kv : s->graphs) (void)hipGraphExecDestroy(kv.second.exec);
    s->graphs.clear();
}

int upload_vec(bild_model* m, const float* src, int n, const float** out) {
    void* d;
    int rc = dev_alloc(m->allocs, &d, (size_t)n * 4);
    if (rc) return rc;
    if (hipMemcpy(d, src, (size_t)n * 4, hipMemcpyHostToDevice) != hipSuccess) return BILD_EHIP;
    m->device_bytes += (size_t)n * 4;
    *out = (const float*)d;
    return BILD_OK;
}

// `at`: device memory for the matrix (null: allocated here)
int upload_tiled(bild_model* m, std::vector<char>& staging, int n, int k, TMat* out, void* at = nullptr) {
    const int kt = m->cfg.dtype == BILD_DT_BF16 ? 32 : 16;
    const size_t bytes = tiled_bytes(n, k, m->cfg.dtype);
    void* d = at;
    if (!d) {
        int rc = dev_alloc(m->allocs, &d, bytes);
        if (rc) return rc;
    }
    if (hipMemcpy(d, staging.data(), bytes, hipMemcpyHostToDevice) != hipSuccess) return BILD_EHIP;
    m->device_bytes += bytes;
    out->w = d;
    out->n = n;
    out->k = k;
    out->tn = (n + 15) / 16;
    out->tk = k / kt;
    return BILD_OK;
}

int upload_matrix(bild_model* m, const float* src, bool k_by_n, int n, int k, TMat* out) {
    std::vector<char> st(tiled_bytes(n, k, m->cfg.dtype));
    tile_matrix(src, k_by_n, n, k, m->cfg.dtype, st.data());
    return upload_tiled(m, st, n, k, out);
}

int upload_concat(bild_model* m, std::initializer_list<const float*> srcs, int n_each, int k, TMat* out, void* at = nullptr) {
    std::vector<const float*> ps(srcs);
    std::vector<int> ns(ps.size(), n_each);
    const int n = n_each * (int)ps.size();
    std::vector<char> st(tiled_bytes(n, k, m->cfg.dtype));
    tile_concat(ps.data(), ns.data(), (int)ps.size(), k, m->cfg.dtype, st.data());
    return upload_tiled(m, st, n, k, out, at);
}

int upload_ffn_in(bild_model* m, const float* w_in, const float* w_up, TMat* out) {
    const int d = m->cfg.d_model, f = m->cfg.d_ff;
    if (!m->gated()) return upload_matrix(m, w_in, true, f, d, out);
    std::vector<char> st(tiled_bytes(2 * f, d, m->cfg.dtype));
    tile_gated_pair(w_in, w_up, f, d, m->cfg.dtype, st.data());
    return upload_tiled(m, st, 2 * f, d, out);
}

}  // namespace

// ======================================================================= models
extern "C" int bild_model_num_tensors(const bild_model_config* c) {
    if (!c || !config_ok(*c)) return BILD_EINVAL;
    const int gated = c->act != BILD_ACT_RELU;
    int n = 1 + (c->tied_head ? 0 : 1) + (c->n_enc_layers > 0 ? 1 : 0) + 1;
    if (c->pos == BILD_POS_RELATIVE) n += (c->n_enc_layers > 0 ? 1 : 0) + 1;
    n += c->n_enc_layers * (8 + gated);
    n += c->n_dec_layers * (8 + gated + (c->cross_attn ? 5 : 0));
    return n;
}

extern "C" int bild_model_destroy(bild_model* m) {
    if (!m) return BILD_EINVAL;
    for (void* p : m->allocs) (void)hipFree(p);
    delete m;
    return BILD_OK;
}

extern "C" int bild_model_create(const bild_model_config* cfg, const float* const* t, int n_tensors,
                                 bild_model** out) {
    if (!cfg || !t || !out) return BILD_EINVAL;
    if (!config_ok(*cfg)) return BILD_EINVAL;
    if (n_tensors != bild_model_num_tensors(cfg)) return BILD_EINVAL;
    for (int i = 0; i < n_tensors; ++i)
        if (!t[i]) return BILD_EINVAL;
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || ndev < 1) return BILD_EHIP;
    bild_model* m = new (std::nothrow) bild_model();
    if (!m) return BILD_ENOMEM;
    m->cfg = *cfg;
    m->cfg.tie_shift %= cfg->vocab;  // (kernels take the row below vocab with one subtraction)
    const int d = cfg->d_model, I = m->inner(), F = cfg->d_ff, V = cfg->vocab;
    int i = 0, rc = BILD_OK;
#define UP(call)                         \
    do {                                 \
        rc = (call);                     \
        if (rc) {                        \
            bild_model_destroy(m);       \
            return rc;                   \
        }                                \
    } while (0)
    UP(upload_matrix(m, t[i++], false, V, d, &m->emb));
    if (cfg->tied_head)
        m->head = m->emb;
    else
        UP(upload_matrix(m, t[i++], false, V, d, &m->head));
    if (cfg->n_enc_layers > 0) UP(upload_vec(m, t[i++], d, &m->enc_final));
    UP(upload_vec(m, t[i++], d, &m->dec_final));
    if (cfg->pos == BILD_POS_RELATIVE) {
        const int nrel = cfg->n_heads * (2 * cfg->rel_max_dist + 1);
        if (cfg->n_enc_layers > 0) UP(upload_vec(m, t[i++], nrel, &m->enc_rel));
        UP(upload_vec(m, t[i++], nrel, &m->dec_rel));
    }
    m->enc.resize(cfg->n_enc_layers);
    for (auto& L : m->enc) {
        UP(upload_vec(m, t[i], d, &L.ln1));
        UP(upload_concat(m, {t[i + 1], t[i + 2], t[i + 3]}, I, d, &L.wqkv));
        UP(upload_matrix(m, t[i + 4], true, d, I, &L.wo));
        UP(upload_vec(m, t[i + 5], d, &L.ln2));
        i += 6;
        UP(upload_ffn_in(m, t[i], m->gated() ? t[i + 1] : nullptr, &L.win));
        i += m->gated() ? 2 : 1;
        UP(upload_matrix(m, t[i++], true, d, F, &L.wout));
    }
    m->dec.resize(cfg->n_dec_layers);
    // the cross K/V projections of all layers in one block: they read the same input, so one launch can run all of them
    char* cwkv_at = nullptr;
    if (cfg->cross_attn) {
        UP(dev_alloc(m->allocs, (void**)&cwkv_at, tiled_bytes(2 * I, d, cfg->dtype) * cfg->n_dec_layers));
        m->cwkv_all.w = cwkv_at;
        m->cwkv_all.n = 2 * I * cfg->n_dec_layers;
        m->cwkv_all.k = d;
        m->cwkv_all.tn = m->cwkv_all.n / 16;
        m->cwkv_all.tk = d / (cfg->dtype == BILD_DT_BF16 ? 32 : 16);
    }
    for (auto& L : m->dec) {
        UP(upload_vec(m, t[i], d, &L.ln1));
        UP(upload_concat(m, {t[i + 1], t[i + 2], t[i + 3]}, I, d, &L.wqkv));
        UP(upload_matrix(m, t[i + 4], true, d, I, &L.wo));
        i += 5;
        if (cfg->cross_attn) {
            UP(upload_vec(m, t[i], d, &L.lnc));
            UP(upload_matrix(m, t[i + 1], true, I, d, &L.cwq));
            UP(upload_concat(m, {t[i + 2], t[i + 3]}, I, d, &L.cwkv, cwkv_at));
            cwkv_at += tiled_bytes(2 * I, d, cfg->dtype);
            UP(upload_matrix(m, t[i + 4], true, d, I, &L.cwo));
            i += 5;
        }
        UP(upload_vec(m, t[i++], d, &L.ln2));
        UP(upload_ffn_in(m, t[i], m->gated() ? t[i + 1] : nullptr, &L.win));
        i += m->gated() ? 2 : 1;
        UP(upload_matrix(m, t[i++], true, d, F, &L.wout));
    }
#undef UP
    *out = m;
    return BILD_OK;
}

extern "C" int bild_pair_create(bild_model* s, bild_model* l, bild_pair** out) {
    if (!s || !l || !out) return BILD_EINVAL;
    if (s->cfg.vocab != l->cfg.vocab) return BILD_EINVAL;
    if (s->cfg.cross_attn != l->cfg.cross_attn) return BILD_EINVAL;
    if (s->cfg.bos != l->cfg.bos) return BILD_EINVAL;
    const bool dec_only = !l->cfg.cross_attn;
    bool borrows = false;
    if (!dec_only) {
        if (l->cfg.n_enc_layers < 1) return BILD_EINVAL;
        if (s->cfg.n_enc_layers == 0) {
            if (s->cfg.d_model != l->cfg.d_model) return BILD_EINVAL;
            borrows = true;
        }
    }
    bild_pair* p = new (std::nothrow) bild_pair();
    if (!p) return BILD_ENOMEM;
    p->m[0] = s;
    p->m[1] = l;
    p->decoder_only = dec_only;
    p->small_borrows_encoder = borrows;
    *out = p;
    return BILD_OK;
}

extern "C" int bild_pair_create_early_exit(bild_model* l, int k, float small_logit_scale, bild_pair** out) {
    if (!l || !out) return BILD_EINVAL;
    if (k < 1 || k >= l->cfg.n_dec_layers || !(small_logit_scale > 0.f)) return BILD_EINVAL;
    if (l->cfg.cross_attn && l->cfg.n_enc_layers < 1) return BILD_EINVAL;
    bild_model* v = new (std::nothrow) bild_model();
    bild_pair* p = new (std::nothrow) bild_pair();
    if (!v || !p) {
        delete v;
        delete p;
        return BILD_ENOMEM;
    }
    v->cfg = l->cfg;
    v->cfg.n_dec_layers = k;
    v->cfg.n_enc_layers = 0;  // it attends to the large model's encoder output
    v->cfg.logit_scale = small_logit_scale;
    v->emb = l->emb;
    v->head = l->head;
    v->dec_final = l->dec_final;
    v->dec_rel = l->dec_rel;
    v->dec.assign(l->dec.begin(), l->dec.begin() + k);
    v->cwkv_all = l->cwkv_all;  // (a view's cross K/V are the large model's: never projected for the view)
    p->m[0] = v;
    p->m[1] = l;
    p->decoder_only = !l->cfg.cross_attn;
    p->small_borrows_encoder = l->cfg.cross_attn != 0;
    p->trunk_layers = k;
    p->view = v;
    *out = p;
    return BILD_OK;
}

extern "C" int bild_pair_destroy(bild_pair* p) {
    if (!p) return BILD_EINVAL;
    delete p->view;  // a view owns no device memory
    delete p;
    return BILD_OK;
}

// ======================================================================= state
namespace {

// States that are inside a call, by device.  The workgroups of a pass kernel wait for each other, so all of them have to be on the
// chip: two such passes at a time could keep half of each other's out, and a pass of separate kernels crawls where it finds them.
// So only a state that is inside a call alone takes the pass kernel.  When a call returns, its passes have ended, but for the last one with LM
// head and policy inside (pass_head.h), which tells the host itself.  What is left of that kernel waits for nobody else's workgroups: on
// die 0 all are past their last hand-over, the head's are past their partials, or have yet to start and will find the hidden state in its place; of
// a pass that gave up, the waits that are left are bounded and look at its flag.  So it ends by itself, and another state's pass kernel, whose waits are
// for its own workgroups alone, gets its compute units some microseconds later (where somebody else's work keeps the last workgroups
// from starting, they take them no longer than that part of theirs).  The state's own next kernel, its rerun among them, is behind on the stream.
// Two, three, four requests together, six generations each, T5-large / T5-small shapes, tokens/s, each on a hardware queue of its
// own: a pass kernel for whoever finds none in flight 3870, 4066, 4320, this rule 3930, 5050, 5980, and 4100, 5560, 6800 once the
// graphs of the separate kernels are captured (one alone: 3040 with the pass kernel, 2265 without).
// (Three whose streams share a queue: 3600 and 3090.  Staying with separate kernels for 5 ms after two calls have met, for
// requests driven call by call: no gain.)
constexpr int kMaxDevices = 64;
std::atomic<int> g_inside[kMaxDevices];
std::atomic<int>& inside(const bild_state* s) { return g_inside[s->device % kMaxDevices]; }
bool alone(const bild_state* s) { return inside(s).load(std::memory_order_acquire) <= 1; }

}  // namespace

bild::Call::Call(bild_state* state) : s(state) {
    if (s->depth++ == 0) inside(s).fetch_add(1, std::memory_order_acq_rel);
}
bild::Call::~Call() {
    if (--s->depth == 0) inside(s).fetch_sub(1, std::memory_order_acq_rel);
}

extern "C" int bild_state_destroy(bild_state* s) {
    if (!s) return BILD_EINVAL;
    if (s->stream) (void)hipStreamSynchronize(s->stream);
    for (void* p : s->allocs) (void)hipFree(p);
    for (void* p : s->host_allocs) (void)hipHostFree(p);
    for (hipEvent_t e : s->prof_ev) (void)hipEventDestroy(e);
    for (auto& kv : s->graphs) (void)hipGraphExecDestroy(kv.second.exec);
    if (s->own_stream && s->stream) (void)hipStreamDestroy(s->stream);
    delete s;
    return BILD_OK;
}

extern "C" int bild_state_create(const bild_pair* p, int max_src, int max_len, int n_max, void* hip_stream,
                                 bild_state** out) {
    if (!p || !out) return BILD_EINVAL;
    if (max_src < 1 || max_len < 2 || n_max < 0 || n_max > kMaxRows - 1) return BILD_EINVAL;
    if (p->decoder_only && max_len < max_src + 1) return BILD_EINVAL;
    bild_state* s = new (std::nothrow) bild_state();
    if (!s) return BILD_ENOMEM;
    s->pair = p;
    s->max_src = max_src;
    s->max_len = max_len;
    s->n_max = n_max;
    s->cap_len = (max_len + 31) / 32 * 32;
    s->cap_src = (max_src + 31) / 32 * 32;
    if (kernels_init() != hipSuccess) {
        delete s;
        return BILD_EHIP;
    }
    if (hipGetDevice(&s->device) != hipSuccess || hipDeviceGetAttribute(&s->cus, hipDeviceAttributeMultiprocessorCount, s->device) != hipSuccess) {
        delete s;
        return BILD_EHIP;
    }
    if (hip_stream) {
        s->stream = (hipStream_t)hip_stream;
    } else {
        s->stream = p->spare.take(s->device);
        if (!s->stream) {
            delete s;
            return BILD_EHIP;
        }
        s->own_stream = true;
    }
    if (!p->decoder_only && !p->small_borrows_encoder) p->spare.renew(s->device);
    // All device memory of the state is one allocation (dozens of separate ones cost a request about a millisecond); what has
    // to start zeroed lies together at its front.
    struct Want { void** p; size_t bytes; bool zero; };
    std::vector<Want> wants;
    auto want = [&](auto& ptr, size_t bytes, bool zero = false) { wants.push_back({(void**)&ptr, (bytes + 255) / 256 * 256, zero}); };
    want(s->ctl, sizeof(Ctl), true);
    want(s->y, sizeof(int) * (size_t)(max_len + 1));
    want(s->src, sizeof(int) * (size_t)max_src);
    void* h = nullptr;
    if (hipHostMalloc(&h, 1024 + sizeof(int) * ((size_t)max_len + 1 + max_src), hipHostMallocMapped) != hipSuccess) {
        bild_state_destroy(s);
        return BILD_ENOMEM;
    }
    s->host_allocs.push_back(h);
    s->hctl = (Ctl*)h;
    static_assert(sizeof(Ctl) <= 1024, "the tokens follow behind the control block");
    s->hy = (int*)((char*)h + 1024);
    s->hsrc = s->hy + max_len + 1;
    void* hd = nullptr;
    if (hipHostGetDevicePointer(&hd, h, 0) != hipSuccess) {
        bild_state_destroy(s);
        return BILD_EHIP;
    }
    s->hctl_dev = (Ctl*)hd;
    {
        const char* ng = std::getenv("BILD_NO_GRAPH");
        s->use_graphs = !(ng && ng[0] == '1');
        if (const char* ok = std::getenv("BILD_ONE_KERNEL")) s->one_kernel = ok[0] != '0';  // tests and measurements
        if (const char* od = std::getenv("BILD_ONE_DIE")) s->one_die = od[0] != '0';  // tests and measurements
        if (const char* sp = std::getenv("BILD_PASS_SPINS")) s->pass_spins = std::atoi(sp);  // tests
        if (const char* pm = std::getenv("BILD_PRE_MIN_ROWS")) s->pre_min_rows = std::atoi(pm);  // experiments; > 32 turns the planes off
        if (const char* fa = std::getenv("BILD_FUSE_ATTN")) s->fuse_attn = fa[0] != '0';      // experiments / tests
        if (const char* fk = std::getenv("BILD_FUSE_MAX_KV")) s->fuse_max_kv = std::atoi(fk);
        if (const char* dw = std::getenv("BILD_DRAW_ONE_WG")) s->draw_spread = dw[0] == '0';
        if (const char* fe = std::getenv("BILD_FUSE_EMBED")) s->fuse_embed = std::atoi(fe) != 0;  // tests and measurements
        if (const char* kd = std::getenv("BILD_KSPLIT_MAX_D")) s->ksplit_max_d = std::atoi(kd);
        if (const char* tr = std::getenv("BILD_THIN_MIN_ROWS")) s->thin_min_rows = std::atoi(tr);  // tests and measurements
        if (const char* wr = std::getenv("BILD_WIDE_ROWS")) s->wide_most_rows = std::atoi(wr);  // tests and measurements
        if (const char* km = std::getenv("BILD_KSPLIT_MIN_F")) s->ksplit_min_f = std::atoi(km);  // tests: small widths; 0 turns the split off
    }
    const int positions = std::max(s->cap_len, s->cap_src);
    if (s->one_kernel) want(s->pass_sync, sizeof(unsigned) * (kPassSyncWords + kPassTurnWords + 2 * kPassHeadWords), true);
    if (p->m[0]->cfg.dtype == BILD_DT_BF16 || p->m[1]->cfg.dtype == BILD_DT_BF16) {
        want(s->thin_sums, sizeof(float) * kThinSums);
        want(s->thin_arrived, sizeof(unsigned) * kThinArrivals, true);
        want(s->split_part, sizeof(float) * kAttnSplitFloats);
        want(s->split_arrived, sizeof(unsigned) * kAttnSplitHeads, true);
    }
    for (int w = 0; w < 2; ++w) {
        ModelState& M = s->ms[w];
        const bild_model* m = p->m[w];
        M.m = m;
        const size_t I = m->inner(), d = m->cfg.d_model, F = m->cfg.d_ff, L = m->cfg.n_dec_layers;
        const size_t esz = m->esz();
        const bool bf16 = m->cfg.dtype == BILD_DT_BF16, has_enc = m->cfg.n_enc_layers > 0;
        // every K/V buffer starts zeroed: rows past the valid length must hold finite values
        if (!(w == 0 && p->trunk_layers > 0)) {  // (an early-exit pair's trunk is the large model's first layers: one cache serves both)
            want(M.kcache, L * (size_t)s->cap_len * I * esz, true);
            want(M.vcache, L * (size_t)s->cap_len * I * esz, true);
            if (m->cfg.cross_attn) {
                want(M.ck, L * (size_t)s->cap_src * I * esz, true);
                want(M.cv, L * (size_t)s->cap_src * I * esz, true);
            }
        }
        // a decoder-only model prefills its whole prompt in one pass of many row blocks
        M.rows_cap = p->decoder_only ? std::max(kMaxRows, max_src) : kMaxRows;
        const size_t rows16 = (size_t)(M.rows_cap + 15) / 16 * 16, src16 = (size_t)(max_src + 15) / 16 * 16;  // (tile planes hold whole row tiles)
        // the two residual-stream buffers in one block: a reader of partial results gets the other buffer as a 32-bit
        // offset from the one it reads (GemmArgs::x_out)
        want(M.x, sizeof(float) * ((size_t)M.rows_cap + kMaxRows) * d);
        want(M.q, sizeof(float) * M.rows_cap * I);
        want(M.a, sizeof(float) * rows16 * I);
        want(M.h, sizeof(float) * rows16 * F);
        want(M.px, sizeof(float) * kPartSlices * kMaxRows * d);
        if (d <= 1024) want(M.pxh, sizeof(float) * kMaxHeadParts * kMaxRows * d, true);  // slots of heads a model does not have stay zero
        if (m->cfg.pos == BILD_POS_SINUSOIDAL) want(M.pe, sizeof(float) * (size_t)positions * d);
        if (m->cfg.pos == BILD_POS_ROPE) want(M.rope, sizeof(double2) * (size_t)positions * (m->cfg.d_head / 2));
        if (bf16 && (has_enc || M.rows_cap > kMaxRows || (w == 0 && p->small_borrows_encoder))) {
            M.rows_t = p->decoder_only ? M.rows_cap : max_src;
            want(M.xt, plane_bytes(M.rows_t, d));
            want(M.ssq_t, sizeof(float) * (size_t)M.rows_t * (d / 16));  // at most one part per feature tile
        }
        if (bf16) {
            want(M.xb, sizeof(uint16_t) * 2 * kMaxRows * d);
            want(M.ab, sizeof(uint16_t) * 2 * kMaxRows * I);
            want(M.hb, sizeof(uint16_t) * 2 * kMaxRows * F);
            want(M.ssq, sizeof(float) * (kMaxSsqParts + 8) * kMaxRows);
        }
        const bool in_int = cache_in_int(s->cap_len, I, esz) && (!m->cfg.cross_attn || cache_in_int(s->cap_src, I, esz));
        if (s->one_kernel && in_int && m->cfg.pos != BILD_POS_ROPE) {
            const int die = s->one_die && s->cus == 256 ? pass_die_groups((int)d, m->cfg.n_heads, m->cfg.d_head, (int)F, m->gated(), !bf16) : 0;
            M.pass_groups = bf16 ? pass_groups((int)d, m->cfg.n_heads, m->cfg.d_head, (int)F, m->gated(), s->cus, false) : die;
            if (M.pass_groups) {
                M.pass_die_groups = die;
                M.pass_die_rows = die == 0 ? 0 : !bf16 ? kPassRows : w == 0 ? 1 : kPassDieRows;
            }
        }
        if (s->one_kernel && in_int && bf16 && !m->cfg.cross_attn && m->cfg.pos != BILD_POS_RELATIVE && !M.pass_groups) {
            M.pass_groups = wide_groups((int)d, m->cfg.n_heads, m->cfg.d_head, (int)F, m->gated(), s->cus);
            M.pass_wide = M.pass_groups > 0;
            if (M.pass_wide) {
                const int most = wide_most((int)d, m->cfg.n_heads, (int)F, m->gated(), s->cus);
                M.pass_wide_rows = s->wide_most_rows > 0 ? std::min(most, s->wide_most_rows) : wide_rows((int)d, m->cfg.n_heads, (int)F, m->gated(), s->cus);
                // (no room above eight rows for reviews that this state's own drafts do not reach: of the 7B shape 13 MB for 16 and 26 for 32 rows)
                M.pass_wide_rows = std::min(M.pass_wide_rows, std::max(kWideRows, w == 0 ? 1 : 1 << pass_room_index(n_max + 1)));
            }
        }
        M.nparts_cap = m->head.tn + 1;  // at most one partial per feature tile
        want(M.part, sizeof(StatPart) * (size_t)M.nparts_cap * kMaxRows);
        want(M.zt, sizeof(float) * kMaxRows);
        M.max_splits = std::max(8, std::min(64, (std::max(max_len, max_src) + 511) / 512));
        want(M.att_o, sizeof(float) * (size_t)M.max_splits * kMaxRows * I);
        want(M.att_ml, sizeof(float) * (size_t)M.max_splits * kMaxRows * m->cfg.n_heads * 2);
        if (has_enc) {
            want(M.enc_x, sizeof(float) * (size_t)max_src * d);
            want(M.enc_q, sizeof(float) * (size_t)max_src * I);
            want(M.enc_a, sizeof(float) * src16 * I);
            want(M.enc_h, sizeof(float) * src16 * F);
            want(M.enc_k, (size_t)s->cap_src * I * esz, true);
            want(M.enc_v, (size_t)s->cap_src * I * esz, true);
        }
    }
    if (p->trunk_layers > 0) want(s->trunk_x, sizeof(float) * (size_t)s->cap_len * p->m[1]->cfg.d_model);
    // passes in one kernel: what both models' hand over, one behind the other, and their layers
    size_t turns_bytes = 0, layers_n = 0;
    for (ModelState& M : s->ms)
        for (int r = 0; M.pass_groups && r <= pass_room_index(M.pass_wide ? M.pass_wide_rows : kPassRows); ++r) {
            want(M.pass_turns[r], pass_turns_bytes(M, r));
            turns_bytes += wants.back().bytes;
        }
    for (const ModelState& M : s->ms) layers_n += M.pass_groups ? M.m->dec.size() : 0;
    PassLayer* pass_layers = nullptr;
    if (layers_n) want(pass_layers, sizeof(PassLayer) * layers_n);
    size_t zeroed = 0, total = 0;
    for (int pass = 0; pass < 2; ++pass) {
        for (Want& q : wants)
            if (q.zero == (pass == 0)) total += q.bytes;
        if (pass == 0) zeroed = total;
    }
    char* block = nullptr;
    if (int rc = dev_alloc(s->allocs, (void**)&block, total)) {
        bild_state_destroy(s);
        return rc;
    }
    char* at[2] = {block + zeroed, block};  // by zero
    for (Want& q : wants) {
        *q.p = at[q.zero];
        at[q.zero] += q.bytes;
    }
    hipError_t e = hipMemsetAsync(block, 0, zeroed, s->stream);
    for (int w = 0; w < 2 && e == hipSuccess; ++w) {
        ModelState& M = s->ms[w];
        const bild_model_config& c = p->m[w]->cfg;
        M.x2 = M.x + (size_t)M.rows_cap * c.d_model;
        if (M.pe) e = launch_pe_table(M.pe, positions, c.d_model, s->stream);
        if (M.rope && e == hipSuccess) e = launch_rope_table(M.rope, positions, c.d_head, c.rope_base, s->stream);
    }
    if (p->trunk_layers > 0) {
        s->ms[0].kcache = s->ms[1].kcache;
        s->ms[0].vcache = s->ms[1].vcache;
        s->ms[0].ck = s->ms[1].ck;
        s->ms[0].cv = s->ms[1].cv;
    }
    // One fill and one copy for both models.  (Making a state of the fp32, T5, 7B pair beside others, us, two runs: a fill and a copy for each
    // 164 to 237, 154 to 207, 262 to 276; now 166 to 175, 161 to 168, 244 to 273.  With the layers in the pinned block, which then takes more
    // than a page, some states took 200 us more.)
    if (e == hipSuccess && turns_bytes) e = hipMemsetAsync(s->ms[s->ms[0].pass_groups ? 0 : 1].pass_turns[0], 0xFF, turns_bytes, s->stream);
    std::vector<PassLayer> host_layers(layers_n);
    size_t filled = 0;
    for (ModelState& M : s->ms) {
        if (!M.pass_groups) continue;
        M.pass_layers = pass_layers + filled;
        const size_t kv = (size_t)s->cap_len * M.m->inner() * M.m->esz(), ckv = (size_t)s->cap_src * M.m->inner() * M.m->esz();
        for (size_t l = 0; l < M.m->dec.size(); ++l) {
            const LayerW& W = M.m->dec[l];
            PassLayer q = {W.wqkv.w, W.wo.w, W.cwq.w, W.cwo.w, W.win.w, W.wout.w, W.ln1, W.lnc, W.ln2, M.kcache + l * kv, M.vcache + l * kv, nullptr, nullptr};
            if (M.m->cfg.cross_attn) {
                q.ck = M.ck + l * ckv;
                q.cv = M.cv + l * ckv;
            }
            host_layers[filled++] = q;
        }
    }
    if (e == hipSuccess && filled) e = hipMemcpyAsync(pass_layers, host_layers.data(), sizeof(PassLayer) * filled, hipMemcpyHostToDevice, s->stream);
    if (e != hipSuccess || hipStreamSynchronize(s->stream) != hipSuccess) {
        bild_state_destroy(s);
        return BILD_EHIP;
    }
    *out = s;
    return BILD_OK;
}

namespace {

CtlArgs ctl_args(const bild_state* s) {
    CtlArgs a;
    std::memset((void*)&a, 0, sizeof(a));
    a.ctl = s->ctl;
    const int head[6] = {s->y_len, s->draft_start, s->len[0], s->len[1], s->n_src, s->n_max};
    std::memcpy(a.head, head, sizeof(head));
    std::memcpy(a.head + 6, &s->alpha_fb, 4);
    std::memcpy(a.head + 7, &s->alpha_rb, 4);
    a.seq = s->seq_issued;
    return a;
}

// address as the device sees it of something in the pinned block
const int* on_device(const bild_state* s, const int* p) { return (const int*)((const char*)s->hctl_dev + ((const char*)p - (const char*)s->hctl)); }

// The host's view of the request becomes the device's, with `n` tokens of hy from position `first` on and all of hsrc if
// `sources`.  A token of hy or hsrc that the host changes again before the kernel has read it is copied by the next call.
int push_ctl(bild_state* s, int first = 0, int n = 0, bool sources = false) {
    Ctl* h = s->hctl;
    if (__atomic_load_n(&h->seq, __ATOMIC_ACQUIRE) != s->seq_issued) HIPC(hipStreamSynchronize(s->stream));  // (an earlier call failed half way)
    std::memset(h, 0, sizeof(Ctl));
    h->y_len = s->y_len;
    h->draft_start = s->draft_start;
    h->len[0] = s->len[0];
    h->len[1] = s->len[1];
    h->n_src = s->n_src;
    h->n_max = s->n_max;
    h->alpha_fb = s->alpha_fb;
    h->alpha_rb = s->alpha_rb;
    h->seq = s->seq_issued;
    CtlArgs a = ctl_args(s);
    a.src = on_device(s, s->hy + first);
    a.dst = s->y + first;
    a.n = n;
    a.src2 = on_device(s, s->hsrc);
    a.dst2 = s->src;
    a.n2 = sources ? s->n_src : 0;
    HIPC(launch_ctl(a, s->stream));
    return BILD_OK;
}

// Thresholds live in the device control block so that captured passes need no new arguments.
int set_alpha(bild_state* s, float fb, float rb) {
    // compare bit patterns so that +-inf and every other value round-trip exactly
    if (std::memcmp(&fb, &s->alpha_fb, 4) == 0 && std::memcmp(&rb, &s->alpha_rb, 4) == 0) return BILD_OK;
    s->alpha_fb = fb;
    s->alpha_rb = rb;
    CtlArgs a = ctl_args(s);
    a.thresholds_only = 1;
    HIPC(launch_ctl(a, s->stream));
    return BILD_OK;
}

// Waits for the last pass; its policy kernel has mirrored the control block into pinned host memory.  The mirror's pass
// counter is polled first (the kernel writes it past the caches once its stores of the other words have been acknowledged): that
// sees the result a few microseconds before the stream's completion reaches the host.  If the count does not arrive in time (a failed
// launch) the stream is waited for as usual and the two counts are brought together again.
constexpr int kPassFailed = 1;  // (never leaves this file)
int pull_ctl(bild_state* s) {
    bool seen = false;
    {
        const int* seq = &s->hctl->seq;
        const auto t0 = std::chrono::steady_clock::now();
        for (unsigned spins = 1;; ++spins) {
            // acquire: the other words of the mirror are read after the count that was written behind them
            if (__atomic_load_n(seq, __ATOMIC_ACQUIRE) == s->seq_issued) {
                seen = true;
                break;
            }
            if ((spins & 1023) == 0 && std::chrono::steady_clock::now() - t0 > std::chrono::milliseconds(500)) break;
        }
    }
    if (!seen) {
        HIPC(hipStreamSynchronize(s->stream));
        s->seq_issued = __atomic_load_n(&s->hctl->seq, __ATOMIC_ACQUIRE);
    }
    if (s->hctl->res_flag & kFlagFailed) return kPassFailed;
    s->y_len = s->hctl->y_len;
    s->draft_start = s->hctl->draft_start;
    s->len[0] = s->hctl->len[0];
    s->len[1] = s->hctl->len[1];
    return BILD_OK;
}

}  // namespace

namespace bild {
// Key splits of one attention launch and whether the consumer projection merges them (`defer`).
// A workgroup's time grows with the K/V bytes it streams (about 2 us for 32 KiB, 3 us for 128 KiB, then in
// proportion).  Partials merged by the consumer cost no kernel: it works out the normalised weights once per
// (row, head) and then reads `splits` float4 per piece.  Measured on 512 keys of 64 dims, 24 layers: four
// splits of 32 KiB against none: 1055 / 1127 us per single-row pass, 1319 / 1351 us at 8 rows, 1585 / 1649 us at
// 16 rows, so the route is taken up to 16 rows (bounds: 8 splits, rows * heads <= 256, rows * heads * splits <= 1024
// - what the consumer's threads and its weight table in LDS hold).  The merge kernel costs about 5 us and therefore only pays when it
// brings a workgroup from above 160 KiB down to 128 KiB.
int pick_splits_raw(int d_head, int esz, int max_splits, int nkeys, int heads, int T, bool* defer) {
    const size_t per_head = (size_t)nkeys * d_head * 2 * esz;
    const size_t want = (size_t)(T <= 16 ? 32 : 128) << 10;
    auto fits = [&](int sp) { return sp <= max_splits && heads * sp <= 512; };
    int d_sp = 1;  // deferred route: as many splits as it allows, up to the wanted size
    // the consumer keeps one (row, head) pair per thread (at least 256 threads) and a table of splits x pairs
    // weights in the 4 KiB its smallest reduction area has
    const bool mergeable = T <= 16 && heads * T <= 256;
    while (per_head / d_sp > want && d_sp * 2 <= 8 && mergeable && heads * T * d_sp * 2 <= 1024 && fits(d_sp * 2)) d_sp *= 2;
    *defer = d_sp > 1;
    if (per_head / d_sp <= ((size_t)160 << 10)) return d_sp;
    int sp = d_sp;
    while (per_head / sp > ((size_t)128 << 10) && fits(sp * 2)) sp *= 2;
    if (sp > d_sp) *defer = false;
    return sp;
}

}  // namespace bild

namespace {

int pick_splits(const ModelState& M, int nkeys, int heads, int T, bool* defer) {
    return pick_splits_raw(M.m->cfg.d_head, M.m->esz(), M.max_splits, nkeys, heads, T, defer);
}

}  // namespace

namespace bild {

int pick_attn_waves(int dtype, int d_head, int T, int nkeys, int splits) {
    // one 32-key block per wave where possible, bounded by the LDS the merge needs
    const int blocks = ((nkeys + 31) / 32 + splits - 1) / splits;
    int nw = 1;
    while (nw < 8 && nw < blocks) nw *= 2;
    // at least four waves all the same: staging q is one piece per thread only from 256 threads on, and with fewer the
    // pieces are fetched one trip to memory after the other (measured: 1730 -> 1757 tokens/s on T5 shapes, whose caches
    // start short; eight waves cost more in the merge than they save)
    if (nw < 4) nw = 4;
    while (nw > 1 && attn_lds_bytes(dtype, d_head, T, nw) > 96 * 1024) nw /= 2;
    return nw;
}

}  // namespace bild

namespace {

GemmArgs gemm_base(const bild_model* m, const TMat& W, const float* x, int ldx, int T, const float* gain) {
    GemmArgs g;
    std::memset(&g, 0, sizeof(g));
    g.W = W;
    g.x = x;
    g.ldx = ldx;
    g.T = T;
    g.gain = gain;
    g.eps = m->cfg.norm_eps;
    g.d_head = m->cfg.d_head;
    g.i_dim = m->inner();
    g.act = m->cfg.act;
    g.vocab = m->cfg.vocab;
    return g;
}

template <class Launch>
int launch_profiled(bild_state* s, const bild_model* m, const TMat& W, int epi, Launch&& launch) {
    const int64_t bytes = (int64_t)W.n * W.k * m->esz();
    s->gemm_count += 1;
    s->stage_count += 1;
    s->gemm_bytes += bytes;
    if (s->prof_on && s->prof_used >= s->prof_cap) s->prof_dropped++;
    if (!s->prof_on || s->prof_used >= s->prof_cap) {
        HIPC(launch());
        return BILD_OK;
    }
    const int i = s->prof_used++;
    HIPC(hipEventRecord(s->prof_ev[2 * i], s->stream));
    HIPC(launch());
    HIPC(hipEventRecord(s->prof_ev[2 * i + 1], s->stream));
    bild_state::ProfRec r;
    r.model = (m == s->pair->m[1]) ? 1 : 0;
    r.cls = epi == EPI_LMHEAD ? 1 : 0;
    r.bytes = bytes;
    s->prof_rec.push_back(r);
    return BILD_OK;
}

int launch_gemm_profiled(bild_state* s, const bild_model* m, const GemmArgs& g) {
    return launch_profiled(s, m, g.W, g.epi, [&] { return launch_gemm(g, m->cfg.dtype, s->stream); });
}

int run_gemm(bild_state* s, const bild_model* m, GemmArgs& g) {
    gemm_pick_shape(g, m->cfg.dtype);
    return launch_gemm_profiled(s, m, g);
}

int emit_gemm(bild_state* s, const bild_model* m, GemmArgs& g) {
    gemm_pick_shape(g, m->cfg.dtype);
    return launch_gemm_profiled(s, m, g);
}

// `deferred` receives the number of key splits whose partials the following output projection must merge
// (1: the attention output is complete; null: it is to be).
int emit_attention(bild_state* s, const ModelState& M, AttnArgs& a, int nkeys, int* deferred) {
    const int dt = M.m->cfg.dtype;
    if (deferred) *deferred = 1;
    bool defer = false;
    a.splits = a.T > kMaxRows ? 1 : pick_splits(M, nkeys, a.heads, a.T, &defer);  // row blocks and key splits do not combine
    a.nw = pick_attn_waves(dt, a.d_head, std::min(a.T, kMaxRows), nkeys, a.splits);
    a.defer_merge = a.splits > 1 && defer && deferred;  // (null: the attention output is to be complete)
    if (a.defer_merge) *deferred = a.splits;
    s->stage_count += (a.splits > 1 && !a.defer_merge) ? 2 : 1;  // (the merge kernel is a stage of its own)
    if (!s->gemm_only) HIPC(launch_attention(a, dt, s->stream));
    return BILD_OK;
}

// Attention over a long cache whose workgroups join their keys themselves (attn_split.hip); 0: not made for it.
int emit_attention_split(bild_state* s, const ModelState& M, const AttnArgs& a, int nkeys, bool* done) {
    AttnSplitArgs b;
    std::memset((void*)&b, 0, sizeof(b));
    *done = false;
    if (M.m->cfg.dtype != BILD_DT_BF16 || a.rel_bias || a.T > kMaxRows || !s->split_part) return BILD_OK;
    attn_split_shape(a.heads, a.d_head, a.i_dim, a.vcap, nkeys, &b.splits, &b.waves);
    if (!b.splits) return BILD_OK;
    b.q = a.q; b.k = a.k; b.v = a.v; b.vcap = a.vcap; b.i_dim = a.i_dim; b.heads = a.heads; b.d_head = a.d_head; b.T = a.T;
    b.causal = a.causal; b.len_ptr = a.len_ptr; b.scale = a.scale;
    b.part = s->split_part; b.arrived = s->split_arrived;
    b.out = a.out; b.ob_t = a.ob_t;
    s->stage_count += 1;
    if (!s->gemm_only) HIPC(launch_attn_split(b, s->stream));
    *done = true;
    return BILD_OK;
}

// ---- bf16 passes over many rows (gemm_tile.hip): encoder, cross K/V, prompt prefill ----
struct TilePass {  // where one such pass works
    bild_state* s;
    const bild_model* m;
    int T;
    float *x, *q;
    char *xt, *at, *ht;
    float* ssq;
    int parts;  // partial sums of squares beside xt
    const double2* rope;
};

TileGemmArgs tile_base(const TilePass& p, const TMat& W, const char* in) {
    TileGemmArgs g;
    std::memset((void*)&g, 0, sizeof(g));
    g.W = W;
    g.xp = in;
    g.M = p.T;
    g.ssq = p.ssq;
    g.ssq_parts = p.parts;
    g.ssq_ld = p.T;
    g.eps = p.m->cfg.norm_eps;
    g.act = p.m->cfg.act;
    g.d_head = p.m->cfg.d_head;
    g.i_dim = p.m->inner();
    return g;
}

int run_tile(const TilePass& p, const TileGemmArgs& g) {
    p.s->gemm_count += 1;
    p.s->stage_count += 1;
    p.s->gemm_bytes += (int64_t)g.W.n * g.W.k * p.m->esz();
    HIPC(launch_gemm_tile(g, p.s->stream));
    return BILD_OK;
}

// Embedding: fp32 rows, their planes times `gain`, sums of squares.
int tile_embed(TilePass& p, const int* tokens, const int* base_ptr, const float* pe, const float* gain) {
    const bild_model_config& c = p.m->cfg;
    EmbedArgs e;
    std::memset((void*)&e, 0, sizeof(e));
    e.E = p.m->emb;
    e.tokens = tokens;
    e.base_ptr = base_ptr;
    e.T = p.T;
    e.d = c.d_model;
    e.vocab = c.vocab;
    e.tie_shift = c.tie_shift;
    e.sinusoidal = c.pos == BILD_POS_SINUSOIDAL;
    e.embed_scale = c.embed_scale;
    e.x = p.x;
    e.pe = pe;
    e.nx_gain = gain;
    e.nx_ssq = p.ssq;
    p.parts = 1;
    p.s->stage_count += 1;
    HIPC(launch_embed_tiles(e, p.xt, p.s->stream));
    return BILD_OK;
}

int tile_qkv(const TilePass& p, const TMat& W, void* k, void* v, int vcap, const int* pos_ptr) {
    TileGemmArgs g = tile_base(p, W, p.xt);
    g.epi = EPI_QKV;
    g.layer_n = W.n;
    g.q_dim = g.i_dim;
    g.q_out = p.q;
    g.k_cache = k;
    g.v_cache = v;
    g.vcap = vcap;
    g.pos_ptr = pos_ptr;
    g.rope = p.rope;
    return run_tile(p, g);
}

// x += in W^T, and the planes of the new x times the gain of the norm that reads it next
int tile_resid(TilePass& p, const TMat& W, const char* in, const float* next_gain) {
    TileGemmArgs g = tile_base(p, W, in);
    g.epi = EPI_RESID;
    g.x = p.x;
    g.ldx = p.m->cfg.d_model;
    g.np = p.xt;
    g.np_tk = p.m->cfg.d_model / 32;
    g.np_gain = next_gain;
    g.np_ssq = p.ssq;
    p.parts = tile_gemm_parts(g);
    return run_tile(p, g);
}

int tile_ffn(TilePass& p, const LayerW& L, const float* next_gain) {
    TileGemmArgs g = tile_base(p, L.win, p.xt);
    g.epi = EPI_ACT;
    g.np = p.ht;
    g.np_tk = p.m->cfg.d_ff / 32;
    int rc = run_tile(p, g);
    if (rc) return rc;
    return tile_resid(p, L.wout, p.ht, next_gain);
}

// Prompt rows y[len .. len+T) of a bf16 decoder-only model: fills the caches of all layers.  What lies behind the last
// layer's K/V projection has no reader (the next token comes from a later pass) unless the rows are an early-exit trunk's.
int emit_prefill(bild_state* s, int w, int T) {
    ModelState& M = s->ms[w];
    const bild_model* m = M.m;
    const bild_model_config& c = m->cfg;
    const int* len_ptr = &s->ctl->len[w];
    const int trunk = s->pair->trunk_layers, layer0 = (trunk > 0 && w == 1) ? trunk : 0;
    const bool keeps_hidden = trunk > 0 && w == 0;
    TilePass p = {s, m, T, M.x, M.q, M.xt, (char*)M.a, (char*)M.h, M.ssq_t, 0, M.rope};
    if (T > M.rows_t) return BILD_ECAP;
    int rc;
    if (layer0 > 0) {  // the hidden state the trunk left for these rows
        RowCopyArgs r;
        std::memset((void*)&r, 0, sizeof(r));
        r.src = s->trunk_x;
        r.src_row_ptr = len_ptr;
        r.dst = M.x;
        r.d = c.d_model;
        r.T = T;
        s->stage_count += 1;
        HIPC(launch_row_tiles(r, m->dec[layer0].ln1, M.xt, M.ssq_t, s->stream));
        p.parts = 1;
    } else {
        rc = tile_embed(p, s->y, len_ptr, M.pe, m->dec[0].ln1);
        if (rc) return rc;
    }
    for (int l = layer0; l < c.n_dec_layers; ++l) {
        const LayerW& L = m->dec[l];
        const bool last = l + 1 == c.n_dec_layers;
        const size_t off = (size_t)l * s->cap_len * m->inner() * m->esz();
        rc = tile_qkv(p, L.wqkv, M.kcache + off, M.vcache + off, s->cap_len, len_ptr);
        if (rc) return rc;
        if (last && !keeps_hidden) break;
        AttnArgs a;
        std::memset((void*)&a, 0, sizeof(a));
        a.q = M.q; a.k = M.kcache + off; a.v = M.vcache + off; a.ob_t = p.at;
        a.T = T; a.heads = c.n_heads; a.d_head = c.d_head; a.i_dim = m->inner();
        a.causal = 1;
        a.len_ptr = len_ptr;
        a.rel_bias = m->dec_rel;
        a.rel_d = c.rel_max_dist;
        a.vcap = s->cap_len;
        a.scale = 1.f / std::sqrt((float)c.d_head);
        s->stage_count += 1;
        HIPC(launch_attention_tile(a, s->stream));
        rc = tile_resid(p, L.wo, p.at, L.ln2);
        if (rc) return rc;
        rc = tile_ffn(p, L, last ? m->dec_final : m->dec[l + 1].ln1);
        if (rc) return rc;
    }
    if (keeps_hidden) {  // (as in emit_layers)
        RowCopyArgs r;
        std::memset((void*)&r, 0, sizeof(r));
        r.src = M.x;
        r.dst = s->trunk_x;
        r.dst_row_ptr = len_ptr;
        r.d = c.d_model;
        r.T = T;
        s->stage_count += 1;
        HIPC(launch_row_copy(r, s->stream));
    }
    return BILD_OK;
}

// ---- bf16 passes of a few rows on gemm_thin.hip: the planes lie where the row-major ones do (M.xb, M.ab, M.hb) ----
int run_thin(bild_state* s, const bild_model* m, const ThinArgs& g) {
    return launch_profiled(s, m, g.W, g.epi, [&] { return launch_gemm_thin(g, s->stream); });
}

ThinArgs thin_base(const bild_state* s, int w, int T, const TMat& W, const void* in, int parts) {
    const ModelState& M = s->ms[w];
    const bild_model_config& c = M.m->cfg;
    ThinArgs g;
    std::memset((void*)&g, 0, sizeof(g));
    g.W = W;
    g.xp = (const char*)in;
    g.T = T;
    g.ssq = M.ssq;
    g.ssq_parts = parts;
    g.eps = c.norm_eps;
    g.act = c.act;
    g.d_head = c.d_head;
    g.i_dim = M.m->inner();
    g.pos_ptr = &s->ctl->len[w];
    g.sums = s->thin_sums;
    g.arrived = s->thin_arrived;
    return g;
}

// Passes of 2 .. kMaxRows rows of models whose planes the thin GEMM reads; `parts` receives the number of partial sums of squares
// beside the final hidden state's planes (M.xb, times the final norm's gain).
int emit_thin(bild_state* s, int w, int T, int key_hint, bool reads_hidden, int* parts_out) {
    ModelState& M = s->ms[w];
    const bild_model* m = M.m;
    const bild_model_config& c = m->cfg;
    const int d = c.d_model, I = m->inner();
    const size_t esz = m->esz();
    const int* len_ptr = &s->ctl->len[w];
    const int trunk = s->pair->trunk_layers, layer0 = (trunk > 0 && w == 1) ? trunk : 0;
    const bool keeps_hidden = trunk > 0 && w == 0;
    int parts = 1;
    s->stage_count += 1;
    if (!s->gemm_only) {
        if (layer0 > 0) {  // the hidden state the trunk left for these rows
            RowCopyArgs r;
            std::memset((void*)&r, 0, sizeof(r));
            r.src = s->trunk_x;
            r.src_row_ptr = len_ptr;
            r.dst = M.x;
            r.d = d;
            r.T = T;
            HIPC(launch_row_tiles(r, m->dec[layer0].ln1, (char*)M.xb, M.ssq, s->stream));
        } else {
            EmbedArgs e;
            std::memset((void*)&e, 0, sizeof(e));
            e.E = m->emb;
            e.tokens = s->y;
            e.base_ptr = len_ptr;
            e.T = T;
            e.d = d;
            e.vocab = c.vocab;
            e.tie_shift = c.tie_shift;
            e.sinusoidal = c.pos == BILD_POS_SINUSOIDAL;
            e.embed_scale = c.embed_scale;
            e.x = M.x;
            e.pe = M.pe;
            e.nx_gain = m->dec[0].ln1;
            e.nx_ssq = M.ssq;
            HIPC(launch_embed_tiles(e, (char*)M.xb, s->stream));
        }
    }
    auto resid = [&](const TMat& W, const void* in, const float* next_gain) {
        ThinArgs g = thin_base(s, w, T, W, in, 0);
        g.epi = EPI_RESID;
        g.out = M.x;
        g.ldo = d;
        g.np = (char*)M.xb;
        g.np_tk = d / 32;
        g.np_gain = next_gain;
        g.np_ssq = M.ssq;
        parts = W.tn;
        return run_thin(s, m, g);
    };
    auto attend = [&](void* k, void* v, int vcap, bool causal, int nkeys) {
        AttnArgs a;
        std::memset((void*)&a, 0, sizeof(a));
        a.q = M.q; a.k = k; a.v = v; a.vcap = vcap;
        a.T = T; a.heads = c.n_heads; a.d_head = c.d_head; a.i_dim = I;
        a.causal = causal;
        a.len_ptr = causal ? len_ptr : &s->ctl->n_src;
        if (causal) { a.rel_bias = m->dec_rel; a.rel_d = c.rel_max_dist; }
        a.part_o = M.att_o; a.part_ml = M.att_ml;
        a.scale = 1.f / std::sqrt((float)c.d_head);
        a.ob_t = (char*)M.ab;
        bool done = false;
        const int rc = emit_attention_split(s, M, a, nkeys, &done);
        return rc || done ? rc : emit_attention(s, M, a, nkeys, nullptr);
    };
    int rc;
    for (int l = layer0; l < c.n_dec_layers; ++l) {
        const LayerW& L = m->dec[l];
        const bool last = l + 1 == c.n_dec_layers;
        const size_t off = (size_t)l * s->cap_len * I * esz, coff = (size_t)l * s->cap_src * I * esz;
        ThinArgs g = thin_base(s, w, T, L.wqkv, M.xb, parts);
        g.epi = EPI_QKV;
        g.q_dim = I;
        g.q_out = M.q;
        g.k_cache = M.kcache + off;
        g.v_cache = M.vcache + off;
        g.vcap = s->cap_len;
        g.rope = M.rope;
        if ((rc = run_thin(s, m, g))) return rc;
        if (last && !reads_hidden && !keeps_hidden) break;
        if ((rc = attend(M.kcache + off, M.vcache + off, s->cap_len, true, key_hint))) return rc;
        if ((rc = resid(L.wo, M.ab, c.cross_attn ? L.lnc : L.ln2))) return rc;
        if (c.cross_attn) {
            ThinArgs q = thin_base(s, w, T, L.cwq, M.xb, parts);
            q.epi = EPI_STORE;
            q.out = M.q;
            q.ldo = I;
            if ((rc = run_thin(s, m, q))) return rc;
            if ((rc = attend(M.ck + coff, M.cv + coff, s->cap_src, false, s->n_src))) return rc;
            if ((rc = resid(L.cwo, M.ab, L.ln2))) return rc;
        }
        ThinArgs f = thin_base(s, w, T, L.win, M.xb, parts);
        f.epi = EPI_ACT;
        f.np = (char*)M.hb;
        f.np_tk = c.d_ff / 32;
        if ((rc = run_thin(s, m, f))) return rc;
        if ((rc = resid(L.wout, M.hb, last ? m->dec_final : m->dec[l + 1].ln1))) return rc;
    }
    if (keeps_hidden) s->stage_count += 1;
    if (keeps_hidden && !s->gemm_only) {  // remember what the trunk produced for these positions
        RowCopyArgs r;
        std::memset((void*)&r, 0, sizeof(r));
        r.src = M.x;
        r.dst = s->trunk_x;
        r.dst_row_ptr = len_ptr;
        r.d = d;
        r.T = T;
        HIPC(launch_row_copy(r, s->stream));
    }
    *parts_out = parts;
    return BILD_OK;
}

// Embedding and all decoder layers of model w over rows y[len .. len+T).
// `reads_hidden`: an LM head follows (without one, nothing reads what lies behind the last layer's K/V projection, unless
// the rows are an early-exit trunk's).
int emit_layers(bild_state* s, int w, int T, int key_hint, bool reads_hidden, bool head_reads_parts, int* xb_parts_out, float** x_out, bool* parts_pending) {
    ModelState& M = s->ms[w];
    const bild_model* m = M.m;
    const bild_model_config& c = m->cfg;
    const int d = c.d_model, I = m->inner(), F = c.d_ff, dt = c.dtype;
    const size_t esz = m->esz();
    const int* len_ptr = &s->ctl->len[w];
    EmbedArgs e;
    std::memset((void*)&e, 0, sizeof(e));
    e.E = m->emb;
    e.tokens = s->y;
    e.base_ptr = len_ptr;
    e.T = T;
    e.d = d;
    e.vocab = c.vocab;
    e.tie_shift = c.tie_shift;
    e.sinusoidal = c.pos == BILD_POS_SINUSOIDAL;
    e.embed_scale = c.embed_scale;
    e.x = M.x;
    e.pe = M.pe;
    // Early-exit pair: the large model's pass starts from the hidden state the trunk (model 0) left for these
    // rows and runs the layers above the trunk only.
    const int trunk = s->pair->trunk_layers;
    const bool above_trunk = trunk > 0 && w == 1;
    const int layer0 = above_trunk ? trunk : 0;
    // Passes of a few rows of a bf16 model: every producer leaves its output as high / low bf16 planes for the
    // projection that follows (x times that projection's norm gain, the attention output, the FFN hidden state).
    // Measured (us per large-model pass, planes / fp32 hand-over): 1024-wide model 2 rows 1002 / 947, 5 rows 1121 / 1148,
    // 16 rows 1332 / 1429, 32 rows 1831 / 2018; 4096-wide model 2 rows 3398 / 3487, 11 rows 3904 / 4326, 32 rows 5321 / 6384.
    // Below five rows the narrow models keep the kernels specialised for one and for two to four rows.
    const int planes_from = s->pre_min_rows > 0 ? s->pre_min_rows : (d >= 2048 ? 2 : 5);
    const bool planes = dt == BILD_DT_BF16 && T >= planes_from && T <= kMaxRows && M.xb != nullptr;
    uint16_t *xb_hi = M.xb, *xb_lo = M.xb ? M.xb + (size_t)kMaxRows * d : nullptr;
    uint16_t *ab_hi = M.ab, *ab_lo = M.ab ? M.ab + (size_t)kMaxRows * I : nullptr;
    uint16_t *hb_hi = M.hb, *hb_lo = M.hb ? M.hb + (size_t)kMaxRows * F : nullptr;
    int xb_parts = 0;  // > 0: xb holds the current residual stream, with this many partial sums of squares in M.ssq
    // the norm gain in front of the projection that reads the residual stream next
    auto set_in = [&](GemmArgs& g) {  // input from the residual-stream planes, if they are current
        if (xb_parts > 0) { g.xb_hi = xb_hi; g.xb_lo = xb_lo; g.ssq_part = M.ssq; g.ssq_parts = xb_parts; }
    };
    auto set_out = [&](GemmArgs& g, const float* next_gain) {  // residual epilogue: also planes for the next projection
        if (!planes) return;
        g.nx_hi = xb_hi; g.nx_lo = xb_lo; g.nx_gain = next_gain; g.nx_ssq = M.ssq; g.nx_ld = d;
    };
    auto after_out = [&](const GemmArgs& g) {  // (after gemm_pick_shape) one partial per wave that owns output tiles
        xb_parts = planes ? (int)gemm_num_blocks(g) * (g.nwv / g.wk) : 0;
        if (xb_parts > kMaxSsqParts) xb_parts = 0;  // more than a consumer adds up: the next projection converts x itself
    };
    // The FFN output projection of a narrow model at one to four rows (64 feature tiles x thousands of inputs: too few
    // workgroups with too long a stream each) is cut into kPartSlices slices of its inputs; the next layer's first
    // projection (or the LM head of a single-row pass) adds the slices to the residual stream while staging and leaves the
    // sum in the other of two residual buffers.  Measured on the T5-large shape: see the design notes.
    const int kt = dt == BILD_DT_BF16 ? 32 : 16;
    const bool split_ffn = !planes && T <= 4 && d <= s->ksplit_max_d && s->ksplit_min_f > 0 && F >= s->ksplit_min_f &&
                           (F / kt) % kPartSlices == 0 && (T == 1 || ((d / 4) % 64 == 0 && (F / kPartSlices / 4) % 64 == 0)) && M.px != nullptr;
    float *xcur = M.x, *xoth = M.x2;
    // > 0: the residual stream is xcur + that many partial results in pend_buf (slices of a split FFN output projection,
    // or one per head of an attention fused with its output projection), to be added by the next reader
    int pending = 0;
    const float* pend_buf = nullptr;
    auto set_parts_in = [&](GemmArgs& g) {
        if (!pending) return;
        g.px = pend_buf; g.px_stride = (int64_t)kMaxRows * d; g.pn = pending; g.x_out = xoth;
    };
    auto after_parts_in = [&]() {
        if (!pending) return;
        std::swap(xcur, xoth);
        pending = 0;
    };
    // Single-row passes of the narrow models: attention and its output projection as one kernel per (head, column
    // group); the next projection adds one partial result per head.  A head's cache must be small enough for one
    // workgroup (every column group repeats the head's attention).
    const bool fuse_shape = s->fuse_attn && T == 1 && !planes && d <= 1024 && c.n_heads <= kMaxHeadParts && c.d_head <= 64 &&
                            c.d_head % kt == 0 && M.pxh != nullptr;
    auto fuse_attention = [&](AttnArgs& a, const TMat& wo, int nkeys) -> int {  // 1: launched fused, 0: not applicable, < 0: error
        // (measured on the T5-large shape: 64 keys 6.1 us against 4.7 + 3.5 for attention and projection apart; 512 keys,
        // 128 KiB per head, 11.3 us against 5.1 + 4.5)
        if (!fuse_shape || (size_t)nkeys * c.d_head * 2 * esz > (size_t)s->fuse_max_kv) return 0;
        a.splits = 1;
        a.defer_merge = 0;
        a.nw = pick_attn_waves(dt, a.d_head, T, nkeys, 1);
        const int maxn = dt == BILD_DT_BF16 ? 4 : 2;
        int cg = std::max(1, std::min(wo.tn, 64 / c.n_heads));
        while (cg < wo.tn && ((wo.tn + cg - 1) / cg + a.nw - 1) / a.nw > maxn) cg *= 2;
        if (((wo.tn + cg - 1) / cg + a.nw - 1) / a.nw > maxn) return 0;
        a.wo = wo;
        a.proj_out = M.pxh;
        a.proj_stride = (int64_t)kMaxRows * d;
        a.cgroups = cg;
        a.d_model = d;
        s->stage_count += 1;
        if (!s->gemm_only && launch_attention_proj(a, dt, s->stream) != hipSuccess) return BILD_EHIP;
        pending = kMaxHeadParts;
        pend_buf = M.pxh;
        return 1;
    };
    if (planes && !above_trunk) {
        e.nx_hi = xb_hi; e.nx_lo = xb_lo; e.nx_gain = m->dec[layer0].ln1; e.nx_ssq = M.ssq;
        xb_parts = kEmbedSsqParts;
    }
    // Single-row passes: the first projection gathers the row from the embedding matrix itself (no embedding kernel).
    // The table of positions must exist where positions are added (the kernel does not evaluate sines).
    // Every workgroup of that projection repeats the gather, so it is taken only where one round of two pieces per
    // thread covers the row (a 4096-wide row in workgroups of two waves would be four dependent rounds: measured slower).
    bool embed_in_proj = s->fuse_embed && T == 1 && !planes && !above_trunk && (!e.sinusoidal || e.pe != nullptr) &&
                         layer0 < c.n_dec_layers;
    if (embed_in_proj) {
        GemmArgs probe = gemm_base(m, m->dec[layer0].wqkv, M.x, d, T, m->dec[layer0].ln1);
        probe.epi = EPI_QKV;
        gemm_pick_shape(probe, dt);
        embed_in_proj = d / 4 <= 2 * 64 * probe.nwv && probe.W.k <= probe.kc;
    }
    if (!embed_in_proj) s->stage_count += 1;  // embedding or the trunk's rows
    if (!s->gemm_only && !embed_in_proj) {
        if (above_trunk) {
            RowCopyArgs rc;
            std::memset((void*)&rc, 0, sizeof(rc));
            rc.src = s->trunk_x;
            rc.src_row_ptr = len_ptr;
            rc.dst = M.x;
            rc.d = d;
            rc.T = T;
            HIPC(launch_row_copy(rc, s->stream));
        } else {
            HIPC(launch_embed(e, dt, s->stream));
        }
    }
    const float att_scale = 1.f / std::sqrt((float)c.d_head);
    int merge_splits = 1;
    for (int l = layer0; l < c.n_dec_layers; ++l) {
        const LayerW& L = m->dec[l];
        char* kc = M.kcache + (size_t)l * s->cap_len * I * esz;
        char* vc = M.vcache + (size_t)l * s->cap_len * I * esz;
        int fused = 0;  // this attention ran together with its output projection
        {
            GemmArgs g = gemm_base(m, L.wqkv, xcur, d, T, L.ln1);
            set_parts_in(g);
            g.epi = EPI_QKV;
            g.q_dim = I;
            g.q_out = M.q;
            g.k_cache = kc;
            g.v_cache = vc;
            g.vcap = s->cap_len;
            g.pos_ptr = len_ptr;
            g.rope = M.rope;
            set_in(g);
            if (embed_in_proj && l == layer0) {
                g.e_w = e.E.w; g.e_tk = e.E.tk; g.e_tokens = e.tokens; g.e_base_ptr = e.base_ptr; g.e_base_add = e.base_add;
                g.e_vocab = e.vocab; g.e_shift = e.tie_shift; g.e_scale = e.embed_scale; g.e_pe = e.sinusoidal ? e.pe : nullptr;
                g.x_out = xcur;  // (= g.x: the row is written where the embedding kernel would have left it)
            }
            int rc = emit_gemm(s, m, g);
            if (rc) return rc;
            after_parts_in();
            if (!reads_hidden && l + 1 == c.n_dec_layers && !(trunk > 0 && w == 0)) break;
        }
        {
            AttnArgs a;
            std::memset((void*)&a, 0, sizeof(a));
            a.q = M.q; a.k = kc; a.v = vc; a.out = M.a;
            a.T = T; a.heads = c.n_heads; a.d_head = c.d_head; a.i_dim = I;
            a.causal = 1;
            a.len_ptr = len_ptr;
            a.rel_bias = m->dec_rel;
            a.rel_d = c.rel_max_dist;
            a.vcap = s->cap_len;
            a.part_o = M.att_o; a.part_ml = M.att_ml;
            a.scale = att_scale;
            if (planes) { a.ob_hi = ab_hi; a.ob_lo = ab_lo; }
            fused = fuse_attention(a, L.wo, key_hint);
            if (fused < 0) return fused;
            if (!fused) {
                bool done = false;
                // (16 layers 2048 wide with the projection that joins the keys / with this kernel, 104, 340, 1064, 4137 keys: 632 / 607,
                // 642 / 642, 670 / 659, 777 / 756 us a pass; 8 layers 4096 wide 759 / 743, 767 / 760, 785 / 771, 845 / 843)
                // (it writes fp32 rows, not the planes that the projection reads where producers hand those over)
                int rc = T == 1 && d > 1024 && !planes ? emit_attention_split(s, M, a, key_hint, &done) : BILD_OK;
                if (done) merge_splits = 1;
                if (rc == BILD_OK && !done) rc = emit_attention(s, M, a, key_hint, &merge_splits);
                if (rc) return rc;
            }
        }
        if (!fused) {
            GemmArgs g = gemm_base(m, L.wo, M.a, I, T, nullptr);
            g.epi = EPI_RESID;
            g.out = xcur;
            g.ldo = d;
            if (merge_splits > 1) { g.mg_splits = merge_splits; g.mg_o = M.att_o; g.mg_ml = M.att_ml; g.mg_heads = c.n_heads; }
            else if (planes) { g.xb_hi = ab_hi; g.xb_lo = ab_lo; }
            set_out(g, c.cross_attn ? L.lnc : L.ln2);
            int rc = emit_gemm(s, m, g);
            if (rc) return rc;
            after_out(g);
        }
        if (c.cross_attn) {
            {
                GemmArgs g = gemm_base(m, L.cwq, xcur, d, T, L.lnc);
                g.epi = EPI_STORE;
                g.out = M.q;
                g.ldo = I;
                set_in(g);
                set_parts_in(g);
                int rc = emit_gemm(s, m, g);
                if (rc) return rc;
                after_parts_in();
            }
            {
                AttnArgs a;
                std::memset((void*)&a, 0, sizeof(a));
                a.q = M.q;
                a.k = M.ck + (size_t)l * s->cap_src * I * esz;
                a.v = M.cv + (size_t)l * s->cap_src * I * esz;
                a.vcap = s->cap_src;
                a.out = M.a;
                a.T = T; a.heads = c.n_heads; a.d_head = c.d_head; a.i_dim = I;
                a.causal = 0;
                a.len_ptr = &s->ctl->n_src;
                a.part_o = M.att_o; a.part_ml = M.att_ml;
                a.scale = att_scale;
                if (planes) { a.ob_hi = ab_hi; a.ob_lo = ab_lo; }
                fused = fuse_attention(a, L.cwo, s->n_src);
                if (fused < 0) return fused;
                if (!fused) {
                    int rc = emit_attention(s, M, a, s->n_src, &merge_splits);
                    if (rc) return rc;
                }
            }
            if (!fused) {
                GemmArgs g = gemm_base(m, L.cwo, M.a, I, T, nullptr);
                g.epi = EPI_RESID;
                g.out = xcur;
                g.ldo = d;
                if (merge_splits > 1) { g.mg_splits = merge_splits; g.mg_o = M.att_o; g.mg_ml = M.att_ml; g.mg_heads = c.n_heads; }
                else if (planes) { g.xb_hi = ab_hi; g.xb_lo = ab_lo; }
                set_out(g, L.ln2);
                int rc = emit_gemm(s, m, g);
                if (rc) return rc;
                after_out(g);
            }
        }
        {
            GemmArgs g = gemm_base(m, L.win, xcur, d, T, L.ln2);
            g.epi = EPI_ACT;
            g.out = M.h;
            g.ldo = F;
            set_in(g);
            set_parts_in(g);
            // the hidden state goes on as planes only if this projection itself reads planes (one kernel family per pass)
            const bool h_planes = planes && g.xb_hi != nullptr;
            if (h_planes) { g.nx_hi = hb_hi; g.nx_lo = hb_lo; g.nx_ld = F; }
            int rc = emit_gemm(s, m, g);
            if (rc) return rc;
            after_parts_in();
            GemmArgs g2 = gemm_base(m, L.wout, M.h, F, T, nullptr);
            g2.epi = EPI_RESID;
            g2.out = xcur;
            g2.ldo = d;
            if (split_ffn && (l + 1 < c.n_dec_layers || head_reads_parts)) {
                g2.epi = EPI_PART;
                g2.out = M.px;
                g2.ksplit = kPartSlices;
                g2.part_stride = (int64_t)kMaxRows * d;
                pending = kPartSlices;
                pend_buf = M.px;
            }
            if (h_planes) { g2.xb_hi = hb_hi; g2.xb_lo = hb_lo; }
            // the next reader of the residual stream: the following layer's first norm, or the final norm (LM head)
            if (h_planes) set_out(g2, l + 1 < c.n_dec_layers ? m->dec[l + 1].ln1 : m->dec_final);
            rc = emit_gemm(s, m, g2);
            if (rc) return rc;
            if (h_planes) after_out(g2); else xb_parts = 0;
        }
    }
    if (trunk > 0 && w == 0) s->stage_count += 1;
    if (trunk > 0 && w == 0 && !s->gemm_only) {  // remember what the trunk produced for these positions
        RowCopyArgs rc;
        std::memset((void*)&rc, 0, sizeof(rc));
        rc.src = xcur;
        rc.dst = s->trunk_x;
        rc.dst_row_ptr = len_ptr;
        rc.d = d;
        rc.T = T;
        HIPC(launch_row_copy(rc, s->stream));
    }
    *xb_parts_out = xb_parts;
    *x_out = xcur;
    *parts_pending = pending > 0;
    return BILD_OK;
}

}  // namespace

namespace bild {

// LM heads whose workgroups stay for the whole sweep (head.hip).  One row of a matrix that a chip full of short workgroups reads in
// 15 us loses 1 us there.  us per pass before / with it: 32 128 ids, T5-small shape one row 97.9 / 99.1, T5-large shape 1, 3, 8, 11 rows
// 454 / 455, 463 / 464, 480 / 480, 552 / 551; 250 112 ids 153 / 144, 543 / 527, 555 / 535, 570 / 549, 647 / 626.  (A head alone, 32 000 x 2048,
// 1, 8, 21, 32 rows: 28.4, 31.7, 52.4, 60.8 / 27.7, 30.1, 33.9, 36.1.)
static bool takes_sweep(const bild_model* m, int rows) {
    const size_t bytes = (size_t)m->head.tn * m->head.tk * kTileBytes;
    return m->cfg.dtype == BILD_DT_BF16 && rows > 0 && (rows > 1 || bytes >= (size_t)96 << 20);
}

// Passes on the thin GEMM (gemm_thin.hip): where a projection has about a feature tile per compute unit (4096 wide) always, in
// narrower models where the rows outweigh that.  us per pass, row-major planes / thin, over 1024 keys, 8 layers of the 7B shape, 2, 4, 8,
// 12, 16, 17, 32 rows: 869 / 838, 884 / 841, 931 / 844, 1006 / 890, 1053 / 893, 1128 / 971, 1341 / 982; 16 layers 2048 wide, 2, 4, 8, 16, 32 rows:
// 736 / 797, 790 / 800, 859 / 808, 957 / 881, 1328 / 1105; T5-large shape 16, 17, 24, 32 rows: 1242 / 1258, 1474 / 1563, 1645 / 1564, 1690 / 1571.
static bool takes_thin(const bild_state* s, int w, int T) {
    const bild_model_config& c = s->ms[w].m->cfg;
    const int from = s->thin_min_rows > 0 ? s->thin_min_rows : c.d_model >= 4096 ? 2 : c.d_model >= 2048 ? 5 : 24;
    // (a reader adds kMaxSsqParts sums of squares of sixteen features at most)
    return c.dtype == BILD_DT_BF16 && T >= std::max(2, from) && T <= kMaxRows && c.d_model <= 16 * kMaxSsqParts;
}

// Counts the passes of model w with room for T rows.
static unsigned* pass_turn(const bild_state* s, int w, int T) { return s->pass_sync + kPassSyncWords + w * kPassRooms + pass_room_index(T); }
static_assert(2 * kPassRooms <= kPassTurnWords, "a word for each model's rooms");
// Counts what has started of its passes with the head inside (PassHead::started).
static unsigned* pass_heads(const bild_state* s, int w) { return s->pass_sync + kPassSyncWords + kPassTurnWords + w * kPassHeadWords; }

static bool two_tiles(const bild_state* s, int w, int T) {
    const ModelState& M = s->ms[w];
    const bild_model_config& c = M.m->cfg;
    return M.pass_wide && wide_two(c.d_model, c.n_heads, c.d_ff, M.m->gated(), M.pass_groups, s->len[w] + T);
}

// One decoder pass of model w over rows y[len .. len+T): embed, layers, and (lm_rows > 0)
// the LM head over the last lm_rows rows followed by the policy `mode`; lm_rows == 0
// only advances the cache (catch-up / prefill).
// `one`: as the pass kernel (takes_one_kernel).
int decoder_pass(bild_state* s, int w, int T, int lm_rows, int mode, int key_hint, bool one) {
    ModelState& M = s->ms[w];
    const bild_model* m = M.m;
    const bild_model_config& c = m->cfg;
    const int d = c.d_model, dt = c.dtype;
    const int* len_ptr = &s->ctl->len[w];
    s->stage_count = 0;
    int xb_parts = 0;  // > 0: the final hidden state also sits in M.xb as bf16 planes (times the final norm's gain)
    float* xfin = M.x;  // the residual stream after the last layer ...
    int thin_parts = 0;  // > 0: the final hidden state lies in M.xb as tile planes (times the final norm's gain)
    bool parts = false; // ... to which the partial results in M.px are still to be added (split FFN output projection)
    if (one) {
        const int trunk = s->pair->trunk_layers, layer0 = w == 1 ? trunk : 0;
        PassArgs p;
        std::memset((void*)&p, 0, sizeof(p));
        p.layers = M.pass_layers + layer0;
        p.n_layers = c.n_dec_layers - layer0;
        p.T = T; p.d = d; p.heads = c.n_heads; p.I = m->inner(); p.F = c.d_ff; p.act = c.act; p.cross = c.cross_attn;
        p.emb = layer0 ? nullptr : m->emb.w;
        p.tokens = s->y;
        p.pe = M.pe;
        p.x_in = s->trunk_x;
        p.vocab = c.vocab; p.tie_shift = c.tie_shift; p.embed_scale = c.embed_scale;
        p.len_ptr = len_ptr; p.nsrc_ptr = &s->ctl->n_src;
        p.vcap = s->cap_len; p.scap = s->cap_src;
        p.rel_bias = m->dec_rel; p.rel_d = c.rel_max_dist;
        p.att_scale = 1.f / std::sqrt((float)c.d_head); p.eps = c.norm_eps;
        p.x_out = M.x;
        p.x_keep = trunk > 0 && w == 0 ? s->trunk_x : nullptr;
        const bool die = T <= M.pass_die_rows;
        p.die = die;
        p.room = 1 << pass_room_index(T);
        p.f32 = dt == BILD_DT_F32;
        p.at = pass_plan(p.room, d, p.I, p.F, p.f32, M.pass_wide);
        p.turn = pass_turn(s, w, T);
        p.scratch = M.pass_turns[pass_room_index(T)];
        p.sync = s->pass_sync;
        p.spins = s->pass_spins;
        s->stage_count += 1;
        const size_t head = lm_rows > 0 ? (size_t)c.vocab * d * m->esz() : 0;
        p.last = !M.pass_wide && pass_last(d, c.d_ff, m->gated(), T, p.n_layers * m->layer_weight_bytes() + head);
        p.groups = die ? M.pass_die_groups : p.last ? pass_groups(d, c.n_heads, c.d_head, c.d_ff, m->gated(), s->cus, true) : M.pass_groups;
        p.wide = M.pass_wide;
        p.two = two_tiles(s, w, T);
        p.rope = M.rope;
        PassHead in;
        const bool inside = die && T == 1 && lm_rows == 1 && mode != 3 && !s->debug_logits && s->top_p == 0.f;  // (pass_head.h)
        if (inside) {
            std::memset((void*)&in, 0, sizeof(in));
            in.w = m->head.w;
            in.tn = m->head.tn;
            in.vocab = c.vocab;
            in.gain = m->dec_final;
            in.scale = c.logit_scale;
            in.started = pass_heads(s, w);
            pass_head_plan(in, p.at, d, p.f32, s->cus);
            FinishArgs& f = in.f;
            f.ctl = s->ctl;
            f.y = s->y;
            f.which = w;
            f.rows_consumed = T;
            f.y_cap = s->max_len;
            f.host_mirror = s->hctl_dev;
            f.sync = s->pass_sync;
            f.turn = pass_turn(s, w, T);
            f.T = 1;
            f.mode = mode;
        }
        HIPC(M.pass_wide ? launch_wide(p, s->stream) : launch_pass(p, inside ? &in : nullptr, die ? s->cus : p.groups, s->stream));
        if (inside) return BILD_OK;
        // Rows wider than the sweep of the vocabulary takes, from five on: as tile planes for the thin GEMM.  (The entry points, whose call is the head alone, ask
        // for 16 MB of matrix with five to eight rows, see head_route; a review of eight rows of two layers with that line / with none, us:
        // 2560 wide, 700, 1500, 2500 ids 131.3, 131.6, 132.1 / 130.1, 130.2, 131.4, 4096 wide 201.0, 200.7, 202.7 / 200.1, 199.0, 200.9.)
        if (lm_rows > 4 && d > 2048 && dt == BILD_DT_BF16) {
            RowCopyArgs r;
            std::memset((void*)&r, 0, sizeof(r));
            r.src = M.x;
            r.d = d;
            r.T = T;
            s->stage_count += 1;
            HIPC(launch_row_tiles(r, m->dec_final, (char*)M.xb, M.ssq, s->stream));
            thin_parts = 1;
        }
    } else if (takes_thin(s, w, T)) {
        const int rc = emit_thin(s, w, T, key_hint, lm_rows > 0, &thin_parts);
        if (rc) return rc;
    } else if (dt == BILD_DT_BF16 && T > kMaxRows) {
        if (lm_rows > 0) return BILD_EINVAL;
        const int rc = emit_prefill(s, w, T);
        if (rc) return rc;
    } else {
        // a single-row pass whose LM head is the one-row kernel with one feature tile per wave can add them itself
        const bool head_reads_parts = T == 1 && lm_rows == 1 && s->pair->trunk_layers == 0 && m->head.tn < 8192;
        int rc = emit_layers(s, w, T, key_hint, lm_rows > 0, head_reads_parts, &xb_parts, &xfin, &parts);
        if (rc) return rc;
    }
    FinishArgs f;
    std::memset((void*)&f, 0, sizeof(f));
    f.ctl = s->ctl;
    f.y = s->y;
    f.which = w;
    f.rows_consumed = T;
    f.y_cap = s->max_len;
    f.host_mirror = s->hctl_dev;
    if (one) {
        f.sync = s->pass_sync;
        f.turn = pass_turn(s, w, T);
    }
    if (lm_rows > 0 && thin_parts > 0) {
        ThinArgs g = thin_base(s, w, T, m->head, M.xb, thin_parts);
        g.epi = EPI_LMHEAD;
        g.first = T - lm_rows;
        g.scale = c.logit_scale;
        g.vocab = c.vocab;
        g.y = s->y;
        g.ylen_ptr = &s->ctl->y_len;
        g.part = M.part;
        g.part_ld = M.nparts_cap;
        g.zt = M.zt;
        g.dbg = (s->debug_logits || s->top_p > 0.f) ? M.dbg : nullptr;
        f.nparts = thin_shape(g.W, g.epi, g.act, T).groups;
        if (f.nparts > M.nparts_cap) return BILD_ECAP;
        const int rc = run_thin(s, m, g);
        if (rc) return rc;
    } else if (const int groups = takes_sweep(m, lm_rows) && !parts ? head_groups(m->head, lm_rows, false) : 0; groups > 0) {
        HeadArgs h;
        std::memset((void*)&h, 0, sizeof(h));
        h.W = m->head;
        h.x = xfin + (size_t)(T - lm_rows) * d;
        h.ldx = d;
        h.T = lm_rows;
        h.gain = m->dec_final;
        h.eps = c.norm_eps;
        h.scale = c.logit_scale;
        h.vocab = c.vocab;
        h.y = s->y;
        h.ylen_ptr = &s->ctl->y_len;
        h.pos_ptr = len_ptr;
        h.pos_add = T - lm_rows;
        h.part = M.part;
        h.part_ld = M.nparts_cap;
        h.zt = M.zt;
        h.dbg = (s->debug_logits || s->top_p > 0.f) ? M.dbg : nullptr;  // the draw of the sampling variant reads the logits
        if (groups > M.nparts_cap) return BILD_ECAP;
        const int rc = launch_profiled(s, m, h.W, EPI_LMHEAD, [&] { return launch_head(h, s->stream); });
        if (rc) return rc;
        f.nparts = groups;
    } else if (lm_rows > 0) {
        GemmArgs g = gemm_base(m, m->head, xfin + (size_t)(T - lm_rows) * d, d, lm_rows, m->dec_final);
        if (parts) { g.px = M.px; g.px_stride = (int64_t)kMaxRows * d; g.pn = kPartSlices; g.x_out = xfin == M.x ? M.x2 : M.x; }
        g.epi = EPI_LMHEAD;
        g.scale = c.logit_scale;
        g.pos_ptr = len_ptr;
        g.pos_add = T - lm_rows;
        g.y = s->y;
        g.ylen_ptr = &s->ctl->y_len;
        g.part = M.part;
        g.part_ld = M.nparts_cap;
        g.zt = M.zt;
        g.dbg = (s->debug_logits || s->top_p > 0.f) ? M.dbg : nullptr;  // the draw of the sampling variant reads the logits
        g.row_off = 0;
        if (xb_parts > 0) {
            g.xb_hi = M.xb + (size_t)(T - lm_rows) * d;
            g.xb_lo = M.xb + (size_t)kMaxRows * d + (size_t)(T - lm_rows) * d;
            g.ssq_part = M.ssq + (T - lm_rows);
            g.ssq_parts = xb_parts;
        }
        gemm_pick_shape(g, dt);
        if ((int)gemm_num_blocks(g) > M.nparts_cap) return BILD_ECAP;
        {
            int rc = launch_gemm_profiled(s, m, g);
            if (rc) return rc;
        }
        f.nparts = (int)gemm_num_blocks(g);
    }
    if (lm_rows > 0) {
        f.part = M.part;
        f.part_ld = M.nparts_cap;
        f.zt = M.zt;
        f.T = lm_rows;
        f.mode = mode;
        if (s->top_p > 0.f) {
            f.top_p = s->top_p;
            f.logits = M.dbg;
            f.vocab = c.vocab;
            f.u = s->u_dev[w];
            if (s->accept_mode == 1) {
                f.accept_mode = 1;
                f.u_acc = s->u_acc;
                f.s_ring = s->s_ring;
                f.s_draw = s->s_draw;
            }
        }
    } else {
        f.mode = 3;
    }
    // sampling variant under the threshold rule: the draw runs spread over the chip (three launches instead of one)
    const bool spread = f.top_p > 0.f && f.mode <= 2 && f.accept_mode == 0 && s->draw_spread && s->draw_ws &&
                        c.vocab <= kDrawMaxVocab;
    s->stage_count += spread ? kFinishDrawStages : 1;
    if (spread) f.dws = s->draw_ws;
    if (!s->gemm_only) HIPC(spread ? launch_finish_draw(f, s->stream) : launch_finish(f, s->stream));
    return BILD_OK;
}

// Passes that produce a token, of shapes and row counts the pass kernel is made for (pass_groups); a caught-up row is rare and
// its passes follow each other without the host's look at their outcome.
//
// Source.  One workgroup per head has all its keys to itself: up to 512 arrive ahead of their use, each further one costs a layer
// 7 to 11 ns, where the separate kernels split them over more workgroups and stay as they are.  us per pass with its head, separate kernels / one
// kernel over the chip, 12 layers, at 512, 1024, 1408 tokens and (two rows and more) 1536: T5-large shape one row 348 / 184, 349 / 237, 369 / 279; two
// rows 406 / 212, 412 / 279, 432 / 326, 433 / 343; eight 510 / 240, 530 / 307, 551 / 353, 551 / 371; eleven 596 / 281, 619 / 349, 637 / 395, 642 / 412;
// mT5-large shape one row 365 / 185, 366 / 239, 390 / 281, two and eleven at 1536 471 / 350, 626 / 406; 768-wide one row 345 / 161, 349 / 209,
// 370 / 246, two and eleven at 1536 398 / 320, 560 / 371.
// On one die one row at 512, 1024, 1280 tokens costs 145 / 79, 146 / 101, 156 / 112 (T5-small shape; mT5-small 196 / 96, 197 / 125, 210 / 139; 256-wide,
// 6 layers 135 / 71, 136 / 92, 145 / 103).
// The lines come from passes that took 676 / 447 us at the T5-large shape (512 tokens, 24 layers) and met at 1580 (one row) to 1720
// tokens; by the costs of a token above they would meet past 2000 now, which has not been measured.
//
// fp32, 256 wide, 4 layers, at 32, 256, 512, 1024 tokens: one row 121 / 58, 127 / 67, 129 / 81, 130 / 109, four 146 / 72, 145 / 82, 147 / 96, 152 / 124, eleven
// 154 / 74, 158 / 84, 164 / 98, 167 / 126.
//
// Sequence.  Its keys past the first 256 are not asked for ahead.  At 256, 512, 1024 positions: T5-large shape, 12 layers, one row 348 / 185, 349 / 213,
// 351 / 267, two 405 / 208, 408 / 240, 416 / 302, eight 501 / 236, 512 / 267, 530 / 330, eleven 575 / 281, 597 / 311, 621 / 377; T5-small shape on one die
// 147 / 79, 147 / 91, 149 / 111: no shape and row count loses before the 1024 that were measured.
//
// Wide models (pass_wide.hip), rows 1, 2, 4, 8, separate kernels / one, 6 layers: 1280 wide at 40 positions 155, 182, 194, 209 / 98, 98, 111, 119,
// at 2200 204, 231, 243, 266 / 133, 134, 148, 159, at 8100 256, 263, 275, 300 / 222, 223, 232, 241; 2048 wide 221, 255, 270, 275 / 156, 158, 166, 180,
// at 2200 274, 314, 331, 327 / 200, 201, 213, 224, at 8100 330, 338, 355, 388 / 295, 297, 302, 312; 3072 wide 366, 384, 425, 374 / 284, 288, 316, 336
// and at 8100 530, 548, 590, 543 / 451, 456, 484, 507; 4096 wide 525, 567, 569, 572 / 455, 458, 465, 480 and 719, 759, 760, 766 / 648, 651,
// 660, 681: never slower up to the 8192 positions that were measured.  More rows: wide_rows, wide_keys.
static bool on_one_die(const bild_state* s, int w, int T) { return T <= s->ms[w].pass_die_rows; }
static bool takes_one_kernel(const bild_state* s, int w, int T, int lm_rows) {
    if (s->ms[w].pass_wide) {
        const bild_model_config& c = s->ms[w].m->cfg;
        const int keys = wide_keys(T, c.d_model, s->wide_most_rows > 0 ? INT_MAX : c.d_ff, s->ms[w].m->gated());  // (set for tests: as of the widest)
        return s->one_kernel && T <= s->ms[w].pass_wide_rows && lm_rows > 0 && !s->gemm_only && !s->prof_on && s->len[w] + T <= keys;
    }
    return s->one_kernel && s->ms[w].pass_groups > 0 && T <= kPassRows && lm_rows > 0 && !s->gemm_only && !s->prof_on &&
           s->n_src <= (s->ms[w].m->cfg.dtype == BILD_DT_F32 ? 1024 : on_one_die(s, w, T) ? 1280 : T == 1 ? 1408 : 1536) && s->len[w] + T <= 1024;
}

int key_bucket(int nkeys) {
    int b = 64;
    while (b < nkeys) b *= 2;
    return b;
}

// One pass, replayed from a captured graph when possible.  Launch parameters that depend on the
// lengths are chosen per power-of-two buckets of the key counts (the sequence's; the source's, which the separate kernels of
// the cross-attention split), so a graph stays valid while the sequence grows inside its bucket; everything else the kernels
// need they read from the control block.
int run_pass(bild_state* s, int w, int T, int lm_rows, int mode) {
    if (s->pair->trunk_layers > 0 && w == 1 && s->len[0] < s->len[1] + T) {
        // early-exit pair: the upper layers continue from what the trunk left for these rows
        const int rc = catch_up(s, 0, s->len[1] + T);
        if (rc) return rc;
    }
    const int bucket = key_bucket(s->len[w] + T);
    if (lm_rows > 0) s->ms[w].last_rows = lm_rows;
    bool one = takes_one_kernel(s, w, T, lm_rows) && alone(s);
    if (one && s->pass_pause > 0) {  // (see pass_gave_up)
        s->pass_pause -= 1;
        one = false;
    }
    s->last_one = one;
    if (lm_rows > 0 && !s->gemm_only) s->routes[!one ? ROUTE_KERNELS : on_one_die(s, w, T) ? ROUTE_DIE : ROUTE_CHIP] += 1;
    if (!s->use_graphs || s->prof_on || mode == 3) {
        const int rc = decoder_pass(s, w, T, lm_rows, mode, bucket, one);
        if (rc == BILD_OK && !s->gemm_only) s->seq_issued += 1;  // its policy kernel will count this pass
        return rc;
    }
    const int source = one || s->pair->decoder_only ? 0 : key_bucket(s->n_src);
    const std::array<int, 7> key = {w, T, lm_rows, mode, bucket, source, (s->debug_logits ? 1 : 0) | (s->gemm_only ? 2 : 0) | (s->top_p > 0.f ? 4 : 0) | (s->accept_mode ? 8 : 0) | (one ? 16 : 0) | (one && two_tiles(s, w, T) ? 32 : 0)};
    auto it = s->graphs.find(key);
    if (it == s->graphs.end()) {
        hipGraph_t g = nullptr;
        HIPC(hipStreamBeginCapture(s->stream, hipStreamCaptureModeThreadLocal));
        const int rc = decoder_pass(s, w, T, lm_rows, mode, bucket, one);
        const hipError_t e = hipStreamEndCapture(s->stream, &g);
        if (rc != BILD_OK || e != hipSuccess) {
            if (g) (void)hipGraphDestroy(g);
            return rc != BILD_OK ? rc : BILD_EHIP;
        }
        hipGraphExec_t ge = nullptr;
        const hipError_t e2 = hipGraphInstantiate(&ge, g, nullptr, nullptr, 0);
        (void)hipGraphDestroy(g);
        if (e2 != hipSuccess) return BILD_EHIP;
        it = s->graphs.emplace(key, bild_state::Captured{ge, s->stage_count}).first;
    }
    s->stage_count = it->second.stages;
    HIPC(hipGraphLaunch(it->second.exec, s->stream));
    if (!s->gemm_only) s->seq_issued += 1;
    return BILD_OK;
}

// After a pass of T rows that gave up.  What kept workgroups out may be gone by the next pass (work of another stream) or stay
// (another process' pass kernel), and each attempt takes 4 ms (a wait for another workgroup; the head's of pass_head.h is longer, and ends
// when one of the others has run out): the state's next 16 passes run as separate kernels, twice as many
// after each further attempt in vain, 65 536 at most (which is 40 s of passes for 4 ms).
int pass_gave_up(bild_state* s, int w, int T) {
    s->routes[ROUTE_GAVE_UP] += 1;
    s->pass_pause = 16 << s->pass_fails;
    s->pass_fails = std::min(s->pass_fails + 1, 12);
    // what it handed over is in no known state: nothing is there yet
    const ModelState& M = s->ms[w];
    HIPC(hipMemsetAsync(M.pass_turns[pass_room_index(T)], 0xFF, pass_turns_bytes(M, pass_room_index(T)), s->stream));
    HIPC(hipMemsetAsync(s->pass_sync, 0, sizeof(unsigned) * kPassSyncWords, s->stream));  // (workgroups may have started behind its end)
    if (T == 1) HIPC(hipMemsetAsync(pass_heads(s, w), 0, sizeof(unsigned) * kPassHeadWords, s->stream));  // (both counts again with one turn, as the memory filled above)
    return BILD_OK;
}

// Brings model w's cache up to `target` consumed rows with LM-head-less passes.
int catch_up(bild_state* s, int w, int target) {
    while (s->len[w] < target) {
        const int T = std::min(s->ms[w].rows_cap, target - s->len[w]);
        int rc = run_pass(s, w, T, 0, 3);
        if (rc) return rc;
        s->len[w] += T;  // the device advances the same amount
    }
    return BILD_OK;
}

}  // namespace bild

namespace {

// One pass and its result.  A pass kernel whose workgroups did not all get to run has changed nothing that counts: the pass runs
// again as separate kernels.
int finish_pass(bild_state* s, int w, int T, int lm_rows, int mode) {
    int rc = run_pass(s, w, T, lm_rows, mode);
    if (rc == BILD_OK) rc = pull_ctl(s);
    if (rc == BILD_OK && s->last_one) s->pass_fails = 0;
    if (rc == kPassFailed) {
        rc = pass_gave_up(s, w, T);
        if (rc == BILD_OK) rc = run_pass(s, w, T, lm_rows, mode);
        if (rc == BILD_OK) rc = pull_ctl(s);
    }
    return rc;
}

// Cross K/V of every decoder layer of each model that uses the output of model w's encoder: K = norm_final(enc_x) Wk,
// V = norm_final(enc_x) Wv.  bf16 models: one launch for all layers, from the planes of `p` (of a bf16 encoder) or from planes
// made here (a bf16 model that borrows an fp32 encoder).
int cross_kv(bild_state* s, int w, const TilePass& p) {
    ModelState& M = s->ms[w];
    const bild_model* m = M.m;
    const int S = s->n_src;
    for (int u = 0; u < 2; ++u) {
        const bool uses = (u == w) || (u == 0 && w == 1 && s->pair->small_borrows_encoder);
        if (!uses || (u == 0 && s->pair->trunk_layers > 0)) continue;  // (a view shares the large model's cross K/V)
        ModelState& U = s->ms[u];
        const bild_model* mu = U.m;
        const int Iu = mu->inner();
        const size_t layer = (size_t)s->cap_src * Iu;
        if (mu->cfg.dtype == BILD_DT_BF16) {
            TilePass q = p;
            if (!q.xt) {
                q.xt = U.xt;
                q.ssq = U.ssq_t;
                q.parts = 1;
                RowCopyArgs r;
                std::memset((void*)&r, 0, sizeof(r));
                r.src = r.dst = M.enc_x;
                r.d = m->cfg.d_model;
                r.T = S;
                HIPC(launch_row_tiles(r, m->enc_final, q.xt, q.ssq, s->stream));
            }
            TileGemmArgs g = tile_base(q, mu->cwkv_all, q.xt);
            g.epi = EPI_QKV;
            g.i_dim = Iu;
            g.layer_n = 2 * Iu;
            g.kv_layer = layer;
            g.k_cache = U.ck;
            g.v_cache = U.cv;
            g.vcap = s->cap_src;
            int rc = run_tile(q, g);
            if (rc) return rc;
            continue;
        }
        for (int l = 0; l < mu->cfg.n_dec_layers; ++l) {
            GemmArgs g = gemm_base(mu, mu->dec[l].cwkv, M.enc_x, m->cfg.d_model, S, m->enc_final);
            g.eps = m->cfg.norm_eps;
            g.epi = EPI_QKV;
            g.q_dim = 0;
            g.i_dim = Iu;
            g.k_cache = U.ck + l * layer * mu->esz();
            g.v_cache = U.cv + l * layer * mu->esz();
            g.vcap = s->cap_src;
            int rc = run_gemm(s, mu, g);
            if (rc) return rc;
        }
    }
    return BILD_OK;
}

// bf16: the same on the tile kernels.
int run_encoder_tiles(bild_state* s, int w) {
    ModelState& M = s->ms[w];
    const bild_model* m = M.m;
    const bild_model_config& c = m->cfg;
    const int S = s->n_src;
    TilePass p = {s, m, S, M.enc_x, M.enc_q, M.xt, (char*)M.enc_a, (char*)M.enc_h, M.ssq_t, 0, M.rope};
    int rc = tile_embed(p, s->src, nullptr, M.pe, m->enc[0].ln1);
    if (rc) return rc;
    for (int l = 0; l < c.n_enc_layers; ++l) {
        const LayerW& L = m->enc[l];
        rc = tile_qkv(p, L.wqkv, M.enc_k, M.enc_v, s->cap_src, nullptr);
        if (rc) return rc;
        AttnArgs a;
        std::memset((void*)&a, 0, sizeof(a));
        a.q = M.enc_q; a.k = M.enc_k; a.v = M.enc_v; a.ob_t = p.at;
        a.T = S; a.heads = c.n_heads; a.d_head = c.d_head; a.i_dim = m->inner();
        a.nkeys_fixed = S;
        a.rel_bias = m->enc_rel;
        a.rel_d = c.rel_max_dist;
        a.len_ptr = &s->ctl->n_src;  // not used with a fixed count, but the kernel reads it
        a.vcap = s->cap_src;
        a.scale = 1.f / std::sqrt((float)c.d_head);
        HIPC(launch_attention_tile(a, s->stream));
        rc = tile_resid(p, L.wo, p.at, L.ln2);
        if (rc) return rc;
        rc = tile_ffn(p, L, l + 1 < c.n_enc_layers ? m->enc[l + 1].ln1 : m->enc_final);
        if (rc) return rc;
    }
    return cross_kv(s, w, p);
}

// Encoder of model w over the source in s->src, then the cross K/V of every decoder
// layer of each model that uses this encoder's output.
int run_encoder(bild_state* s, int w) {
    if (s->ms[w].m->cfg.dtype == BILD_DT_BF16) return run_encoder_tiles(s, w);
    ModelState& M = s->ms[w];
    const bild_model* m = M.m;
    const bild_model_config& c = m->cfg;
    const int d = c.d_model, I = m->inner(), F = c.d_ff, dt = c.dtype, S = s->n_src;
    const float att_scale = 1.f / std::sqrt((float)c.d_head);
    // every launch covers all S source rows (row blocks of kMaxRows inside the kernels)
    {
        EmbedArgs e;
        std::memset((void*)&e, 0, sizeof(e));
        e.E = m->emb; e.tokens = s->src; e.T = S; e.d = d; e.vocab = c.vocab;
        e.tie_shift = c.tie_shift; e.sinusoidal = c.pos == BILD_POS_SINUSOIDAL; e.embed_scale = c.embed_scale;
        e.x = M.enc_x;
        HIPC(launch_embed(e, dt, s->stream));
    }
    for (int l = 0; l < c.n_enc_layers; ++l) {
        const LayerW& L = m->enc[l];
        {
            GemmArgs g = gemm_base(m, L.wqkv, M.enc_x, d, S, L.ln1);
            g.epi = EPI_QKV;
            g.q_dim = I;
            g.q_out = M.enc_q;
            g.k_cache = M.enc_k;
            g.v_cache = M.enc_v;
            g.vcap = s->cap_src;
            g.rope = M.rope;
            int rc = run_gemm(s, m, g);
            if (rc) return rc;
        }
        {
            AttnArgs a;
            std::memset((void*)&a, 0, sizeof(a));
            a.q = M.enc_q; a.k = M.enc_k; a.v = M.enc_v; a.out = M.enc_a;
            a.T = S; a.heads = c.n_heads; a.d_head = c.d_head; a.i_dim = I;
            a.causal = 0;
            a.nkeys_fixed = S;
            a.rel_bias = m->enc_rel;
            a.rel_d = c.rel_max_dist;
            a.len_ptr = &s->ctl->n_src;  // not used with a fixed count, but the kernel reads it
            a.vcap = s->cap_src;
            a.splits = 1;
            a.nw = pick_attn_waves(dt, c.d_head, std::min(S, kMaxRows), S, 1);
            a.scale = att_scale;
            HIPC(launch_attention(a, dt, s->stream));
        }
        {
            GemmArgs g = gemm_base(m, L.wo, M.enc_a, I, S, nullptr);
            g.epi = EPI_RESID;
            g.out = M.enc_x;
            g.ldo = d;
            int rc = run_gemm(s, m, g);
            if (rc) return rc;
        }
        {
            GemmArgs g = gemm_base(m, L.win, M.enc_x, d, S, L.ln2);
            g.epi = EPI_ACT;
            g.out = M.enc_h;
            g.ldo = F;
            int rc = run_gemm(s, m, g);
            if (rc) return rc;
        }
        {
            GemmArgs g = gemm_base(m, L.wout, M.enc_h, F, S, nullptr);
            g.epi = EPI_RESID;
            g.out = M.enc_x;
            g.ldo = d;
            int rc = run_gemm(s, m, g);
            if (rc) return rc;
        }
    }
    const TilePass none = {s, m, S, M.enc_x, nullptr, nullptr, nullptr, nullptr, nullptr, 0, nullptr};
    return cross_kv(s, w, none);
}

// Both encoders; the small model's beside the large one's on the pair's spare stream: neither fills the chip over a few hundred
// rows.  One after the other / beside: T5 shapes, 77, 512, 1531 tokens 1.22 / 1.06, 2.13 / 1.94, 4.69 / 4.41 ms; mT5 shapes, 64 and 512
// tokens 1.24 / 1.04, 2.30 / 2.01 ms (nothing gained where the two streams share a hardware queue).
int run_encoders(bild_state* s) {
    auto large = [&] { return run_encoder(s, 1); };
    if (s->pair->small_borrows_encoder) return large();
    auto small = [&] { return run_encoder(s, 0); };
    int rc = BILD_OK;
    if (s->pair->spare.beside(s->device, s->stream, large, small, &rc)) return rc;
    rc = large();
    return rc ? rc : small();
}

}  // namespace

// ======================================================================= request API
extern "C" int bild_encode(bild_state* s, const int32_t* src, int n_src) {
    if (!s || !src) return BILD_EINVAL;
    const Call call(s);
    if (n_src < 1) return BILD_EINVAL;
    if (n_src > s->max_src) return BILD_ECAP;
    const int V = s->pair->m[1]->cfg.vocab;
    for (int i = 0; i < n_src; ++i)
        if (src[i] < 0 || src[i] >= V) return BILD_EINVAL;
    const bool dec_only = s->pair->decoder_only;
    if (dec_only && n_src + 1 > s->max_len) return BILD_ECAP;
    s->encoded = false;
    s->n_src = n_src;
    s->len[0] = s->len[1] = 0;
    if (dec_only) {
        std::memcpy(s->hy, src, sizeof(int) * (size_t)n_src);
        s->y_len = n_src;
    } else {
        std::memcpy(s->hsrc, src, sizeof(int) * (size_t)n_src);
        s->hy[0] = s->pair->m[1]->cfg.bos;
        s->y_len = 1;
    }
    s->n0 = s->y_len;
    s->draft_start = s->y_len;
    int rc = push_ctl(s, 0, s->y_len, !dec_only);
    if (rc) return rc;
    if (dec_only) {
        for (int w = 0; w < 2; ++w) {
            rc = catch_up(s, w, n_src - 1);
            if (rc) return rc;
        }
    } else {
        rc = run_encoders(s);
        if (rc) return rc;
        FinishArgs f;  // the encoder's end is counted like a pass (of no rows), so that it is waited for like one
        std::memset((void*)&f, 0, sizeof(f));
        f.ctl = s->ctl;
        f.mode = 3;
        f.host_mirror = s->hctl_dev;
        HIPC(launch_finish(f, s->stream));
        s->seq_issued += 1;
    }
    rc = pull_ctl(s);
    if (rc) return rc;
    s->encoded = true;
    return BILD_OK;
}

extern "C" int bild_small_step(bild_state* s, float alpha_fb, int32_t* token, int32_t* fallback_flag,
                               float* max_prob) {
    if (!s || !token || !fallback_flag) return BILD_EINVAL;
    const Call call(s);
    if (!s->encoded) return BILD_ESTATE;
    if (s->len[0] >= s->y_len) return BILD_ESTATE;  // nothing unconsumed
    if (s->y_len >= s->max_len) return BILD_ECAP;
    int rc = set_alpha(s, alpha_fb, s->alpha_rb);
    if (rc) return rc;
    rc = catch_up(s, 0, s->y_len - 1);
    if (rc) return rc;
    rc = finish_pass(s, 0, 1, 1, 0);
    if (rc) return rc;
    *token = s->hctl->res_tok;
    *fallback_flag = s->hctl->res_flag & 1;
    if (!*fallback_flag) s->hy[s->y_len - 1] = *token;
    if (max_prob) *max_prob = s->hctl->res_pmax;
    return BILD_OK;
}

extern "C" int bild_large_verify(bild_state* s, const int32_t* draft, int n, float alpha_rb, int32_t* out_tokens,
                                 int32_t* n_out, int32_t* rollback_pos, float* nll) {
    if (!s || !out_tokens || !n_out || !rollback_pos) return BILD_EINVAL;
    const Call call(s);
    if (!s->encoded) return BILD_ESTATE;
    if (draft) {
        if (n < 0) return BILD_EINVAL;
        if (n + 1 > kMaxRows) return BILD_ECAP;
        if (s->draft_start + n + 1 > s->max_len) return BILD_ECAP;
        const int V = s->pair->m[1]->cfg.vocab;
        for (int i = 0; i < n; ++i)
            if (draft[i] < 0 || draft[i] >= V) return BILD_EINVAL;
        if (n > 0) std::memcpy(s->hy + s->draft_start, draft, sizeof(int) * (size_t)n);
        s->y_len = s->draft_start + n;
        s->len[0] = std::min(s->len[0], s->draft_start);
        s->len[1] = std::min(s->len[1], s->draft_start - 1);
        int rc = push_ctl(s, s->draft_start, n);
        if (rc) return rc;
    } else {
        n = s->y_len - s->draft_start;
        if (n + 1 > kMaxRows) return BILD_ECAP;
        if (s->y_len + 1 > s->max_len) return BILD_ECAP;
    }
    if (s->len[1] > s->draft_start - 1) return BILD_ESTATE;
    int rc = set_alpha(s, s->alpha_fb, alpha_rb);
    if (rc) return rc;
    rc = catch_up(s, 1, s->draft_start - 1);
    if (rc) return rc;
    const int ds = s->draft_start;
    rc = finish_pass(s, 1, n + 1, n + 1, 1);
    if (rc) return rc;
    const int r = s->hctl->res_r;
    *rollback_pos = r;
    *n_out = r + 1;
    s->hy[ds + r] = s->hctl->res_tok;  // behind the drafts that stand
    std::memcpy(out_tokens, s->hy + ds, sizeof(int) * (size_t)(r + 1));
    if (nll)
        for (int i = 0; i < n; ++i) nll[i] = (i <= r) ? s->hctl->res_nll[i] : NAN;
    return BILD_OK;
}

extern "C" int bild_kv_truncate(bild_state* s, int which, int pos) {
    if (!s || which < 1 || which > 3 || pos < 0) return BILD_EINVAL;
    if (!s->encoded) return BILD_ESTATE;
    if ((which & 1) && pos > s->len[0]) return BILD_EINVAL;
    if ((which & 2) && pos > s->len[1]) return BILD_EINVAL;
    // the large model must never be ahead of draft_start - 1; cutting only lowers lengths
    if (which & 1) s->len[0] = pos;
    if (which & 2) s->len[1] = pos;
    return push_ctl(s);
}

extern "C" int bild_seq_truncate(bild_state* s, int n_keep) {
    if (!s) return BILD_EINVAL;
    if (!s->encoded) return BILD_ESTATE;
    if (n_keep < s->n0 || n_keep > s->y_len) return BILD_EINVAL;
    s->y_len = n_keep;
    s->draft_start = std::min(s->draft_start, n_keep);
    s->len[0] = std::min(s->len[0], n_keep - 1);
    s->len[1] = std::min(s->len[1], s->draft_start - 1);
    return push_ctl(s);
}

extern "C" int bild_force_tokens(bild_state* s, int first, const int32_t* tokens, int n, int draft_start) {
    if (!s || n < 0 || (n > 0 && !tokens)) return BILD_EINVAL;
    if (!s->encoded) return BILD_ESTATE;
    if (first < s->n0 || first > s->y_len) return BILD_EINVAL;
    if (first + n >= s->max_len) return BILD_ECAP;
    if (draft_start < s->n0 || draft_start > first + n) return BILD_EINVAL;
    const int V = s->pair->m[1]->cfg.vocab;
    for (int i = 0; i < n; ++i)
        if (tokens[i] < 0 || tokens[i] >= V) return BILD_EINVAL;
    if (n > 0) std::memcpy(s->hy + first, tokens, sizeof(int) * (size_t)n);
    s->y_len = first + n;
    s->draft_start = draft_start;
    s->len[0] = std::min(s->len[0], first);
    s->len[1] = std::min(s->len[1], std::min(first, draft_start - 1));
    return push_ctl(s, first, n);
}

extern "C" int bild_get_lengths(bild_state* s, int32_t* y_len, int32_t* draft_start, int32_t* len_small,
                                int32_t* len_large) {
    if (!s) return BILD_EINVAL;
    if (y_len) *y_len = s->y_len;
    if (draft_start) *draft_start = s->draft_start;
    if (len_small) *len_small = s->len[0];
    if (len_large) *len_large = s->len[1];
    return BILD_OK;
}

extern "C" int bild_get_sequence(bild_state* s, int32_t* out, int cap, int32_t* n) {
    if (!s || !out || !n) return BILD_EINVAL;
    if (cap < s->y_len) return BILD_ECAP;
    if (s->y_len > 0) std::memcpy(out, s->hy, sizeof(int) * (size_t)s->y_len);
    *n = s->y_len;
    return BILD_OK;
}

extern "C" int bild_generate(bild_state* s, const int32_t* src, int n_src, float alpha_fb, float alpha_rb,
                             int max_new, int32_t eos, int32_t* out, int32_t* n_out, bild_stats* stats) {
    if (!s || !out || !n_out || max_new < 0) return BILD_EINVAL;
    const Call call(s);
    int rc = BILD_OK;
    if (src) {
        rc = bild_encode(s, src, n_src);
        if (rc) return rc;
    } else if (!s->encoded) {
        return BILD_ESTATE;
    }
    if (s->n0 + max_new > s->max_len) return BILD_ECAP;
    bild_stats st;
    std::memset(&st, 0, sizeof(st));
    int last = -1;
    while (s->y_len - s->n0 < max_new && !(s->y_len > s->n0 && last == eos && eos >= 0)) {
        int32_t tok, flag;
        rc = bild_small_step(s, alpha_fb, &tok, &flag, nullptr);
        if (rc) return rc;
        st.small_steps++;
        if (!flag) {
            last = tok;
            continue;
        }
        if (s->hctl->res_flag & 2)
            st.fallbacks_forced++;
        else
            st.fallbacks_conf++;
        int32_t toks[kMaxRows], cnt, r;
        const int n = s->y_len - s->draft_start;
        rc = bild_large_verify(s, nullptr, 0, alpha_rb, toks, &cnt, &r, nullptr);
        if (rc) return rc;
        st.large_calls++;
        st.rows_verified += n + 1;
        if (r < n) {
            st.rollbacks++;
            st.tokens_discarded += n - r;
        }
        last = toks[r];
    }
    st.n_generated = s->y_len - s->n0;
    *n_out = st.n_generated;
    if (st.n_generated > 0) std::memcpy(out, s->hy + s->n0, sizeof(int) * (size_t)st.n_generated);
    if (stats) *stats = st;
    return BILD_OK;
}

extern "C" int bild_greedy(bild_state* s, int which, const int32_t* src, int n_src, int max_new, int32_t eos,
                           int32_t* out, int32_t* n_out) {
    if (!s || !out || !n_out || max_new < 0 || which < 1 || which > 2) return BILD_EINVAL;
    const Call call(s);
    int rc = BILD_OK;
    if (src) {
        rc = bild_encode(s, src, n_src);
        if (rc) return rc;
    } else if (!s->encoded) {
        return BILD_ESTATE;
    }
    if (s->n0 + max_new > s->max_len) return BILD_ECAP;
    const int w = which - 1;
    int last = -1;
    while (s->y_len - s->n0 < max_new && !(s->y_len > s->n0 && last == eos && eos >= 0)) {
        rc = catch_up(s, w, s->y_len - 1);
        if (rc) return rc;
        rc = finish_pass(s, w, 1, 1, 2);
        if (rc) return rc;
        last = s->hctl->res_tok;
        s->hy[s->y_len - 1] = last;
    }
    // leave the state consistent for a following BiLD call: the other model lags, which is allowed
    *n_out = s->y_len - s->n0;
    if (*n_out > 0) std::memcpy(out, s->hy + s->n0, sizeof(int) * (size_t)*n_out);
    return BILD_OK;
}

namespace {
int alloc_logit_buffers(bild_state* s) {
    for (int w = 0; w < 2; ++w) {
        if (s->ms[w].dbg) continue;
        int rc = dev_alloc(s->allocs, (void**)&s->ms[w].dbg, sizeof(float) * kMaxRows * (size_t)s->ms[w].m->cfg.vocab);
        if (rc) return rc;
    }
    return BILD_OK;
}
}  // namespace

extern "C" int bild_debug_enable_logits(bild_state* s, int enable) {
    if (!s) return BILD_EINVAL;
    if (enable) {
        int rc = alloc_logit_buffers(s);
        if (rc) return rc;
    }
    s->debug_logits = enable != 0;
    return BILD_OK;
}

extern "C" int bild_set_sampling(bild_state* s, float top_p, const float* u_small, const float* u_large, int n) {
    if (!s) return BILD_EINVAL;
    if (!(top_p > 0.f)) {  // back to argmax (and to the threshold rule of the review, which is all argmax decoding has)
        if (s->top_p > 0.f) drop_graphs(s);
        s->top_p = 0.f;
        s->accept_mode = 0;
        return BILD_OK;
    }
    if (top_p > 1.f || !u_small || !u_large || n < s->max_len) return BILD_EINVAL;
    const float* us[2] = {u_small, u_large};
    for (int w = 0; w < 2; ++w)
        for (int i = 0; i < s->max_len; ++i)
            if (!(us[w][i] >= 0.f && us[w][i] < 1.f)) return BILD_EINVAL;
    int rc = alloc_logit_buffers(s);
    if (rc) return rc;
    HIPC(hipStreamSynchronize(s->stream));
    for (int w = 0; w < 2; ++w) {
        if (!s->u_dev[w]) {
            rc = dev_alloc(s->allocs, (void**)&s->u_dev[w], sizeof(float) * (size_t)(s->max_len + 1));
            if (rc) return rc;
        }
        HIPC(hipMemcpy(s->u_dev[w], us[w], sizeof(float) * (size_t)s->max_len, hipMemcpyHostToDevice));
    }
    if (!s->draw_ws) {
        rc = dev_alloc(s->allocs, (void**)&s->draw_ws, std::max(draw_ws_bytes(s->ms[0].m->cfg.vocab), draw_ws_bytes(s->ms[1].m->cfg.vocab)));
        if (rc) return rc;
        drop_graphs(s);  // (none can have been captured with a draw yet; kept for safety)
    }
    if (s->top_p != top_p) drop_graphs(s);
    s->top_p = top_p;
    return BILD_OK;
}

extern "C" int bild_set_acceptance(bild_state* s, int rule, const float* u_accept, int n) {
    if (!s || (rule != BILD_ACCEPT_THRESHOLD && rule != BILD_ACCEPT_REJECTION)) return BILD_EINVAL;
    if (rule == BILD_ACCEPT_THRESHOLD) {
        if (s->accept_mode != 0) drop_graphs(s);
        s->accept_mode = 0;
        return BILD_OK;
    }
    if (!(s->top_p > 0.f)) return BILD_ESTATE;
    if (!u_accept || n < s->max_len) return BILD_EINVAL;
    for (int i = 0; i < s->max_len; ++i)
        if (!(u_accept[i] >= 0.f && u_accept[i] < 1.f)) return BILD_EINVAL;
    HIPC(hipStreamSynchronize(s->stream));
    if (!s->u_acc) {
        const size_t V = (size_t)s->pair->m[0]->cfg.vocab;
        int rc = dev_alloc(s->allocs, (void**)&s->u_acc, sizeof(float) * (size_t)(s->max_len + 1));
        if (rc) return rc;
        rc = dev_alloc(s->allocs, (void**)&s->s_ring, sizeof(float) * (size_t)kMaxRows * V);
        if (rc) return rc;
        rc = dev_alloc(s->allocs, (void**)&s->s_draw, sizeof(float4) * (size_t)(s->max_len + 1));
        if (rc) return rc;
        HIPC(hipMemset(s->s_ring, 0, sizeof(float) * (size_t)kMaxRows * V));
        HIPC(hipMemset(s->s_draw, 0, sizeof(float4) * (size_t)(s->max_len + 1)));
    }
    HIPC(hipMemcpy(s->u_acc, u_accept, sizeof(float) * (size_t)s->max_len, hipMemcpyHostToDevice));
    if (s->accept_mode != 1) drop_graphs(s);
    s->accept_mode = 1;
    return BILD_OK;
}

extern "C" int bild_debug_pass_spins(bild_state* s, int spins) {
    if (!s || spins < 1) return BILD_EINVAL;
    drop_graphs(s);
    s->pass_spins = spins;
    return BILD_OK;
}

extern "C" int bild_debug_logits(bild_state* s, int which, int row, float* out) {
    if (!s || !out || which < 1 || which > 2) return BILD_EINVAL;
    ModelState& M = s->ms[which - 1];
    if (!s->debug_logits || !M.dbg) return BILD_ESTATE;
    if (row < 0 || row >= M.last_rows) return BILD_EINVAL;
    const size_t V = M.m->cfg.vocab;
    HIPC(hipMemcpyAsync(out, M.dbg + (size_t)row * V, sizeof(float) * V, hipMemcpyDeviceToHost, s->stream));
    HIPC(hipStreamSynchronize(s->stream));
    return BILD_OK;
}

extern "C" int bild_debug_kv(bild_state* s, int which, int layer, int is_v, int pos0, int n, float* out) {
    if (!s || !out || which < 1 || which > 2 || n < 1 || pos0 < 0) return BILD_EINVAL;
    if (!s->encoded) return BILD_ESTATE;
    const ModelState& M = s->ms[which - 1];
    const bild_model* m = M.m;
    // an early-exit pair keeps the trunk's rows in the large model's buffers: the view has its own layer count
    if (layer < 0 || layer >= m->cfg.n_dec_layers || pos0 + n > s->len[which - 1]) return BILD_EINVAL;
    const size_t I = m->inner(), esz = m->esz(), cap = s->cap_len;
    std::vector<char> raw((size_t)(is_v ? I * cap : (size_t)n * I) * esz);
    const char* base = (is_v ? M.vcache : M.kcache) + (size_t)layer * cap * I * esz;
    HIPC(hipStreamSynchronize(s->stream));
    // K is [position][I]; V is stored transposed, [I][capacity]
    HIPC(hipMemcpy(raw.data(), is_v ? base : base + (size_t)pos0 * I * esz, raw.size(), hipMemcpyDeviceToHost));
    auto widen = [&](size_t idx) -> float {
        if (esz == 4) return ((const float*)raw.data())[idx];
        const uint32_t u = (uint32_t)((const uint16_t*)raw.data())[idx] << 16;
        float f;
        std::memcpy(&f, &u, 4);
        return f;
    };
    for (int t = 0; t < n; ++t)
        for (size_t i = 0; i < I; ++i) out[(size_t)t * I + i] = is_v ? widen(i * cap + pos0 + t) : widen((size_t)t * I + i);
    return BILD_OK;
}

extern "C" const char* bild_strerror(int code) {
    switch (code) {
        case BILD_OK: return "ok";
        case BILD_EINVAL: return "invalid argument";
        case BILD_ESTATE: return "call not valid in the current state";
        case BILD_ECAP: return "capacity exceeded";
        case BILD_EHIP: return "HIP runtime error";
        case BILD_ENOMEM: return "out of memory";
        default: return "unknown error";
    }
}
