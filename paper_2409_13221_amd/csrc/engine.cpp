// Host side of the fused generation + inference stage: the C ABI of include/rlhf.h, the
// continuous-batching bookkeeping (admission against the KV budget, page tables, retirement,
// scoring-batch formation) and the launch sequences of the decode step and of the prefill /
// scoring forward.  All arithmetic of the method runs in the HIP kernels declared in
// kernels.h; this file only decides what to launch, on which stream, over which rows.
#include "../../include/rlhf.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <deque>
#include <string>
#include <utility>
#include <vector>

#include "kernels.h"

using namespace rlhf;

namespace {

thread_local char g_create_error[512] = "";

struct RoleWeights {
    bool bound = false;
    rlhf_weights w{};
    // IEEE-half copies of the bf16 matrices for the tall (prefill / scoring) passes, owned by the
    // library (engine option half_weight_copies); NULL members: no copy, the bf16 tensor is used
    rlhf_weights h16{};
    std::vector<void*> owned;
};

// Pinned host staging + one device arena for small per-pass integer metadata.  The host runs
// ahead of the device, so host slots form a ring guarded by events; the device arena is
// rewritten by a stream-ordered copy, after the kernels of the previous pass on that stream.
struct MetaRing {
    static constexpr int kSlots = 8;
    int* host[kSlots] = {};
    hipEvent_t ev[kSlots] = {};
    bool used[kSlots] = {};
    int* dev = nullptr;
    size_t cap = 0;
    int next = 0;

    hipError_t init(size_t cap_ints) {
        cap = cap_ints;
        hipError_t e = hipMalloc((void**)&dev, cap * sizeof(int));
        if (e != hipSuccess) return e;
        for (int i = 0; i < kSlots; ++i) {
            e = hipHostMalloc((void**)&host[i], cap * sizeof(int), hipHostMallocDefault);
            if (e != hipSuccess) return e;
            e = hipEventCreateWithFlags(&ev[i], hipEventDisableTiming);
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    void destroy() {
        for (int i = 0; i < kSlots; ++i) {
            if (host[i]) (void)hipHostFree(host[i]);
            if (ev[i]) (void)hipEventDestroy(ev[i]);
        }
        if (dev) (void)hipFree(dev);
    }
    hipError_t begin(int** out) {
        if (used[next]) {
            hipError_t e = hipEventSynchronize(ev[next]);
            if (e != hipSuccess) return e;
        }
        *out = host[next];
        return hipSuccess;
    }
    hipError_t commit(hipStream_t st, size_t n_ints) {
        hipError_t e = hipMemcpyAsync(dev, host[next], n_ints * sizeof(int), hipMemcpyHostToDevice, st);
        if (e != hipSuccess) return e;
        e = hipEventRecord(ev[next], st);
        used[next] = true;
        next = (next + 1) % kSlots;
        return e;
    }
};

struct Workspace {
    int rows_cap = 0;
    float* h = nullptr;       // [rows, d] residual stream (float)
    void* xn = nullptr;       // [rows, d] normed activations (storage type)
    float* part = nullptr;    // split-K partial outputs of the GEMM in flight
    size_t part_cap = 0;      // floats
    void* q = nullptr;        // [rows, Hq*hd]
    void* k = nullptr;        // [rows, Hkv*hd] (batch passes)
    void* v = nullptr;
    void* attn = nullptr;     // [rows, Hq*hd]
    void* act = nullptr;      // [rows, ffn]
    void* xsel = nullptr;     // [rows, d] final-norm rows selected for the head (storage type; float for d -> 1 heads)
    float* logits = nullptr;  // [logit_rows, vocab] (batch passes; decode uses `part`)
    int logit_rows = 0;
    float* pick_scratch = nullptr;  // per-chunk partial results of the greedy pick
    float* ssq = nullptr;       // few-row passes: partial sums of h^2 of the rows in flight
    float* scale = nullptr;     // [2][few]: scales of the normed rows, ping and pong
    int few = 0;                // rows these two have room for
    float* attn_acc = nullptr;  // decode split-KV partials
    float* attn_ml = nullptr;
    size_t attn_slots = 0;
    std::vector<void*> owned;
};

// Rows from which a batch pass without half copies of the weights converts each matrix before its projection, into the part
// of the workspace that is there for planes and that this projection leaves free (gate||up of d_model beyond 6144 fits
// where a pass may have d_model / 2 rows): the tall kernel runs at 1.4 PFLOP/s on half weights, at 1.15 where it converts
// them itself, once per tile; a conversion reads and writes the matrix once (7B gate||up 73 us beside 1250).  Prefill of
// 1100, 2048, 3072, 4096, 6144, 8192 rows, converting in the kernel / before it: 7B widths, 4 layers, ms, 2.45 3.99 5.60
// 6.54 10.3 12.5 / 2.70 3.94 5.37 6.22 9.4 11.3; 70B widths, 1 layer 2.40 3.43 4.96 6.37 9.4 12.4 / 2.70 3.54 4.89 6.10 8.6
// 11.1.  Narrow layers gain less and lose nothing: 3072 and 8192 rows, d = 512, 8 layers 1.00 1.55 / 1.00 1.51, d = 768, 12 layers
// 1.85 3.38 / 1.83 3.30, d = 1536, 6 layers 2.12 3.96 / 2.03 3.70.
constexpr int kConvertRows = 3072;

// Optional per-kernel-class timing: every `every`-th launch of a class is bracketed by two
// events on its stream; algorithmic bytes / flops of the sampled launches are summed beside.
enum KClass { kGemmDecode = 0, kGemmBatch = 1, kAttnDecode = 2, kAttnBatch = 3, kClassCount = 4 };

struct Profiler {
    bool on = false;
    int every = 1;
    // Event pairs in flight.  rlhf_run_stage folds them into the sums below once the stage has
    // drained, so the cap bounds the samples of ONE stage; launches beyond it go untimed and are
    // counted in `dropped` (a caller who sees dropped > 0 should raise sample_every).
    static constexpr size_t kMaxSamples = 1 << 16;
    struct Rec { hipEvent_t a, b; int cls; double bytes, flops; };
    std::vector<Rec> recs;                 // recs[0..n_used) are live; events are reused across runs
    size_t n_used = 0;
    int64_t launches[kClassCount] = {};
    double tot_bytes[kClassCount] = {}, tot_flops[kClassCount] = {};
    int64_t sampled[kClassCount] = {}, dropped[kClassCount] = {};
    double bracket_overhead_ms = 0;        // cost of an event bracket beyond its kernels, measured at begin
    double s_ms[kClassCount] = {}, s_bytes[kClassCount] = {}, s_flops[kClassCount] = {};
};

struct Sample {
    int P = 0, max_new = 0, target = 0, reserve = 0;
    int ctx = 0, gen_len = 0, admit_step = -1;
    bool has_forced_len = false, finished = false, retired = false;
    std::vector<int> pages;
};

}  // namespace

struct rlhf_ctx {
    rlhf_model_cfg mc{};
    rlhf_engine_cfg ec{};
    Dims dm{};
    int dtype = 0, esz = 2;
    int max_pages = 0, pool_pages = 0;
    char err[512] = "";

    hipStream_t sd = nullptr, ss = nullptr;            // the streams decode / scoring work goes to NOW
    hipStream_t sd_full = nullptr, ss_full = nullptr;  // whole chip
    hipStream_t sd_part = nullptr, ss_part = nullptr;  // disjoint CU masks for co-running (optional)
    bool own_sd = false, own_ss = false;
    hipEvent_t ev_sw_d = nullptr, ev_sw_s = nullptr, ev_score_last = nullptr;
    hipEvent_t ev_dep = nullptr;                       // decode -> score dependency
    hipEvent_t ev_d0 = nullptr, ev_d1 = nullptr, ev_s0 = nullptr, ev_s1 = nullptr;
    std::vector<hipEvent_t> step_events;

    RoleWeights roles[4];

    void* pool = nullptr;
    int* d_page_table = nullptr;   // [max_samples, max_pages]
    int* d_tokens = nullptr;       // [max_samples, max_ctx]   prompt + response
    float* d_lp_actor = nullptr;   // [max_samples, max_ctx]   indexed by output index j-1
    float* d_lp_rescored = nullptr;
    float* d_lp_ref = nullptr;
    float* d_values = nullptr;
    float* d_reward = nullptr;     // [max_samples]
    float* d_rope = nullptr;       // [max_ctx, hd/2, 2]
    int* d_nonfinite = nullptr;    // set by the kernels that write results when one is not finite
    int* d_picked = nullptr;       // [max_active] tokens of the last pick (stop_on_eos)
    int* h_picked = nullptr;       // pinned
    uint32_t* h_stage = nullptr;   // pinned: results on their way to the caller's arrays
    size_t stage_words = 0;

    Workspace ws_dec, ws_pre, ws_score;
    MetaRing meta_dec, meta_pre, meta_score;
    Profiler prof;

    // ---- stage state (host integers)
    int N = 0;
    std::vector<Sample> smp;
    std::vector<int> h_prompt;            // packed prompts
    std::vector<int64_t> h_prompt_off;
    std::vector<int> h_forced;            // [N * max_ctx] imposed token per output index, -1 = free
    std::deque<int> waiting;
    std::vector<int> active;
    std::vector<int> free_list;
    int reserved = 0;
    std::vector<int> retired;
    size_t n_scored = 0;
    std::vector<int> batch_offsets{0};
    std::vector<int> batch_step;
    int step = 0;
    bool score_used = false;
    int64_t acc_weight_bytes = 0, acc_kv_bytes = 0, acc_prefill_tokens = 0;

    int fail(int code, const char* fmt, ...) {
        va_list ap;
        va_start(ap, fmt);
        vsnprintf(err, sizeof err, fmt, ap);
        va_end(ap);
        return code;
    }
};

#define HIPCK(ctx, call)                                                                       \
    do {                                                                                       \
        hipError_t e_ = (call);                                                                \
        if (e_ != hipSuccess)                                                                  \
            return (ctx)->fail(RLHF_EDEVICE, "%s failed: %s (%s:%d)", #call, hipGetErrorString(e_), \
                               __FILE__, __LINE__);                                            \
    } while (0)

namespace {

int ceil_div(int a, int b) { return (a + b - 1) / b; }

// Run `launch` (a callable returning hipError_t), timing it if this launch is sampled.
template <typename F>
hipError_t profiled(rlhf_ctx* c, hipStream_t st, int cls, double bytes, double flops, F&& launch) {
    Profiler& p = c->prof;
    if (!p.on) return launch();
    const int64_t k = p.launches[cls]++;
    p.tot_bytes[cls] += bytes;
    p.tot_flops[cls] += flops;
    if (k % p.every != 0) return launch();
    if (p.n_used >= Profiler::kMaxSamples) { p.dropped[cls] += 1; return launch(); }
    if (p.n_used == p.recs.size()) {
        Profiler::Rec r{};
        hipError_t e = hipEventCreate(&r.a);
        if (e != hipSuccess) return e;
        e = hipEventCreate(&r.b);
        if (e != hipSuccess) return e;
        p.recs.push_back(r);
    }
    Profiler::Rec& r = p.recs[p.n_used++];
    r.cls = cls;
    r.bytes = bytes;
    r.flops = flops;
    hipError_t e = hipEventRecord(r.a, st);
    if (e != hipSuccess) return e;
    e = launch();
    if (e != hipSuccess) return e;
    return hipEventRecord(r.b, st);
}

// Fold the finished event pairs into the per-class sums (both streams must have drained).
hipError_t profiler_fold(Profiler& p) {
    for (size_t i = 0; i < p.n_used; ++i) {
        float ms = 0.f;
        hipError_t e = hipEventElapsedTime(&ms, p.recs[i].a, p.recs[i].b);
        if (e != hipSuccess) return e;
        const int k = p.recs[i].cls;
        p.sampled[k] += 1;
        p.s_ms[k] += ms;
        p.s_bytes[k] += p.recs[i].bytes;
        p.s_flops[k] += p.recs[i].flops;
    }
    p.n_used = 0;
    return hipSuccess;
}

// Activation and KV-pool type: float for a float model, IEEE half for a bf16 model.
int act_type(const rlhf_ctx* c, bool /*batch*/) { return c->dtype == kBF16 ? kF16 : kF32; }

hipError_t gemm_profiled(rlhf_ctx* c, hipStream_t st, int cls, int adt, const void* A, const void* W, float* C,
                         int M, int N, int K, int nsplit, bool w_is_half_copy = false) {
    const double bytes = ((double)N * K + (double)M * K) * c->esz + (double)M * N * 4;
    return profiled(c, st, cls, bytes, 2.0 * M * N * K,
                    [&] { return launch_gemm(st, w_is_half_copy ? kF16 : c->dtype, adt, A, W, C, M, N, K, nsplit); });
}

template <typename T>
hipError_t dev_alloc(Workspace* ws, T** p, size_t n_bytes) {
    void* q = nullptr;
    hipError_t e = hipMalloc(&q, n_bytes ? n_bytes : 256);
    if (e == hipSuccess) {
        *p = (T*)q;
        if (ws) ws->owned.push_back(q);
    }
    return e;
}

int alloc_workspace(rlhf_ctx* c, Workspace& ws, int rows, bool decode) {
    const rlhf_model_cfg& m = c->mc;
    const size_t d = m.d_model, qd = (size_t)m.n_q_heads * m.head_dim, kvd = (size_t)m.n_kv_heads * m.head_dim;
    const size_t qkv_w = qd + 2 * kvd, f = m.ffn, V = m.vocab, es = c->esz;
    ws.rows_cap = rows;
    const size_t widest = std::max({qkv_w, 2 * f, d});
    if (decode) {
        // room for split-K partials of few-row GEMMs and for [rows, vocab] logits
        ws.part_cap = std::max((size_t)rows * std::max(widest, V) * 2, (size_t)16 * 16 * std::max(widest, V));
        ws.attn_slots = std::max((size_t)rows * m.n_q_heads, (size_t)16384);
    } else {
        ws.part_cap = (size_t)rows * widest;
        ws.logit_rows = std::min(rows, 2048);
    }
    HIPCK(c, dev_alloc(&ws, &ws.h, rows * d * 4));
    HIPCK(c, dev_alloc(&ws, (char**)&ws.xn, rows * d * es));
    HIPCK(c, dev_alloc(&ws, &ws.part, ws.part_cap * 4));
    HIPCK(c, dev_alloc(&ws, (char**)&ws.q, rows * qd * es));
    HIPCK(c, dev_alloc(&ws, (char**)&ws.attn, rows * qd * es));
    HIPCK(c, dev_alloc(&ws, (char**)&ws.act, rows * f * es));
    HIPCK(c, dev_alloc(&ws, (char**)&ws.xsel, rows * d * 4));    // float rows for the value / reward head
    HIPCK(c, dev_alloc(&ws, &ws.pick_scratch, pick_scratch_floats(rows) * 4));
    const size_t few = c->dtype == kF32 ? std::min(rows, kStreamF32Rows) : kStreamMaxRows;
    HIPCK(c, dev_alloc(&ws, &ws.ssq, few * kSsqStride * 4));
    HIPCK(c, dev_alloc(&ws, &ws.scale, 2 * few * 4));
    ws.few = (int)few;
    if (decode) {
        HIPCK(c, dev_alloc(&ws, &ws.attn_acc, ws.attn_slots * m.head_dim * 4));
        HIPCK(c, dev_alloc(&ws, &ws.attn_ml, ws.attn_slots * 2 * 4));
    } else {
        HIPCK(c, dev_alloc(&ws, (char**)&ws.k, rows * kvd * es));
        HIPCK(c, dev_alloc(&ws, (char**)&ws.v, rows * kvd * es));
        HIPCK(c, dev_alloc(&ws, &ws.logits, (size_t)ws.logit_rows * V * 4));
    }
    return RLHF_OK;
}

void free_workspace(Workspace& ws) {
    for (void* p : ws.owned) (void)hipFree(p);
    ws.owned.clear();
}

const char* layer_ptr(const void* base, int layer, size_t rows, size_t cols, int esz) {
    return (const char*)base + (size_t)layer * rows * cols * esz;
}

int nsplit_for(const rlhf_ctx* c, const Workspace& ws, int M, int N, int K) {
    const size_t per = (size_t)M * N;
    int cap = (int)std::min<size_t>(16, per ? ws.part_cap / per : 1);
    if (cap < 1) cap = 1;
    return gemm_choose_nsplit(c->dtype, M, N, K, cap);
}

enum AttnMode { kModeDecode, kModeBatch };

struct PassMeta {         // device pointers into a MetaRing arena
    const int* tok_idx = nullptr;
    const int* pos = nullptr;
    const int* kv_dst = nullptr;       // NULL: no pool writes
    const int* row_sample = nullptr;   // decode
    const int* ctx_len = nullptr;      // decode
    int max_pages = 0;                 // decode: of the longest context
    const int* tile_start = nullptr;   // batch: query tiles of the packed attention
    const int* tile_q0 = nullptr;
    const int* tile_len = nullptr;
    int n_tiles = 0, longest = 0;      // tiles; rows of the longest sequence
    double attn_bytes = 0, attn_flops = 0;   // algorithmic, per layer (for the profiler)
};

// Few rows: every layer runs on the projections of gemm_stream.hip.  Float ones in groups of 16 rows, each of which reads the
// whole matrix again: up to 32 rows, beyond that as long as the four projections together are estimated no slower than on
// the kernels of gemm.hip and gemm_f32.hip.  Prefill, us a layer, groups / those (/ all in vector code with norm, rotary and
// SwiGLU kernels): d = 256, ffn = 688 192 rows 45 / 58 / 65, 448 69 / 63 / 92; ffn = 4096 48 rows 54 / 59 / 66, 96 69 / 65 / 74, 192
// 92 / 70 / 84; ffn = 11008 24 rows 86 / 89 / 96, 96 128 / 102 / 112; d = 256 with 32 heads 96 rows 62 / 64 / 75, 320 124 / 85 / 116; 512
// 192 rows 69 / 79 / 93, 320 92 / 88 / 123; 1024 96 rows 104 / 105 / 107; 2048 32 rows 172 / 204, 64 265 / 222; 4096 32 rows 556 / 588,
// 64 934 / 633.
bool stream_pass(const rlhf_ctx* c, int rows) {
    const rlhf_model_cfg& m = c->mc;
    if (c->dtype == kF32) {
        if (m.d_model % 16 || rows > kStreamF32Rows) return false;
        if (rows <= 32) return true;
        const int d = m.d_model, qd = m.n_q_heads * m.head_dim, qkv_w = qd + 2 * m.n_kv_heads * m.head_dim;
        double us = 0;
        for (auto [N, K] : {std::pair{qkv_w, d}, std::pair{d, qd}, std::pair{2 * m.ffn, d}, std::pair{d, m.ffn}})
            us += stream_f32_us(rows, N, K) - gemm_f32_us(rows, N, K);
        return us <= 0;
    }
    return c->dtype == kBF16 && rows <= kRowsMaxRows && m.d_model % 64 == 0 && (m.n_q_heads * m.head_dim) % 64 == 0 &&
           m.ffn % 64 == 0;
}

// The LM head of a float model, by its own times; where the groups can take the final norm along, the others need an RMSNorm
// kernel.  us, groups / unsplit (/ vector code): 4096 columns of K = 256 48 rows 7.7 / 8.4, 64 9.5 / 9.4, 200 26 / 11 / 17, 448 53 / 14 / 20;
// 32000 of K = 256 17 rows 28 / 12 / 19, 64 59 / 19 / 21; 515 of K = 256 448 rows 9.7 / 11.3; 4096 of K = 1024 128 rows 31 / 36,
// 200 47 / 37; 32000 of K = 768 32 rows 58 / 32 / 53.
bool head_in_groups(int rows, int vocab, int d, bool norm) {
    if (rows <= 16 || rows > kStreamF32Rows) return rows <= 16;
    return stream_f32_us(rows, vocab, d) <= (norm ? gemm_f32_us(rows, vocab, d) + 4. : gemm_f32_tall_us(rows, vocab, d));
}

// Norm input of a few-row projection over the residual stream: how ws.xn was scaled, the sums of squares
// its producer left, and the stream and gain themselves.
NormIn stream_norm(const rlhf_ctx* c, const Workspace& ws, const float* g, int n_ssq, float* s_in, float* s_out) {
    NormIn ni;
    ni.ssq = ws.ssq;
    ni.h = ws.h;
    ni.g = g;
    ni.n_ssq = n_ssq;
    ni.s_in = s_in;
    ni.s_out = s_out;
    ni.eps = c->mc.rms_eps;
    return ni;
}

// The layers of such a pass, 16-bit activations in the packed layout.  Where stream_resid says so: five
// kernels a layer (six when the contexts are split), the residual stream in ws.h is complete after every
// O and down projection, and ws.xn holds the next norm's input as gemm_stream.hip describes it, at the
// end that of the final norm (scale in ws.scale, sums in ws.ssq: *n_ssq per row; *pend_ns = 0).  Otherwise:
// seven kernels, O and down leave planes that RMSNorm adds, at the end *pend_ns of them.
int forward_layers_stream(rlhf_ctx* c, hipStream_t st, Workspace& ws, const RoleWeights& rw, int rows,
                          const PassMeta& pm, AttnMode mode, int attn_nsplit, int* pend_ns, int* n_ssq) {
    const rlhf_weights& w = rw.w;
    const rlhf_weights& wh = rw.h16;              // half copies (members may be NULL)
    const rlhf_model_cfg& m = c->mc;
    const int d = m.d_model, qd = m.n_q_heads * m.head_dim, kvd = m.n_kv_heads * m.head_dim;
    const int qkv_w = qd + 2 * kvd, f = m.ffn, es = c->esz, dt = c->dtype;
    const int gcls = mode == kModeDecode ? kGemmDecode : kGemmBatch;
    const bool resid = stream_resid(dt, rows, m.d_model);
    const size_t plane = (size_t)rows * d;
    const int cap = (int)std::min<size_t>(16, ws.part_cap / plane);
    const int adt = act_type(c, mode == kModeBatch);
    // row 0: row-major, whatever the width
    const ActLayout packed = adt == kF16 ? ActLayout{8, 8 * rows} : ActLayout{}, attn_layout = mode == kModeDecode ? packed : ActLayout{};
    float* sc[2] = {ws.scale, ws.scale + ws.few};
    auto gain_after = [&](int l) { return l + 1 < m.n_layers ? w.g_attn + (size_t)(l + 1) * d : w.g_final; };
    if (resid)
        HIPCK(c, launch_embed_norm(st, dt, c->d_tokens, pm.tok_idx, w.embed, ws.h, m.n_layers > 0 ? w.g_attn : w.g_final,
                                   ws.xn, packed, sc[0], ws.ssq, rows, d, m.vocab, m.rms_eps));
    else
        HIPCK(c, launch_embed(st, dt, c->d_tokens, pm.tok_idx, w.embed, ws.h, rows, d, m.vocab));
    *n_ssq = 1;
    int ns = 0;
    // k_gemm_rows, and the half copy of layer l's weights where there is one; or k_gemm_stream and the bf16 weights
    const bool many = dt == kBF16 && takes_gemm_rows(rows, d);
    auto project = [&](int md, const void* A, const void* w_bf16, const void* w_half, int l, int N, int K, const RowsEpi& ep,
                       int nsplit = 1) {
        const bool hw = many && w_half;
        const void* W = layer_ptr(hw ? w_half : w_bf16, l, N, K, es);
        const double bytes = ((double)N * K + (double)rows * K) * es + (double)rows * N * (md == 0 ? 4 : es);
        return profiled(c, st, gcls, bytes, 2.0 * rows * N * K,
                        [&] { return launch_gemm_stream(st, hw ? kF16 : dt, adt, md, A, W, ws.part, rows, N, K, ep, nsplit, many); });
    };
    // O and down projections: finish the residual stream, or leave planes and let RMSNorm do it
    auto into_stream = [&](const void* A, const ActLayout& la, const void* w_bf16, const void* w_half, int l, int K,
                           const float* g_next, float* s) -> int {
        RowsEpi ep;
        ep.a = la;
        if (resid) {
            ep.out = packed;
            ep.res.h = ws.h; ep.res.g = g_next; ep.res.x = ws.xn; ep.res.s = s; ep.res.ssq = ws.ssq;
            HIPCK(c, project(3, A, w_bf16, w_half, l, d, K, ep));
            *n_ssq = d / 16;
        } else {
            ns = many ? gemm_rows_nsplit(d, K, cap) : gemm_stream_nsplit(rows, d, K, cap);
            HIPCK(c, project(0, A, w_bf16, w_half, l, d, K, ep, ns));
        }
        return RLHF_OK;
    };
    for (int l = 0; l < m.n_layers; ++l) {
        if (!resid)
            HIPCK(c, launch_rmsnorm(st, adt, ws.h, ws.part, ns, plane, nullptr, w.g_attn + (size_t)l * d, ws.xn, rows, d,
                                    m.rms_eps, packed));
        RowsEpi ep;
        ep.a = packed;
        if (resid) ep.nrm = stream_norm(c, ws, w.g_attn + (size_t)l * d, *n_ssq, sc[0], sc[1]);
        ep.ro.pos = pm.pos;
        ep.ro.kv_dst = pm.kv_dst;
        ep.ro.table = c->d_rope;
        ep.ro.q = ws.q;
        ep.ro.k = mode == kModeBatch ? ws.k : nullptr;
        ep.ro.v = mode == kModeBatch ? ws.v : nullptr;
        ep.ro.pool = pm.kv_dst ? c->pool : nullptr;
        ep.ro.layer = l; ep.ro.n_layers = m.n_layers;
        ep.ro.n_q_heads = m.n_q_heads; ep.ro.n_kv_heads = m.n_kv_heads; ep.ro.head_dim = m.head_dim;
        ep.ro.page_tokens = c->ec.page_tokens;
        HIPCK(c, project(2, ws.xn, w.wqkv, wh.wqkv, l, qkv_w, d, ep));
        if (mode == kModeDecode) {
            HIPCK(c, profiled(c, st, kAttnDecode, pm.attn_bytes, pm.attn_flops, [&] {
                return launch_decode_attn(st, adt, ws.q, c->pool, c->d_page_table, c->max_pages, pm.row_sample,
                                          pm.ctx_len, ws.attn, ws.attn_acc, ws.attn_ml, rows, l, attn_nsplit, c->dm,
                                          attn_layout, pm.max_pages);
            }));
        } else {
            HIPCK(c, profiled(c, st, kAttnBatch, pm.attn_bytes, pm.attn_flops, [&] {
                if (adt == kF16)
                    return launch_flash_attn(st, ws.q, ws.k, ws.v, pm.tile_start, pm.tile_q0, pm.tile_len, ws.attn,
                                             pm.n_tiles, rows, c->dm);
                return launch_flash_attn_f32(st, (const float*)ws.q, (const float*)ws.k, (const float*)ws.v, pm.tile_start,
                                             pm.tile_q0, pm.tile_len, (float*)ws.attn, pm.n_tiles, pm.longest, c->dm);
            }));
        }
        int rc = into_stream(ws.attn, attn_layout, w.wo, wh.wo, l, qd, w.g_mlp + (size_t)l * d, sc[1]);
        if (rc) return rc;
        if (!resid)
            HIPCK(c, launch_rmsnorm(st, adt, ws.h, ws.part, ns, plane, nullptr, w.g_mlp + (size_t)l * d, ws.xn, rows, d,
                                    m.rms_eps, packed));
        RowsEpi eg;
        eg.a = eg.out = packed;
        if (resid) eg.nrm = stream_norm(c, ws, w.g_mlp + (size_t)l * d, *n_ssq, sc[1], sc[0]);
        eg.act = ws.act;
        eg.ffn = f;
        HIPCK(c, project(1, ws.xn, w.w_gate_up, wh.w_gate_up, l, 2 * f, d, eg));
        rc = into_stream(ws.act, packed, w.w_down, wh.w_down, l, f, gain_after(l), sc[0]);
        if (rc) return rc;
    }
    *pend_ns = ns;
    return RLHF_OK;
}

// Embedding and all decoder layers over `rows` rows.  On return ws.h holds the residual
// stream except for the last down-projection, whose split-K partials are still in ws.part:
// (*pend_ns, *pend_stride) describe them for the final norm.
int forward_layers(rlhf_ctx* c, hipStream_t st, Workspace& ws, const RoleWeights& rw, int rows,
                   const PassMeta& pm, AttnMode mode, int attn_nsplit, int* pend_ns,
                   size_t* pend_stride) {
    const rlhf_weights& w = rw.w;
    const rlhf_weights& wh = rw.h16;              // half copies (members may be NULL)
    const rlhf_model_cfg& m = c->mc;
    const int d = m.d_model, qd = m.n_q_heads * m.head_dim, kvd = m.n_kv_heads * m.head_dim;
    const int qkv_w = qd + 2 * kvd, f = m.ffn, es = c->esz, dt = c->dtype;
    const int gcls = mode == kModeDecode ? kGemmDecode : kGemmBatch;
    const int adt = act_type(c, mode == kModeBatch);
    const int qdt = adt;               // q/k/v of a pass share the activation type
    if (mode == kModeBatch && stream_pass(c, rows)) {
        int n_ssq;
        *pend_stride = (size_t)rows * d;
        return forward_layers_stream(c, st, ws, rw, rows, pm, mode, 1, pend_ns, &n_ssq);
    }
    HIPCK(c, launch_embed(st, dt, c->d_tokens, pm.tok_idx, w.embed, ws.h, rows, d, m.vocab));
    // A projection of layer l that leaves `planes` planes: run(W, half) on the bf16 weights, or where the tall kernel takes it
    // on their half copy, if need be made now (behind the planes; earlier ones have been read by then)
    auto project_bf16 = [&](const void* w_bf16, const void* w_half, int l, size_t N, size_t K, bool tall, int planes, double bytes,
                            auto run) {
        const bool copy = w_half && tall;
        const void* W = layer_ptr(copy ? w_half : w_bf16, l, N, K, es);
        const size_t off = ((size_t)planes * rows * N + 63) / 64 * 64;
        const bool convert = !copy && tall && dt == kBF16 && !c->ec.half_weight_copies && rows >= kConvertRows &&
                             half_operands_ok(kF16, rows, (long)N, (long)K) && off + (N * K + 1) / 2 <= ws.part_cap;
        return profiled(c, st, gcls, bytes, 2.0 * rows * N * K, [&] {
            if (!convert) return run(W, copy);
            const hipError_t e = launch_bf16_to_half(st, W, ws.part + off, N * K);
            return e == hipSuccess ? run((const void*)(ws.part + off), true) : e;
        });
    };
    const bool can16 = dt == kBF16 && adt == kF16 && d % 64 == 0;
    // float models: a projection that is not split runs on the kernel of gemm_f32.hip, its consumer in the epilogue
    auto whole_f32 = [&](int N, int K) { return dt == kF32 && nsplit_for(c, ws, rows, N, K) == 1; };
    auto project_f32 = [&](int mode, const void* A, const void* W, int N, int K, const RowsEpi& ep) {
        const double bytes = ((double)N * K + (double)rows * K + (double)rows * N) * es;
        return profiled(c, st, gcls, bytes, 2.0 * rows * N * K,
                        [&] { return launch_gemm_f32_tall(st, mode, (const float*)A, (const float*)W, nullptr, rows, N, K, ep); });
    };
    int pns = 0;
    const size_t pstride = (size_t)rows * d;
    // O and down projections: an unsplit tall one finishes the residual stream, the others leave pns planes that
    // RMSNorm adds
    auto into_stream = [&](const void* A, const void* w_bf16, const void* w_half, int l, int K) -> int {
        if (whole_f32(d, K)) {
            pns = 0;
            RowsEpi ep;
            ep.res.h = ws.h;
            HIPCK(c, project_f32(3, A, layer_ptr(w_bf16, l, d, K, es), d, K, ep));
            return RLHF_OK;
        }
        pns = nsplit_for(c, ws, rows, d, K);
        const bool tall = gemm_is_tall(rows, d, K, pns);
        const bool whole = tall && rows > 256 && pns == 1 && dt == kBF16 && d % 4 == 0;
        if (whole) pns = 0;
        const double bytes = ((double)d * K + (double)rows * K) * es + (double)rows * d * (whole ? 8 : 4);
        HIPCK(c, project_bf16(w_bf16, w_half, l, d, K, tall && adt == kF16, pns, bytes, [&](const void* W, bool half) {
            return whole ? launch_gemm_tall_add(st, half ? kF16 : dt, adt, A, W, ws.h, rows, d, K)
                         : launch_gemm(st, half ? kF16 : dt, adt, A, W, ws.part, rows, d, K, pns);
        }));
        return RLHF_OK;
    };
    for (int l = 0; l < m.n_layers; ++l) {
        HIPCK(c, launch_rmsnorm(st, adt, ws.h, ws.part, pns, pstride, nullptr, w.g_attn + (size_t)l * d,
                                ws.xn, rows, d, m.rms_eps));
        int ns = 0;
        const bool f32 = whole_f32(qkv_w, d);
        if (f32 || (mode == kModeBatch && gemm_rope_supported(dt, adt, rows, d, c->dm))) {
            // tall pass: rotary, rounding and the q / k / v / pool scatter ride in the GEMM's epilogue
            RopeOut ro;
            ro.pos = pm.pos;
            ro.kv_dst = pm.kv_dst;
            ro.table = c->d_rope;
            ro.q = ws.q;
            ro.k = mode == kModeBatch ? ws.k : nullptr;
            ro.v = mode == kModeBatch ? ws.v : nullptr;
            ro.pool = pm.kv_dst ? c->pool : nullptr;
            ro.layer = l; ro.n_layers = m.n_layers;
            ro.n_q_heads = m.n_q_heads; ro.n_kv_heads = m.n_kv_heads; ro.head_dim = m.head_dim;
            ro.page_tokens = c->ec.page_tokens;
            if (f32) {
                RowsEpi ep;
                ep.ro = ro;
                HIPCK(c, project_f32(2, ws.xn, layer_ptr(w.wqkv, l, qkv_w, d, es), qkv_w, d, ep));
            } else {
                const double bytes = ((double)qkv_w * d + (double)rows * d) * es + (double)rows * qkv_w * es;
                HIPCK(c, project_bf16(w.wqkv, wh.wqkv, l, qkv_w, d, can16, 0, bytes, [&](const void* W, bool half) {
                    return launch_gemm_rope(st, half ? kF16 : dt, adt, ws.xn, W, rows, d, ro);
                }));
            }
        } else {
            ns = nsplit_for(c, ws, rows, qkv_w, d);
            const bool hw = wh.wqkv && adt == kF16 && gemm_is_tall(rows, qkv_w, d, ns);
            HIPCK(c, gemm_profiled(c, st, gcls, adt, ws.xn, layer_ptr(hw ? wh.wqkv : w.wqkv, l, qkv_w, d, es), ws.part, rows,
                                   qkv_w, d, ns, hw));
            HIPCK(c, launch_rope_kv(st, qdt, adt, ws.part, ns, (size_t)rows * qkv_w, pm.pos, pm.kv_dst, c->d_rope,
                                    ws.q, mode == kModeBatch ? ws.k : nullptr,
                                    mode == kModeBatch ? ws.v : nullptr, pm.kv_dst ? c->pool : nullptr, l,
                                    rows, c->dm));
        }
        if (mode == kModeDecode) {
            HIPCK(c, profiled(c, st, kAttnDecode, pm.attn_bytes, pm.attn_flops, [&] {
                return launch_decode_attn(st, adt, ws.q, c->pool, c->d_page_table, c->max_pages, pm.row_sample,
                                          pm.ctx_len, ws.attn, ws.attn_acc, ws.attn_ml, rows, l, attn_nsplit,
                                          c->dm, ActLayout{}, pm.max_pages);
            }));
        } else {
            HIPCK(c, profiled(c, st, kAttnBatch, pm.attn_bytes, pm.attn_flops, [&] {
                if (adt == kF16)
                    return launch_flash_attn(st, ws.q, ws.k, ws.v, pm.tile_start, pm.tile_q0, pm.tile_len, ws.attn,
                                             pm.n_tiles, rows, c->dm);
                return launch_flash_attn_f32(st, (const float*)ws.q, (const float*)ws.k, (const float*)ws.v, pm.tile_start,
                                             pm.tile_q0, pm.tile_len, (float*)ws.attn, pm.n_tiles, pm.longest, c->dm);
            }));
        }
        int rc = into_stream(ws.attn, w.wo, wh.wo, l, qd);
        if (rc) return rc;
        HIPCK(c, launch_rmsnorm(st, adt, ws.h, ws.part, pns, pstride, nullptr, w.g_mlp + (size_t)l * d, ws.xn, rows, d,
                                m.rms_eps));
        if (whole_f32(2 * f, d)) {
            RowsEpi ep;
            ep.act = ws.act;
            ep.ffn = f;
            HIPCK(c, project_f32(1, ws.xn, layer_ptr(w.w_gate_up, l, 2 * (size_t)f, d, es), 2 * f, d, ep));
        } else if (gemm_swiglu_supported(dt, adt, rows, f, d)) {
            const double bytes = (2.0 * f * d + (double)rows * d) * es + (double)rows * f * es;
            HIPCK(c, project_bf16(w.w_gate_up, wh.w_gate_up, l, 2 * (size_t)f, d, can16, 0, bytes, [&](const void* W, bool half) {
                return launch_gemm_swiglu(st, half ? kF16 : dt, adt, ws.xn, W, ws.act, rows, f, d);
            }));
        } else {
            ns = nsplit_for(c, ws, rows, 2 * f, d);
            const bool hw = wh.w_gate_up && adt == kF16 && gemm_is_tall(rows, 2 * f, d, ns);
            HIPCK(c, gemm_profiled(c, st, gcls, adt, ws.xn, layer_ptr(hw ? wh.w_gate_up : w.w_gate_up, l, 2 * (size_t)f, d, es),
                                   ws.part, rows, 2 * f, d, ns, hw));
            HIPCK(c, launch_swiglu(st, adt, ws.part, ns, (size_t)rows * 2 * f, ws.act, rows, f));
        }
        rc = into_stream(ws.act, w.w_down, wh.w_down, l, f);
        if (rc) return rc;
    }
    *pend_ns = pns;
    *pend_stride = pstride;
    return RLHF_OK;
}

}  // namespace

// =========================================================================== create/destroy

extern "C" const char* rlhf_last_error(const rlhf_ctx* ctx) { return ctx ? ctx->err : g_create_error; }

// Message of a failed call that has no context (rlhf_create, the kernel-level entry points);
// read back with rlhf_last_error(NULL) on the same thread.
void rlhf::set_global_error(const char* msg) { snprintf(g_create_error, sizeof g_create_error, "%s", msg); }

extern "C" void rlhf_destroy(rlhf_ctx* c) {
    if (!c) return;
    for (hipStream_t st : {c->sd_full, c->ss_full, c->sd_part, c->ss_part})
        if (st) (void)hipStreamSynchronize(st);
    free_workspace(c->ws_dec);
    free_workspace(c->ws_pre);
    free_workspace(c->ws_score);
    for (RoleWeights& r : c->roles) {
        for (void* p : r.owned) (void)hipFree(p);
        r.owned.clear();
    }
    c->meta_dec.destroy();
    c->meta_pre.destroy();
    c->meta_score.destroy();
    void* bufs[] = {c->pool, c->d_page_table, c->d_tokens, c->d_lp_actor, c->d_lp_rescored, c->d_lp_ref,
                    c->d_values, c->d_reward, c->d_rope, c->d_picked, c->d_nonfinite};
    for (void* p : bufs)
        if (p) (void)hipFree(p);
    if (c->h_picked) (void)hipHostFree(c->h_picked);
    if (c->h_stage) (void)hipHostFree(c->h_stage);
    hipEvent_t evs[] = {c->ev_dep, c->ev_d0, c->ev_d1, c->ev_s0, c->ev_s1, c->ev_sw_d, c->ev_sw_s, c->ev_score_last};
    for (hipEvent_t e : evs)
        if (e) (void)hipEventDestroy(e);
    for (hipEvent_t e : c->step_events) (void)hipEventDestroy(e);
    for (auto& r : c->prof.recs) { (void)hipEventDestroy(r.a); (void)hipEventDestroy(r.b); }
    if (c->own_sd && c->sd_full) (void)hipStreamDestroy(c->sd_full);
    if (c->own_ss && c->ss_full) (void)hipStreamDestroy(c->ss_full);
    if (c->sd_part) (void)hipStreamDestroy(c->sd_part);
    if (c->ss_part) (void)hipStreamDestroy(c->ss_part);
    delete c;
}

static int create_impl(rlhf_ctx* c) {
    const rlhf_model_cfg& m = c->mc;
    const rlhf_engine_cfg& e = c->ec;
    if (m.n_layers < 0 || m.d_model <= 0 || m.n_q_heads <= 0 || m.n_kv_heads <= 0 || m.ffn <= 0 || m.vocab <= 1)
        return c->fail(RLHF_EINVAL, "model dimensions must be positive");
    if (m.dtype != RLHF_FP32 && m.dtype != RLHF_BF16) return c->fail(RLHF_EINVAL, "dtype must be FP32 or BF16");
    if (m.d_model % 8 || m.ffn % 8 || m.d_model > 8192)
        return c->fail(RLHF_EINVAL, "d_model and ffn must be multiples of 8, d_model <= 8192");
    if (m.n_q_heads % m.n_kv_heads) return c->fail(RLHF_EINVAL, "n_q_heads must be a multiple of n_kv_heads");
    const int G = m.n_q_heads / m.n_kv_heads;
    const bool attn_ok = (m.head_dim == 128 && (G == 1 || (G == 8 && m.dtype == RLHF_BF16))) ||
                         (m.head_dim == 64 && G == 1);
    if (!attn_ok)
        return c->fail(RLHF_EINVAL, "unsupported attention shape: head_dim %d, group %d (have 128x{1,8}, 64x1)",
                       m.head_dim, G);
    if (e.page_tokens != 16) return c->fail(RLHF_EINVAL, "page_tokens must be 16");
    if (e.max_samples <= 0 || e.max_ctx <= 1 || e.max_active <= 0 || e.max_batch_tokens < e.max_ctx)
        return c->fail(RLHF_EINVAL, "engine limits: need max_samples, max_active > 0, max_batch_tokens >= max_ctx > 1");
    if (e.eos_id < 0 || e.eos_id >= m.vocab) return c->fail(RLHF_EINVAL, "eos_id out of range");
    if (!(m.rms_eps >= 0.f) || !(m.rope_base > 1.f)) return c->fail(RLHF_EINVAL, "rms_eps / rope_base");

    c->dtype = m.dtype == RLHF_BF16 ? kBF16 : kF32;
    c->esz = m.dtype == RLHF_BF16 ? 2 : 4;
    c->dm = Dims{m.n_layers, m.d_model, m.n_q_heads, m.n_kv_heads, m.head_dim, m.ffn, m.vocab, e.page_tokens};
    c->max_pages = ceil_div(e.max_ctx, e.page_tokens);
    const size_t page_bytes = std::max<size_t>(pool_page_elems(c->dm) * c->esz, 1);
    const int64_t pages = e.kv_pool_bytes / (int64_t)page_bytes;
    if (pages < 1 || pages > (int64_t)1 << 27)
        return c->fail(RLHF_ENOMEM, "kv_pool_bytes %lld holds %lld pages of %zu bytes",
                       (long long)e.kv_pool_bytes, (long long)pages, page_bytes);
    c->pool_pages = (int)pages;

    int n_cus = 0;
    {
        int dev = 0;
        HIPCK(c, hipGetDevice(&dev));
        HIPCK(c, hipDeviceGetAttribute(&n_cus, hipDeviceAttributeMultiprocessorCount, dev));
    }
    if (e.half_weight_copies != 0 && e.half_weight_copies != 1)
        return c->fail(RLHF_EINVAL, "half_weight_copies must be 0 or 1");
    if (e.corun_decode_cus < 0 || e.corun_decode_cus >= n_cus || e.corun_decode_cus % 32 || (e.optimistic_admission != 0 && e.optimistic_admission != 1))
        return c->fail(RLHF_EINVAL, "corun_decode_cus must be a multiple of 32 in [0, %d) and optimistic_admission 0 or 1", n_cus);
    auto make_masked = [&](hipStream_t* st, int lo, int hi) -> hipError_t {   // CU-mask bits [lo, hi)
        std::vector<uint32_t> mask((n_cus + 31) / 32, 0u);
        for (int bit = lo; bit < hi; ++bit) mask[bit >> 5] |= 1u << (bit & 31);
        return hipExtStreamCreateWithCUMask(st, (uint32_t)mask.size(), mask.data());
    };
    if (e.decode_stream) c->sd_full = (hipStream_t)e.decode_stream;
    else { HIPCK(c, hipStreamCreateWithFlags(&c->sd_full, hipStreamNonBlocking)); c->own_sd = true; }
    if (e.score_stream) c->ss_full = (hipStream_t)e.score_stream;
    else { HIPCK(c, hipStreamCreateWithFlags(&c->ss_full, hipStreamNonBlocking)); c->own_ss = true; }
    if (e.corun_decode_cus > 0) {
        HIPCK(c, make_masked(&c->sd_part, 0, e.corun_decode_cus));
        HIPCK(c, make_masked(&c->ss_part, e.corun_decode_cus, n_cus));
    }
    c->sd = c->sd_full;
    c->ss = c->ss_full;
    HIPCK(c, hipEventCreateWithFlags(&c->ev_sw_d, hipEventDisableTiming));
    HIPCK(c, hipEventCreateWithFlags(&c->ev_sw_s, hipEventDisableTiming));
    HIPCK(c, hipEventCreateWithFlags(&c->ev_score_last, hipEventDisableTiming));
    HIPCK(c, hipEventCreateWithFlags(&c->ev_dep, hipEventDisableTiming));
    HIPCK(c, hipEventCreate(&c->ev_d0));
    HIPCK(c, hipEventCreate(&c->ev_d1));
    HIPCK(c, hipEventCreate(&c->ev_s0));
    HIPCK(c, hipEventCreate(&c->ev_s1));

    const size_t ns = e.max_samples, mc = e.max_ctx;
    HIPCK(c, hipMalloc(&c->pool, (size_t)c->pool_pages * page_bytes));
    HIPCK(c, hipMalloc((void**)&c->d_page_table, ns * c->max_pages * sizeof(int)));
    HIPCK(c, hipMalloc((void**)&c->d_tokens, ns * mc * sizeof(int)));
    HIPCK(c, hipMalloc((void**)&c->d_lp_actor, ns * mc * 4));
    HIPCK(c, hipMalloc((void**)&c->d_lp_rescored, ns * mc * 4));
    HIPCK(c, hipMalloc((void**)&c->d_lp_ref, ns * mc * 4));
    HIPCK(c, hipMalloc((void**)&c->d_values, ns * mc * 4));
    HIPCK(c, hipMalloc((void**)&c->d_reward, ns * 4));
    HIPCK(c, hipMalloc((void**)&c->d_picked, (size_t)e.max_active * sizeof(int)));
    HIPCK(c, hipMalloc((void**)&c->d_nonfinite, sizeof(int)));
    HIPCK(c, hipMemset(c->d_nonfinite, 0, sizeof(int)));
    HIPCK(c, hipHostMalloc((void**)&c->h_picked, (size_t)e.max_active * sizeof(int), hipHostMallocDefault));
    // one sample's five result arrays at least, normally a whole stage's
    c->stage_words = std::max<size_t>((size_t)1 << 20, 5 * mc + ns + 64);
    HIPCK(c, hipHostMalloc((void**)&c->h_stage, c->stage_words * 4, hipHostMallocDefault));
    HIPCK(c, hipMemset(c->d_page_table, 0, ns * c->max_pages * sizeof(int)));

    {   // rotary table in double, stored as float (cos, sin) per (position, pair)
        const int half = m.head_dim / 2;
        std::vector<float> tab((size_t)e.max_ctx * m.head_dim);
        for (int p = 0; p < e.max_ctx; ++p)
            for (int k = 0; k < half; ++k) {
                const double ang = (double)p * std::pow((double)m.rope_base, -2.0 * k / m.head_dim);
                tab[((size_t)p * half + k) * 2] = (float)std::cos(ang);
                tab[((size_t)p * half + k) * 2 + 1] = (float)std::sin(ang);
            }
        HIPCK(c, hipMalloc((void**)&c->d_rope, tab.size() * 4));
        HIPCK(c, hipMemcpy(c->d_rope, tab.data(), tab.size() * 4, hipMemcpyHostToDevice));
    }

    int rc;
    if ((rc = alloc_workspace(c, c->ws_dec, e.max_active, true))) return rc;
    if ((rc = alloc_workspace(c, c->ws_pre, e.max_batch_tokens, false))) return rc;
    if ((rc = alloc_workspace(c, c->ws_score, e.max_batch_tokens, false))) return rc;
    HIPCK(c, c->meta_dec.init((size_t)e.max_active * 10 + (size_t)e.max_active * 2 + 64));
    // prefill metadata also carries the page-table updates of the admitted prompts
    HIPCK(c, c->meta_pre.init((size_t)e.max_batch_tokens * 8 + (size_t)e.max_samples * 12 +
                              2 * ((size_t)e.max_batch_tokens / e.page_tokens + e.max_samples) + 64));
    HIPCK(c, c->meta_score.init((size_t)e.max_batch_tokens * 8 + (size_t)e.max_samples * 8 + 64));
    return RLHF_OK;
}

extern "C" int rlhf_create(const rlhf_model_cfg* model, const rlhf_engine_cfg* engine, rlhf_ctx** out) {
    if (out) *out = nullptr;
    if (!model || !engine || !out) {
        snprintf(g_create_error, sizeof g_create_error, "rlhf_create: NULL argument");
        return RLHF_EINVAL;
    }
    rlhf_ctx* c = new rlhf_ctx();
    c->mc = *model;
    c->ec = *engine;
    const int rc = create_impl(c);
    if (rc != RLHF_OK) {
        snprintf(g_create_error, sizeof g_create_error, "%s", c->err);
        rlhf_destroy(c);
        return rc;
    }
    *out = c;
    return RLHF_OK;
}

extern "C" int rlhf_load_weights(rlhf_ctx* c, int role, const rlhf_weights* w) {
    if (!c) return RLHF_EINVAL;
    if (role < 0 || role > 3 || !w) return c->fail(RLHF_EINVAL, "rlhf_load_weights: bad role or NULL weights");
    if (!w->embed || !w->g_final || !w->head ||
        (c->mc.n_layers > 0 && (!w->wqkv || !w->wo || !w->w_gate_up || !w->w_down || !w->g_attn || !w->g_mlp)))
        return c->fail(RLHF_EINVAL, "rlhf_load_weights: NULL tensor");
    const void* ptrs[] = {w->embed, w->wqkv, w->wo, w->w_gate_up, w->w_down, w->g_attn, w->g_mlp, w->g_final, w->head};
    for (const void* p : ptrs)
        if (p && ((uintptr_t)p & 15)) return c->fail(RLHF_EINVAL, "rlhf_load_weights: tensors must be 16-byte aligned");
    RoleWeights& rw = c->roles[role];
    int rc = rlhf_sync(c);                       // nothing in flight may still read copies about to be freed
    if (rc) return rc;
    for (void* p : rw.owned) (void)hipFree(p);
    rw.owned.clear();
    rw.h16 = rlhf_weights{};
    rw.w = *w;
    rw.bound = true;
    if (c->ec.half_weight_copies && c->dtype == kBF16) {
        const rlhf_model_cfg& m = c->mc;
        const size_t d = m.d_model, qd = (size_t)m.n_q_heads * m.head_dim, kvd = (size_t)m.n_kv_heads * m.head_dim;
        const size_t L = m.n_layers, f = m.ffn;
        struct Item { const void* src; const void** dst; size_t n, per_matrix; };
        const Item items[] = {
            {w->wqkv, &rw.h16.wqkv, L * (qd + 2 * kvd) * d, (qd + 2 * kvd) * d},
            {w->wo, &rw.h16.wo, L * d * qd, d * qd},
            {w->w_gate_up, &rw.h16.w_gate_up, L * 2 * f * d, 2 * f * d},
            {w->w_down, &rw.h16.w_down, L * d * f, d * f},
            {w->head, &rw.h16.head, (role == RLHF_ACTOR || role == RLHF_REF) ? (size_t)m.vocab * d : 0, (size_t)m.vocab * d},
        };
        // launches with copies are for operands below 4 GiB: a matrix, or a pass's activations, beyond that stays on
        // the bf16-weight path
        const size_t lim = (size_t)1 << 32;
        const bool acts_fit = (size_t)c->ec.max_batch_tokens * std::max(d, f) * 2 < lim;
        for (const Item& it : items) {
            if (it.n == 0 || !it.src || !acts_fit || it.per_matrix * 2 >= lim) continue;
            void* p = nullptr;
            if (hipMalloc(&p, it.n * 2) != hipSuccess) {
                (void)hipGetLastError();
                for (void* q : rw.owned) (void)hipFree(q);
                rw.owned.clear();
                rw.h16 = rlhf_weights{};
                rw.bound = false;
                return c->fail(RLHF_ENOMEM, "rlhf_load_weights: no device memory for the half copies of role %d "
                                            "(%zu bytes); leave room beside kv_pool_bytes or turn half_weight_copies off",
                               role, it.n * 2);
            }
            rw.owned.push_back(p);
            HIPCK(c, launch_bf16_to_half(c->sd_full, it.src, p, it.n));
            *it.dst = p;
        }
        HIPCK(c, hipStreamSynchronize(c->sd_full));
    }
    return RLHF_OK;
}

extern "C" int rlhf_sync(rlhf_ctx* c) {
    if (!c) return RLHF_EINVAL;
    for (hipStream_t st : {c->sd_full, c->ss_full, c->sd_part, c->ss_part})
        if (st) HIPCK(c, hipStreamSynchronize(st));
    return RLHF_OK;
}

namespace {
// Continue a logical stream (decode or scoring) on another HIP stream: the new one first waits
// for everything issued on the old one.
int switch_stream(rlhf_ctx* c, hipStream_t* cur, hipStream_t next, hipEvent_t ev) {
    if (*cur == next || !next) return RLHF_OK;
    HIPCK(c, hipEventRecord(ev, *cur));
    HIPCK(c, hipStreamWaitEvent(next, ev, 0));
    *cur = next;
    return RLHF_OK;
}
}  // namespace

// =================================================================================== submit

extern "C" int rlhf_submit(rlhf_ctx* c, int32_t n, const int32_t* prompt_tokens,
                           const int64_t* prompt_offsets, const int32_t* max_new,
                           const int32_t* forced_len, const int32_t* forced_tokens,
                           const int64_t* forced_offsets) {
    if (!c) return RLHF_EINVAL;
    if (n < 0 || n > c->ec.max_samples) return c->fail(RLHF_EINVAL, "rlhf_submit: n = %d outside [0, %d]", n, c->ec.max_samples);
    if (n > 0 && (!prompt_tokens || !prompt_offsets || !max_new)) return c->fail(RLHF_EINVAL, "rlhf_submit: NULL array");
    if (forced_tokens && !forced_offsets) return c->fail(RLHF_EINVAL, "rlhf_submit: forced_tokens without forced_offsets");
    const int mc = c->ec.max_ctx, pt = c->ec.page_tokens;
    std::vector<Sample> smp(n);
    for (int i = 0; i < n; ++i) {
        const int64_t P = prompt_offsets[i + 1] - prompt_offsets[i];
        if (P < 1 || max_new[i] < 1 || P + max_new[i] > mc)
            return c->fail(RLHF_EINVAL, "rlhf_submit: sample %d has prompt %lld, max_new %d (need >= 1, sum <= max_ctx %d)",
                           i, (long long)P, max_new[i], mc);
        Sample& s = smp[i];
        s.P = (int)P;
        s.max_new = max_new[i];
        s.target = max_new[i];
        if (forced_len) {
            if (forced_len[i] < 1 || forced_len[i] > max_new[i])
                return c->fail(RLHF_EINVAL, "rlhf_submit: forced_len[%d] = %d outside [1, max_new]", i, forced_len[i]);
            s.target = forced_len[i];
            s.has_forced_len = true;
        }
        s.reserve = ceil_div(s.P + s.max_new, pt);
        if (s.reserve > c->pool_pages)
            return c->fail(RLHF_ENOMEM, "rlhf_submit: sample %d reserves %d pages, the pool has %d", i, s.reserve, c->pool_pages);
        for (int64_t k = prompt_offsets[i]; k < prompt_offsets[i + 1]; ++k)
            if (prompt_tokens[k] < 0 || prompt_tokens[k] >= c->mc.vocab)
                return c->fail(RLHF_EINVAL, "rlhf_submit: token %d of sample %d out of range", prompt_tokens[k], i);
        if (forced_tokens) {
            const int64_t fl = forced_offsets[i + 1] - forced_offsets[i];
            if (fl < 0 || fl > s.max_new) return c->fail(RLHF_EINVAL, "rlhf_submit: forced_offsets of sample %d", i);
            for (int64_t k = forced_offsets[i]; k < forced_offsets[i + 1]; ++k)
                if (forced_tokens[k] >= c->mc.vocab) return c->fail(RLHF_EINVAL, "rlhf_submit: forced token out of range");
        }
    }
    int rc = rlhf_sync(c);
    if (rc) return rc;

    c->N = n;
    c->smp.swap(smp);
    c->h_prompt.assign(prompt_tokens, prompt_tokens + (n ? prompt_offsets[n] : 0));
    c->h_prompt_off.assign(prompt_offsets, prompt_offsets + (n ? n + 1 : 0));
    c->h_forced.assign((size_t)n * mc, -1);
    std::vector<int> tok((size_t)n * mc, 0);
    for (int i = 0; i < n; ++i) {
        Sample& s = c->smp[i];
        std::copy(prompt_tokens + prompt_offsets[i], prompt_tokens + prompt_offsets[i + 1], tok.begin() + (size_t)i * mc);
        if (forced_tokens)
            for (int64_t k = forced_offsets[i]; k < forced_offsets[i + 1]; ++k)
                c->h_forced[(size_t)i * mc + (k - forced_offsets[i])] = forced_tokens[k] < 0 ? -1 : forced_tokens[k];
        if (s.has_forced_len) c->h_forced[(size_t)i * mc + s.target - 1] = c->ec.eos_id;
    }
    if (n) HIPCK(c, hipMemcpy(c->d_tokens, tok.data(), tok.size() * sizeof(int), hipMemcpyHostToDevice));
    // results of roles that are never scored read back as NaN (all-ones bit pattern), not as
    // leftovers of an earlier stage
    for (float* r : {c->d_lp_actor, c->d_lp_rescored, c->d_lp_ref, c->d_values})
        HIPCK(c, hipMemset(r, 0xFF, (size_t)c->ec.max_samples * mc * 4));
    HIPCK(c, hipMemset(c->d_reward, 0xFF, (size_t)c->ec.max_samples * 4));
    HIPCK(c, hipMemset(c->d_nonfinite, 0, sizeof(int)));
    c->waiting.clear();
    for (int i = 0; i < n; ++i) c->waiting.push_back(i);
    c->active.clear();
    c->free_list.resize(c->pool_pages);
    for (int p = 0; p < c->pool_pages; ++p) c->free_list[p] = c->pool_pages - 1 - p;   // pop_back issues 0, 1, 2, ...
    c->reserved = 0;
    c->retired.clear();
    c->n_scored = 0;
    c->batch_offsets.assign(1, 0);
    c->batch_step.clear();
    c->step = 0;
    c->score_used = false;
    c->acc_weight_bytes = c->acc_kv_bytes = c->acc_prefill_tokens = 0;
    return RLHF_OK;
}

// ============================================================================ generate step

namespace {

int take_page(rlhf_ctx* c, Sample& s) {
    const int pg = c->free_list.back();
    c->free_list.pop_back();
    s.pages.push_back(pg);
    return pg;
}

// Imposed token at output index j (1-based) of sample i, or -1.
int forced_at(const rlhf_ctx* c, int i, int j) { return c->h_forced[(size_t)i * c->ec.max_ctx + (j - 1)]; }

// Head over selected rows of a batch pass: logits in row chunks, then pick / gather.
struct HeadPlan {
    int n_sel = 0;
    const int* sel_rows = nullptr;     // device: rows of the pass whose hidden state feeds the head
    // pick (prefill): per selected row
    const int* forced = nullptr;
    const int* tok_dst = nullptr;
    const int* lp_dst = nullptr;
    // gather (scoring log-probs): per selected row
    const int* target_idx = nullptr;
    const int* out_dst = nullptr;
    float* out = nullptr;
};

int lm_head_chunks(rlhf_ctx* c, hipStream_t st, Workspace& ws, const rlhf_weights& w, const HeadPlan& hp,
                   bool pick) {
    const rlhf_model_cfg& m = c->mc;
    const int d = m.d_model, V = m.vocab;
    for (int r0 = 0; r0 < hp.n_sel; r0 += ws.logit_rows) {
        const int nr = std::min(ws.logit_rows, hp.n_sel - r0);
        const char* x = (const char*)ws.xsel + (size_t)r0 * d * c->esz;
        if (gemm_stream_supported(c->dtype, act_type(c, true), nr, d) && (c->dtype != kF32 || head_in_groups(nr, V, d, false))) {
            const double bytes = ((double)V * d + (double)nr * d) * c->esz + (double)nr * V * 4;
            HIPCK(c, profiled(c, st, kGemmBatch, bytes, 2.0 * nr * V * d, [&] {
                return launch_gemm_stream(st, c->dtype, act_type(c, true), 0, x, w.head, ws.logits, nr, V, d, RowsEpi{});
            }));
        } else {
            HIPCK(c, gemm_profiled(c, st, kGemmBatch, act_type(c, true), x, w.head, ws.logits, nr, V, d, 1));
        }
        if (pick)
            HIPCK(c, launch_pick(st, ws.logits, 1, 0, nr, V, hp.forced + r0, c->d_tokens, hp.tok_dst + r0,
                                 c->d_lp_actor, hp.lp_dst + r0, nullptr, ws.pick_scratch, c->d_nonfinite));
        else
            HIPCK(c, launch_gather_lp(st, ws.logits, 1, 0, nr, V, c->d_tokens, hp.target_idx + r0, hp.out,
                                      hp.out_dst + r0, c->d_nonfinite));
    }
    return RLHF_OK;
}

// LM head of a scoring pass with the log-softmax gather fused into the GEMM's epilogue: the
// [rows, vocab] logits never reach memory, only 2 * ceil(vocab / 256) (max, sum exp) pairs and the
// target logit per row, which a merge kernel turns into log-probs.  The partials live in the
// workspace's logits buffer.
int lm_head_logprob_fused(rlhf_ctx* c, hipStream_t st, Workspace& ws, const RoleWeights& rw, const HeadPlan& hp) {
    const bool hw = rw.h16.head != nullptr && act_type(c, true) == kF16;
    const void* head = hw ? rw.h16.head : rw.w.head;
    const int wdt = hw ? kF16 : c->dtype;
    const rlhf_model_cfg& m = c->mc;
    const int d = m.d_model, V = m.vocab, adt = act_type(c, true);
    const int n_part = gemm_lse_partials(V);
    const size_t per_row = (size_t)2 * n_part + 1;
    const size_t cap_rows = (size_t)ws.logit_rows * V / per_row;
    if (cap_rows < 1) return c->fail(RLHF_EINVAL, "internal: no room for the LM head's partials");
    for (int r0 = 0; r0 < hp.n_sel; r0 += (int)std::min<size_t>(cap_rows, 1 << 30)) {
        const int nr = (int)std::min<size_t>(cap_rows, (size_t)(hp.n_sel - r0));
        LseOut lo;
        lo.tokens = c->d_tokens;
        lo.target_idx = hp.target_idx + r0;
        lo.part_max = ws.logits;
        lo.part_sum = ws.logits + (size_t)nr * n_part;
        lo.tgt = ws.logits + (size_t)2 * nr * n_part;
        lo.n_part = n_part;
        const char* x = (const char*)ws.xsel + (size_t)r0 * d * c->esz;
        const double bytes = ((double)V * d + (double)nr * d) * c->esz + (double)nr * per_row * 4;
        HIPCK(c, profiled(c, st, kGemmBatch, bytes, 2.0 * nr * V * d,
                          [&] { return launch_gemm_lse(st, wdt, adt, x, head, nr, V, d, lo); }));
        HIPCK(c, launch_lse_merge(st, lo.part_max, lo.part_sum, lo.tgt, n_part, nr, hp.out, hp.out_dst + r0,
                                  c->d_nonfinite));
    }
    return RLHF_OK;
}

// Query tiles of the MFMA attention for sequences of the given lengths packed back to back:
// writes tile_start / tile_q0 / tile_len (n each) at dst, dst + n, dst + 2n; returns n.
int count_tiles(const std::vector<int>& lens) {
    int n = 0;
    for (int L : lens) n += ceil_div(L, kFlashTile);
    return n;
}
void fill_tiles(const std::vector<int>& lens, int* dst) {
    const int n = count_tiles(lens);
    int t = 0, start = 0;
    for (int L : lens) {
        for (int q0 = 0; q0 < L; q0 += kFlashTile, ++t) {
            dst[t] = start;
            dst[n + t] = q0;
            dst[2 * n + t] = L;
        }
        start += L;
    }
}

// Algorithmic cost of one layer's packed causal attention over sequences of the given lengths.
void batch_attn_cost(const rlhf_ctx* c, const std::vector<int>& lens, int T, PassMeta* pm) {
    const double qd = (double)c->mc.n_q_heads * c->mc.head_dim, kvd = (double)c->mc.n_kv_heads * c->mc.head_dim;
    double pairs = 0;
    for (int L : lens) {
        const double t = L;
        pairs += t * (t + 1) / 2;
    }
    pm->attn_flops = 4.0 * qd * pairs;
    pm->attn_bytes = (double)T * (2 * qd + 2 * kvd) * c->esz;
}

// Rows a sample needs when it is (re-)admitted: its prompt, plus, after a migration (Section
// 4.2, "Migration mechanism", second choice: only the tokens travel and the KV cache is
// regenerated by rerunning the prefill), every generated token but the newest, which the same
// step's decode feeds.
int prefill_rows(const Sample& s) { return s.P + std::max(s.gen_len - 1, 0); }

// Prefill of newly admitted samples [group], whose rows total `T` <= max_batch_tokens.  A
// first-time sample gets its first output token from the last prompt row; a migrated one emits
// nothing.
int prefill_group(rlhf_ctx* c, const std::vector<int>& group, int T) {
    const int mc = c->ec.max_ctx, pt = c->ec.page_tokens, n = (int)group.size();
    int* hm;
    HIPCK(c, c->meta_pre.begin(&hm));
    // layout: tok_idx[T] pos[T] kv_dst[T] | sel[n] forced[n] tok_dst[n] lp_dst[n] | upd_idx[U] upd_val[U]
    int* tok_idx = hm;
    int* pos = hm + T;
    int* kv_dst = hm + 2 * T;
    int* sel = hm + 3 * T;
    int* forced = sel + n;
    int* tok_dst = forced + n;
    int* lp_dst = tok_dst + n;
    int* upd = lp_dst + n;
    std::vector<int> upd_idx, upd_val, lens;
    int row = 0, n_sel = 0;
    for (int gi = 0; gi < n; ++gi) {
        const int i = group[gi];
        Sample& s = c->smp[i];
        const int rows_i = prefill_rows(s);
        lens.push_back(rows_i);
        for (int p = 0; p < rows_i; ++p, ++row) {
            if (p % pt == 0) {
                const int pg = take_page(c, s);
                upd_idx.push_back(i * c->max_pages + p / pt);
                upd_val.push_back(pg);
            }
            tok_idx[row] = i * mc + p;
            pos[row] = p;
            kv_dst[row] = s.pages[p / pt] * pt + p % pt;
        }
        s.ctx = rows_i;
        s.admit_step = c->step;
        if (s.gen_len == 0) {
            s.gen_len = 1;
            sel[n_sel] = row - 1;
            forced[n_sel] = forced_at(c, i, 1);
            tok_dst[n_sel] = i * mc + s.P;
            lp_dst[n_sel] = i * mc + 0;
            ++n_sel;
        }
    }
    const int U = (int)upd_idx.size();
    std::copy(upd_idx.begin(), upd_idx.end(), upd);
    std::copy(upd_val.begin(), upd_val.end(), upd + U);
    const int n_tiles = count_tiles(lens);
    const size_t tiles_off = (size_t)3 * T + 4 * n + 2 * U;
    const size_t n_ints = tiles_off + 3 * (size_t)n_tiles;
    if (n_ints > c->meta_pre.cap) return c->fail(RLHF_EINVAL, "internal: prefill metadata overflow");
    fill_tiles(lens, hm + tiles_off);
    HIPCK(c, c->meta_pre.commit(c->sd, n_ints));
    const int* dm_ = c->meta_pre.dev;
    HIPCK(c, launch_scatter_int(c->sd, c->d_page_table, dm_ + 3 * T + 4 * n, dm_ + 3 * T + 4 * n + U, U));

    PassMeta pm;
    pm.tok_idx = dm_;
    pm.pos = dm_ + T;
    pm.kv_dst = dm_ + 2 * T;
    pm.tile_start = dm_ + tiles_off;
    pm.tile_q0 = dm_ + tiles_off + n_tiles;
    pm.tile_len = dm_ + tiles_off + 2 * n_tiles;
    pm.n_tiles = n_tiles;
    pm.longest = *std::max_element(lens.begin(), lens.end());
    batch_attn_cost(c, lens, T, &pm);
    const rlhf_weights& w = c->roles[RLHF_ACTOR].w;
    Workspace& ws = c->ws_pre;
    int pns;
    size_t pstride;
    int rc = forward_layers(c, c->sd, ws, c->roles[RLHF_ACTOR], T, pm, kModeBatch, 1, &pns, &pstride);
    if (rc) return rc;
    if (n_sel > 0) {
        HIPCK(c, launch_rmsnorm(c->sd, act_type(c, true), ws.h, ws.part, pns, pstride, dm_ + 3 * T, w.g_final, ws.xsel,
                                n_sel, c->mc.d_model, c->mc.rms_eps));
        HeadPlan hp;
        hp.n_sel = n_sel;
        hp.forced = dm_ + 3 * T + n;
        hp.tok_dst = dm_ + 3 * T + 2 * n;
        hp.lp_dst = dm_ + 3 * T + 3 * n;
        rc = lm_head_chunks(c, c->sd, ws, w, hp, true);
        if (rc) return rc;
    }
    c->acc_prefill_tokens += T;
    return RLHF_OK;
}

int decode_rows(rlhf_ctx* c, const std::vector<int>& rows_ids) {
    const int R = (int)rows_ids.size();
    const int mc = c->ec.max_ctx, pt = c->ec.page_tokens;
    int* hm;
    HIPCK(c, c->meta_dec.begin(&hm));
    // layout: tok_idx pos kv_dst row_sample ctx_len tok_dst lp_dst forced (R each) | upd_idx[U] upd_val[U]
    int* a[8];
    for (int k = 0; k < 8; ++k) a[k] = hm + k * R;
    int* upd = hm + 8 * R;
    int U = 0;
    int64_t kv_tokens = 0;
    int max_ctx_len = 0;
    for (int r = 0; r < R; ++r) {
        const int i = rows_ids[r];
        Sample& s = c->smp[i];
        const int p = s.ctx;                 // position being written
        if (p % pt == 0) {
            const int pg = take_page(c, s);
            upd[U] = i * c->max_pages + p / pt;
            upd[R + U] = pg;                 // provisional slot; compacted below
            ++U;
        }
        a[0][r] = i * mc + p;
        a[1][r] = p;
        a[2][r] = s.pages[p / pt] * pt + p % pt;
        a[3][r] = i;
        a[4][r] = p + 1;
        a[5][r] = i * mc + p + 1;
        a[6][r] = i * mc + (p + 1 - s.P);
        a[7][r] = forced_at(c, i, p + 2 - s.P);
        s.ctx = p + 1;
        s.gen_len += 1;
        kv_tokens += p + 2;                  // p+1 keys read, one written
        max_ctx_len = std::max(max_ctx_len, p + 1);
    }
    for (int u = 0; u < U; ++u) upd[U + u] = upd[R + u];
    HIPCK(c, c->meta_dec.commit(c->sd, (size_t)8 * R + 2 * U));
    const int* dmeta = c->meta_dec.dev;
    HIPCK(c, launch_scatter_int(c->sd, c->d_page_table, dmeta + 8 * R, dmeta + 8 * R + U, U));

    PassMeta pm;
    pm.tok_idx = dmeta;
    pm.pos = dmeta + R;
    pm.kv_dst = dmeta + 2 * R;
    pm.row_sample = dmeta + 3 * R;
    pm.ctx_len = dmeta + 4 * R;
    pm.max_pages = ceil_div(max_ctx_len, pt);
    {
        const double kvd_ = (double)c->mc.n_kv_heads * c->mc.head_dim, qd_ = (double)c->mc.n_q_heads * c->mc.head_dim;
        const double keys = (double)(kv_tokens - R);           // sum of visible keys over rows
        pm.attn_bytes = (keys * 2 * kvd_ + 2.0 * R * qd_) * c->esz;
        pm.attn_flops = 4.0 * keys * qd_;
    }
    // split long contexts so that a handful of samples still fills the chip
    Workspace& ws = c->ws_dec;
    const int max_split = (int)std::min<size_t>(32, ws.attn_slots / ((size_t)R * c->mc.n_q_heads));
    const int asplit = decode_attn_nsplit(R, pm.max_pages, c->dm, std::max(1, max_split));

    const rlhf_weights& w = c->roles[RLHF_ACTOR].w;
    const int d = c->mc.d_model, V = c->mc.vocab;
    int ns = 1;
    if (stream_pass(c, R)) {
        int n_ssq, pns;
        int rc = forward_layers_stream(c, c->sd, ws, c->roles[RLHF_ACTOR], R, pm, kModeDecode, asplit, &pns, &n_ssq);
        if (rc) return rc;
        RowsEpi ep;
        const int adt = act_type(c, false);
        if (adt == kF16) ep.a = ActLayout{8, 8 * R};
        const bool many = adt == kF16 && takes_gemm_rows(R, d), hw = many && c->roles[RLHF_ACTOR].h16.head;
        const bool head_stream = adt != kF32 || head_in_groups(R, V, d, true);
        if (R <= kStreamResidRows || (adt == kF32 && head_stream))
            ep.nrm = stream_norm(c, ws, w.g_final, n_ssq, ws.scale, nullptr);
        else
            HIPCK(c, launch_rmsnorm(c->sd, adt, ws.h, ws.part, pns, (size_t)R * d, nullptr, w.g_final, ws.xn, R, d,
                                    c->mc.rms_eps, ep.a));
        if (head_stream) {
            const double bytes = ((double)V * d + (double)R * d) * c->esz + (double)R * V * 4;
            HIPCK(c, profiled(c, c->sd, kGemmDecode, bytes, 2.0 * R * V * d, [&] {
                return launch_gemm_stream(c->sd, hw ? kF16 : c->dtype, adt, 0, ws.xn, hw ? c->roles[RLHF_ACTOR].h16.head : w.head, ws.part, R,
                                          V, d, ep, 1, many);
            }));
        } else {
            ns = nsplit_for(c, ws, R, V, d);
            HIPCK(c, gemm_profiled(c, c->sd, kGemmDecode, adt, ws.xn, w.head, ws.part, R, V, d, ns));
        }
    } else {
        int pns;
        size_t pstride;
        int rc = forward_layers(c, c->sd, ws, c->roles[RLHF_ACTOR], R, pm, kModeDecode, asplit, &pns, &pstride);
        if (rc) return rc;
        HIPCK(c, launch_rmsnorm(c->sd, act_type(c, false), ws.h, ws.part, pns, pstride, nullptr, w.g_final, ws.xsel, R, d,
                                c->mc.rms_eps));
        ns = nsplit_for(c, ws, R, V, d);
        HIPCK(c, gemm_profiled(c, c->sd, kGemmDecode, act_type(c, false), ws.xsel, w.head, ws.part, R, V, d, ns));
    }
    HIPCK(c, launch_pick(c->sd, ws.part, ns, (size_t)R * V, R, V, dmeta + 7 * R, c->d_tokens, dmeta + 5 * R,
                         c->d_lp_actor, dmeta + 6 * R, c->d_picked, ws.pick_scratch, c->d_nonfinite));
    // algorithmic bytes of this step
    const rlhf_model_cfg& m = c->mc;
    const int64_t qd = (int64_t)m.n_q_heads * m.head_dim, kvd = (int64_t)m.n_kv_heads * m.head_dim;
    const int64_t per_layer = (qd + 2 * kvd) * m.d_model + m.d_model * qd + 3LL * m.d_model * m.ffn;
    c->acc_weight_bytes += (m.n_layers * per_layer + (int64_t)m.vocab * m.d_model) * c->esz;
    c->acc_kv_bytes += kv_tokens * 2 * m.n_layers * kvd * c->esz;
    return RLHF_OK;
}

// stop_on_eos: fetch the tokens just picked for `ids` (pick order) and mark finished samples.
int check_eos(rlhf_ctx* c, const std::vector<int>& ids, const int* d_src) {
    if (!c->ec.stop_on_eos || ids.empty()) return RLHF_OK;
    HIPCK(c, hipMemcpyAsync(c->h_picked, d_src, ids.size() * sizeof(int), hipMemcpyDeviceToHost, c->sd));
    HIPCK(c, hipStreamSynchronize(c->sd));
    for (size_t r = 0; r < ids.size(); ++r)
        if (c->h_picked[r] == c->ec.eos_id) c->smp[ids[r]].finished = true;
    return RLHF_OK;
}

bool sample_done(const Sample& s) { return s.finished || s.gen_len >= s.target; }

// The listed active samples give their pages back (each in reverse page-table order), release
// their reservation and leave the active array; the caller puts them back into the queue.
void release_samples(rlhf_ctx* c, const int* ids, int n) {
    std::vector<char> listed(c->smp.size(), 0);
    for (int k = 0; k < n; ++k) {
        Sample& s = c->smp[ids[k]];
        listed[ids[k]] = 1;
        for (auto it = s.pages.rbegin(); it != s.pages.rend(); ++it) c->free_list.push_back(*it);
        s.pages.clear();
        s.ctx = 0;
        c->reserved -= s.reserve;
    }
    std::vector<int> keep;
    for (int i : c->active)
        if (!listed[i]) keep.push_back(i);
    c->active.swap(keep);
}

}  // namespace

extern "C" int rlhf_generate_step(rlhf_ctx* c, rlhf_step_info* out) {
    if (!c) return RLHF_EINVAL;
    if (!c->roles[RLHF_ACTOR].bound) return c->fail(RLHF_ESTATE, "rlhf_generate_step: Actor weights not loaded");
    if (c->waiting.empty() && c->active.empty()) return c->fail(RLHF_ESTATE, "rlhf_generate_step: nothing to generate");
    // admission: FIFO, first misfit blocks the queue.  The test is the reservation at the cap, or,
    // under optimistic admission, the pages needed now plus one spare page per running sample.
    std::vector<int> newcomers;
    int free_now = (int)c->free_list.size();
    while (!c->waiting.empty() && (int)(c->active.size() + newcomers.size()) < c->ec.max_active) {
        const int i = c->waiting.front();
        if (c->ec.optimistic_admission) {
            const int need = ceil_div(prefill_rows(c->smp[i]) + 1, c->ec.page_tokens);
            const int running = (int)(c->active.size() + newcomers.size());
            if (need > free_now || (running > 0 && free_now - need < running)) break;
            free_now -= need;
        } else if (c->reserved + c->smp[i].reserve > c->pool_pages) {
            break;
        }
        c->waiting.pop_front();
        c->reserved += c->smp[i].reserve;
        newcomers.push_back(i);
    }
    int n_prefill = 0;
    // prefill in groups that fit one batch pass
    size_t g0 = 0;
    while (g0 < newcomers.size()) {
        std::vector<int> group;
        int T = 0;
        size_t g1 = g0;
        std::vector<int> fresh;
        while (g1 < newcomers.size() && T + prefill_rows(c->smp[newcomers[g1]]) <= c->ec.max_batch_tokens) {
            T += prefill_rows(c->smp[newcomers[g1]]);
            group.push_back(newcomers[g1]);
            if (c->smp[newcomers[g1]].gen_len == 0) fresh.push_back(newcomers[g1]);
            ++g1;
        }
        int rc = prefill_group(c, group, T);
        if (rc) return rc;
        if (c->ec.stop_on_eos) {
            // picked tokens of a prefill are not in d_picked; read them from the token buffer
            for (int i : fresh) {
                int y;
                HIPCK(c, hipMemcpyAsync(&y, c->d_tokens + (size_t)i * c->ec.max_ctx + c->smp[i].P, sizeof(int),
                                        hipMemcpyDeviceToHost, c->sd));
                HIPCK(c, hipStreamSynchronize(c->sd));
                if (y == c->ec.eos_id) c->smp[i].finished = true;
            }
        }
        n_prefill += T;
        g0 = g1;
    }
    for (int i : newcomers) c->active.push_back(i);
    int n_preempted = 0;
    if (c->ec.optimistic_admission) {
        // the decode below takes a page for every sample that sits on a page boundary: if they are
        // not all there, the most recently admitted unfinished samples give theirs back
        std::vector<int> victims;
        for (;;) {
            int need = 0, last = -1;
            for (int i : c->active)
                if (!sample_done(c->smp[i])) {
                    need += c->smp[i].ctx % c->ec.page_tokens == 0;
                    last = i;
                }
            if (need <= (int)c->free_list.size()) break;
            release_samples(c, &last, 1);
            victims.push_back(last);
        }
        for (int v : victims) c->waiting.push_front(v);   // earliest admitted victim ends up first
        n_preempted = (int)victims.size();
    }
    std::vector<int> rows;
    for (int i : c->active)
        if (!sample_done(c->smp[i])) rows.push_back(i);
    if (!rows.empty()) {
        int rc = decode_rows(c, rows);
        if (rc) return rc;
        rc = check_eos(c, rows, c->d_picked);
        if (rc) return rc;
    }
    if (out) {
        out->step = c->step;
        out->n_admitted = (int)newcomers.size();
        out->n_prefill_tokens = n_prefill;
        out->n_decoded = (int)rows.size();
        out->n_active = (int)c->active.size();
        out->n_preempted = n_preempted;
    }
    c->step += 1;
    return RLHF_OK;
}

extern "C" int rlhf_retire(rlhf_ctx* c, int32_t* retired_ids, int32_t* n_retired) {
    if (!c) return RLHF_EINVAL;
    int n = 0;
    std::vector<int> keep;
    keep.reserve(c->active.size());
    for (int i : c->active) {
        Sample& s = c->smp[i];
        if (sample_done(s)) {
            for (auto it = s.pages.rbegin(); it != s.pages.rend(); ++it) c->free_list.push_back(*it);
            s.pages.clear();
            c->reserved -= s.reserve;
            s.retired = true;
            c->retired.push_back(i);
            if (retired_ids) retired_ids[n] = i;
            ++n;
        } else {
            keep.push_back(i);
        }
    }
    c->active.swap(keep);
    if (n_retired) *n_retired = n;
    return RLHF_OK;
}

extern "C" int rlhf_migrate(rlhf_ctx* c, const int32_t* ids, int32_t n, int32_t to_back) {
    if (!c || n < 0 || (n > 0 && !ids)) return RLHF_EINVAL;
    std::vector<char> listed(c->smp.size(), 0);
    for (int k = 0; k < n; ++k) {
        const int i = ids[k];
        if (i < 0 || i >= (int)c->smp.size()) return c->fail(RLHF_EINVAL, "rlhf_migrate: id %d out of range", i);
        if (listed[i]) return c->fail(RLHF_EINVAL, "rlhf_migrate: id %d listed twice", i);
        listed[i] = 1;
        const bool is_active = std::find(c->active.begin(), c->active.end(), i) != c->active.end();
        if (!is_active || sample_done(c->smp[i]))
            return c->fail(RLHF_EINVAL, "rlhf_migrate: sample %d is not an unfinished active sample", i);
    }
    // work already enqueued on the decode stream that reads these pages runs before whatever is
    // enqueued later and writes them again: stream order is the only ordering needed
    release_samples(c, ids, n);
    if (to_back)
        for (int k = 0; k < n; ++k) c->waiting.push_back(ids[k]);
    else
        for (int k = n - 1; k >= 0; --k) c->waiting.push_front(ids[k]);
    return RLHF_OK;
}

// ================================================================================== scoring

namespace {

// One packed pass over samples ids[lo, hi) (total T rows) for one role.
int score_pass(rlhf_ctx* c, hipStream_t st, MetaRing& meta, Workspace& ws, const int* ids, int n, int T, int role) {
    const int mc = c->ec.max_ctx;
    int* hm;
    HIPCK(c, meta.begin(&hm));
    int n_sel = 0;
    for (int k = 0; k < n; ++k) n_sel += role == RLHF_REWARD ? 1 : c->smp[ids[k]].gen_len;
    // layout: tok_idx[T] pos[T] | sel[n_sel] target_idx[n_sel] out_dst[n_sel]
    int* tok_idx = hm;
    int* pos = hm + T;
    int* sel = hm + 2 * T;
    int* target = sel + n_sel;
    int* out_dst = target + n_sel;
    std::vector<int> lens;
    for (int k = 0; k < n; ++k) lens.push_back(c->smp[ids[k]].P + c->smp[ids[k]].gen_len);
    const int n_tiles = count_tiles(lens);
    const size_t tiles_off = (size_t)2 * T + 3 * n_sel;
    if (tiles_off + 3 * (size_t)n_tiles > meta.cap) return c->fail(RLHF_EINVAL, "internal: scoring metadata overflow");
    fill_tiles(lens, hm + tiles_off);
    int row = 0, si = 0;
    for (int k = 0; k < n; ++k) {
        const int i = ids[k];
        const Sample& s = c->smp[i];
        const int Ti = s.P + s.gen_len, start = row;
        for (int p = 0; p < Ti; ++p, ++row) {
            tok_idx[row] = i * mc + p;
            pos[row] = p;
        }
        if (role == RLHF_REWARD) {
            sel[si] = start + Ti - 1;
            target[si] = 0;
            out_dst[si] = i;
            ++si;
        } else {
            for (int j = 1; j <= s.gen_len; ++j, ++si) {
                sel[si] = start + s.P + j - 2;          // the position that predicts y_j (0-based)
                target[si] = i * mc + s.P + j - 1;      // y_j itself sits one position later
                out_dst[si] = i * mc + j - 1;
            }
        }
    }
    HIPCK(c, meta.commit(st, tiles_off + 3 * (size_t)n_tiles));
    const int* dmeta = meta.dev;
    PassMeta pm;
    pm.tok_idx = dmeta;
    pm.pos = dmeta + T;
    pm.tile_start = dmeta + tiles_off;
    pm.tile_q0 = dmeta + tiles_off + n_tiles;
    pm.tile_len = dmeta + tiles_off + 2 * n_tiles;
    pm.n_tiles = n_tiles;
    pm.longest = *std::max_element(lens.begin(), lens.end());
    batch_attn_cost(c, lens, T, &pm);
    const rlhf_weights& w = c->roles[role].w;
    int pns;
    size_t pstride;
    int rc = forward_layers(c, st, ws, c->roles[role], T, pm, kModeBatch, 1, &pns, &pstride);
    if (rc) return rc;
    const int d = c->mc.d_model;
    // selected rows may exceed the workspace rows only if n_sel > T, which cannot happen
    // The d -> 1 heads read the final-norm row in float (no rounding to the 16-bit activation type
    // in front of a single dot product); the LM head's GEMM takes the activation type.
    const bool scalar_head = role == RLHF_CRITIC || role == RLHF_REWARD;
    const int adt = scalar_head ? kF32 : act_type(c, true);
    HIPCK(c, launch_rmsnorm(st, adt, ws.h, ws.part, pns, pstride, dmeta + 2 * T, w.g_final, ws.xsel, n_sel, d,
                            c->mc.rms_eps));
    if (role == RLHF_CRITIC)
        HIPCK(c, launch_head_dot(st, adt, c->dtype, ws.xsel, w.head, n_sel, d, c->d_values, dmeta + 2 * T + 2 * n_sel,
                                 c->d_nonfinite));
    else if (role == RLHF_REWARD)
        HIPCK(c, launch_head_dot(st, adt, c->dtype, ws.xsel, w.head, n_sel, d, c->d_reward, dmeta + 2 * T + 2 * n_sel,
                                 c->d_nonfinite));
    else {
        HeadPlan hp;
        hp.n_sel = n_sel;
        hp.target_idx = dmeta + 2 * T + n_sel;
        hp.out_dst = dmeta + 2 * T + 2 * n_sel;
        hp.out = role == RLHF_REF ? c->d_lp_ref : c->d_lp_rescored;
        rc = gemm_lse_supported(c->dtype, adt, d) ? lm_head_logprob_fused(c, st, ws, c->roles[role], hp)
                                                  : lm_head_chunks(c, st, ws, w, hp, false);
        if (rc) return rc;
    }
    return RLHF_OK;
}

int score_ids(rlhf_ctx* c, const int* ids, int n, uint32_t role_mask, bool on_score_stream) {
    if (n <= 0) return RLHF_OK;
    for (int role = 0; role < 4; ++role)
        if ((role_mask & RLHF_ROLE_BIT(role)) && !c->roles[role].bound)
            return c->fail(RLHF_ESTATE, "rlhf_score: role %d has no weights", role);
    for (int k = 0; k < n; ++k) {
        if (ids[k] < 0 || ids[k] >= c->N) return c->fail(RLHF_EINVAL, "rlhf_score: sample id %d out of range", ids[k]);
        if (!sample_done(c->smp[ids[k]]) || c->smp[ids[k]].gen_len < 1)
            return c->fail(RLHF_ESTATE, "rlhf_score: sample %d is still generating", ids[k]);
    }
    if (on_score_stream && c->ss_part) {
        // generation still running: keep to the scoring share of the chip; otherwise take it all
        const bool generating = !c->waiting.empty() || !c->active.empty();
        int rc = switch_stream(c, &c->ss, generating ? c->ss_part : c->ss_full, c->ev_sw_s);
        if (rc) return rc;
    }
    hipStream_t st = on_score_stream ? c->ss : c->sd;
    Workspace& ws = on_score_stream ? c->ws_score : c->ws_pre;
    MetaRing& meta = on_score_stream ? c->meta_score : c->meta_pre;
    if (on_score_stream) {
        // the tokens being scored were written by work already enqueued on the decode stream
        HIPCK(c, hipEventRecord(c->ev_dep, c->sd));
        HIPCK(c, hipStreamWaitEvent(c->ss, c->ev_dep, 0));
        if (!c->score_used) {
            HIPCK(c, hipEventRecord(c->ev_s0, c->ss));
            c->score_used = true;
        }
    }
    // sub-passes bounded by the workspace rows; a sample is never split
    int lo = 0;
    while (lo < n) {
        int hi = lo, T = 0;
        while (hi < n && T + c->smp[ids[hi]].P + c->smp[ids[hi]].gen_len <= c->ec.max_batch_tokens) {
            T += c->smp[ids[hi]].P + c->smp[ids[hi]].gen_len;
            ++hi;
        }
        for (int role = 0; role < 4; ++role)
            if (role_mask & RLHF_ROLE_BIT(role)) {
                int rc = score_pass(c, st, meta, ws, ids + lo, hi - lo, T, role);
                if (rc) return rc;
            }
        lo = hi;
    }
    if (on_score_stream) HIPCK(c, hipEventRecord(c->ev_score_last, c->ss));
    return RLHF_OK;
}

// Cut the un-scored part of the retired FIFO into batches of <= chunk tokens (at least one sample
// each): a batch closes once the next retired sample would not fit.  Flush the rest when
// generation is over.  Returns the number of batches closed.
int form_batches(rlhf_ctx* c, int chunk_tokens) {
    const long chunk = std::max(1, chunk_tokens);
    const bool done = c->waiting.empty() && c->active.empty();
    int closed = 0;
    for (;;) {
        size_t k = c->n_scored;
        long tok = 0;
        while (k < c->retired.size()) {
            const Sample& s = c->smp[c->retired[k]];
            const long t = s.P + s.gen_len;
            if (k > c->n_scored && tok + t > chunk) break;
            tok += t;
            ++k;
        }
        const bool full = k < c->retired.size();      // the next sample is there and does not fit
        if (k > c->n_scored && (full || done)) {
            c->n_scored = k;
            c->batch_offsets.push_back((int)k);
            c->batch_step.push_back(c->step - 1);
            ++closed;
        } else {
            break;
        }
    }
    return closed;
}

}  // namespace

extern "C" int rlhf_score(rlhf_ctx* c, int32_t n, const int32_t* sample_ids, uint32_t role_mask,
                          int32_t on_score_stream) {
    if (!c) return RLHF_EINVAL;
    if (n < 0 || (n > 0 && !sample_ids)) return c->fail(RLHF_EINVAL, "rlhf_score: bad arguments");
    if (role_mask & ~0xFu) return c->fail(RLHF_EINVAL, "rlhf_score: unknown role bits");
    return score_ids(c, sample_ids, n, role_mask, on_score_stream != 0);
}

// ================================================================================ run stage

namespace {
// Whether the serial plan is the faster one for the submitted samples.  Scoring passes gain by running beside
// decode steps whatever bounds these, as soon as there is more than one pass of them: with passes of 8192 tokens,
// serial / fused time 1.03-1.12 for the 2-layer float model from 9.7 k prompt + response tokens on, 1.01-1.05 for
// d_model 512 to 1536 from 11 k, 1.03 at 2048 and 3072, 1.02 at 4096, 1.01 at 5120 and 8192.  With one pass nothing
// runs beside anything and the second stream only adds its events: 0.96 and 0.98 for the float model (0.6 k and
// 5 k tokens), 0.995-0.998 for d_model 512 to 2048 (6-9.5 k), 0.999 at 4096 (smaller passes may overlap there).
// So: few tokens, and a decode step whose chain of dependent kernels (five a layer where the few-row kernels
// finish the residual stream, else seven; at least ~4 us each) takes longer than streaming its weights at ~5 TB/s.
bool serial_is_faster(const rlhf_ctx* c) {
    int64_t tokens = 0;
    for (const Sample& s : c->smp) tokens += s.P + s.target;
    if (tokens >= 10000) return false;
    const rlhf_model_cfg& m = c->mc;
    const double qd = (double)m.n_q_heads * m.head_dim, kvd = (double)m.n_kv_heads * m.head_dim;
    const double per_layer = (qd + 2 * kvd) * m.d_model + m.d_model * qd + 3.0 * m.d_model * m.ffn;
    const double stream_us = (m.n_layers * per_layer + (double)m.vocab * m.d_model) * c->esz / 5.0e6;
    const int rows = std::min(c->N, c->ec.max_active);
    const int launches = stream_resid(c->dtype, rows, m.d_model) && (c->dtype != kF32 || stream_pass(c, rows)) ? 5 : 7;
    return stream_us < (launches * m.n_layers + 6) * 4.0;
}
}  // namespace

extern "C" int rlhf_run_stage(rlhf_ctx* c, const rlhf_stage_opts* opts, rlhf_stage_stats* out) {
    if (!c) return RLHF_EINVAL;
    if (!opts) return c->fail(RLHF_EINVAL, "rlhf_run_stage: NULL options");
    if (opts->fused < 0 || opts->fused > 2) return c->fail(RLHF_EINVAL, "rlhf_run_stage: fused must be 0, 1 or 2");
    rlhf_stage_opts resolved = *opts;
    if (resolved.fused == 2) resolved.fused = serial_is_faster(c) ? 0 : 1;
    const rlhf_stage_opts* o = &resolved;
    if (c->step != 0 || !c->retired.empty()) return c->fail(RLHF_ESTATE, "rlhf_run_stage: call rlhf_submit first");
    if (o->role_mask & ~0xFu) return c->fail(RLHF_EINVAL, "rlhf_run_stage: unknown role bits");
    const bool timing = o->trace_step_ms && o->trace_cap > 0;
    int rc = rlhf_sync(c);
    if (rc) return rc;
    const auto t0 = std::chrono::steady_clock::now();
    HIPCK(c, hipEventRecord(c->ev_d0, c->sd));
    const size_t first_batch = c->batch_step.size();
    int n_steps = 0;
    auto run_new_batches = [&](int closed) -> int {
        const size_t nb = c->batch_step.size();
        for (size_t b = nb - closed; b < nb; ++b) {
            const int lo = c->batch_offsets[b], hi = c->batch_offsets[b + 1];
            int r = score_ids(c, c->retired.data() + lo, hi - lo, o->role_mask, o->fused != 0);
            if (r) return r;
        }
        return RLHF_OK;
    };
    while (!c->waiting.empty() || !c->active.empty()) {
        if (c->sd_part) {
            // share the chip only while scoring work is actually in flight
            const bool scoring = c->score_used && hipEventQuery(c->ev_score_last) == hipErrorNotReady;
            rc = switch_stream(c, &c->sd, scoring ? c->sd_part : c->sd_full, c->ev_sw_d);
            if (rc) return rc;
        }
        if (timing && n_steps < o->trace_cap) {
            while ((int)c->step_events.size() < 2 * (n_steps + 1)) {
                hipEvent_t e;
                HIPCK(c, hipEventCreate(&e));
                c->step_events.push_back(e);
            }
            HIPCK(c, hipEventRecord(c->step_events[2 * n_steps], c->sd));
        }
        rlhf_step_info info;
        const int64_t bytes_before = c->acc_weight_bytes + c->acc_kv_bytes;
        rc = rlhf_generate_step(c, &info);
        if (rc) return rc;
        if (timing && n_steps < o->trace_cap) HIPCK(c, hipEventRecord(c->step_events[2 * n_steps + 1], c->sd));
        int nret;
        rc = rlhf_retire(c, nullptr, &nret);
        if (rc) return rc;
        if (n_steps < o->trace_cap) {
            if (o->trace_active) o->trace_active[n_steps] = (int)c->active.size();
            if (o->trace_decoded) o->trace_decoded[n_steps] = info.n_decoded;
            if (o->trace_prefill_tokens) o->trace_prefill_tokens[n_steps] = info.n_prefill_tokens;
            if (o->trace_step_bytes)
                o->trace_step_bytes[n_steps] = c->acc_weight_bytes + c->acc_kv_bytes - bytes_before;
        }
        ++n_steps;
        const int remaining = (int)(c->waiting.size() + c->active.size());
        if (o->fused && remaining > 0 && remaining < o->R_t) {
            rc = run_new_batches(form_batches(c, o->score_chunk_tokens));
            if (rc) return rc;
        }
    }
    HIPCK(c, hipEventRecord(c->ev_d1, c->sd));
    if ((rc = switch_stream(c, &c->sd, c->sd_full, c->ev_sw_d))) return rc;
    rc = run_new_batches(form_batches(c, o->score_chunk_tokens));   // generation is over: flush
    if (rc) return rc;
    if (c->score_used) HIPCK(c, hipEventRecord(c->ev_s1, c->ss));
    else HIPCK(c, hipEventRecord(c->ev_d1, c->sd));                  // serial scoring ran on the decode stream
    if ((rc = switch_stream(c, &c->ss, c->ss_full, c->ev_sw_s))) return rc;
    rc = rlhf_sync(c);
    if (rc) return rc;
    const auto t1 = std::chrono::steady_clock::now();
    if (c->prof.on) HIPCK(c, profiler_fold(c->prof));
    if (timing)
        for (int s = 0; s < std::min(n_steps, o->trace_cap); ++s)
            HIPCK(c, hipEventElapsedTime(&o->trace_step_ms[s], c->step_events[2 * s], c->step_events[2 * s + 1]));
    if (out) {
        memset(out, 0, sizeof *out);
        out->n_steps = n_steps;
        out->n_batches = (int)(c->batch_step.size() - first_batch);
        for (const Sample& s : c->smp) {
            out->generated_tokens += s.gen_len;
            out->scored_tokens += s.P + s.gen_len;
        }
        out->prefill_tokens = c->acc_prefill_tokens;
        out->wall_ms = std::chrono::duration<double, std::milli>(t1 - t0).count();
        float ms = 0.f;
        HIPCK(c, hipEventElapsedTime(&ms, c->ev_d0, c->ev_d1));
        out->decode_stream_ms = ms;
        if (c->score_used) {
            HIPCK(c, hipEventElapsedTime(&ms, c->ev_s0, c->ev_s1));
            out->score_stream_ms = ms;
        }
        out->decode_weight_bytes = c->acc_weight_bytes;
        out->decode_kv_bytes = c->acc_kv_bytes;
        out->fused_used = o->fused;
    }
    return RLHF_OK;
}

// ======================================================================== results / snapshot

namespace {
// Rows of the samples i0 .. *i1 - 1 at the head of the staging area: as many as leave room for n_arrays
// packed arrays and n_scalars words behind them (one sample always fits).  *words: packed entries.
void stage_rows(rlhf_ctx* c, int i0, int n_arrays, size_t n_scalars, int* i1, int64_t* words) {
    PackRow* rows = (PackRow*)c->h_stage;
    int i = i0;
    int64_t w = 0;
    for (; i < c->N; ++i) {
        const Sample& s = c->smp[i];
        const size_t need = 4 * (size_t)(i - i0 + 1) + n_scalars + (size_t)n_arrays * (w + s.gen_len);
        if (i > i0 && need > c->stage_words) break;
        rows[i - i0] = PackRow{i, s.P, s.gen_len, (int)w};
        w += s.gen_len;
    }
    *i1 = i;
    *words = w;
}
}  // namespace

extern "C" int rlhf_get_results(rlhf_ctx* c, rlhf_results* out) {
    if (!c) return RLHF_EINVAL;
    if (!out) return c->fail(RLHF_EINVAL, "rlhf_get_results: NULL");
    int rc = rlhf_sync(c);
    if (rc) return rc;
    const int n = c->N, mc = c->ec.max_ctx;
    int64_t total = 0;
    for (int i = 0; i < n; ++i) total += c->smp[i].gen_len;
    const bool packed = out->tokens || out->lp_actor || out->lp_actor_rescored || out->lp_ref || out->values;
    if (packed && out->packed_capacity < total)
        return c->fail(RLHF_EINVAL, "rlhf_get_results: packed_capacity %lld < %lld", (long long)out->packed_capacity, (long long)total);
    if (out->gen_len)
        for (int i = 0; i < n; ++i) out->gen_len[i] = c->smp[i].gen_len;
    if (out->resp_offsets) {
        out->resp_offsets[0] = 0;
        for (int i = 0; i < n; ++i) out->resp_offsets[i + 1] = out->resp_offsets[i] + c->smp[i].gen_len;
    }
    // packed on the device into the pinned staging area, as many samples at a time as fit it
    struct Array { const void* src; void* dst; int after_prompt; };
    std::vector<Array> arrays;
    for (const Array& x : {Array{c->d_tokens, out->tokens, 1}, Array{c->d_lp_actor, out->lp_actor, 0},
                           Array{c->d_lp_rescored, out->lp_actor_rescored, 0}, Array{c->d_lp_ref, out->lp_ref, 0},
                           Array{c->d_values, out->values, 0}})
        if (x.dst) arrays.push_back(x);
    int bad = 0;
    int64_t done = 0;
    for (int i0 = 0, first = 1; i0 < n || first; first = 0) {
        int i1;
        int64_t words;
        const size_t n_scalars = first ? (size_t)n + 1 : 0;
        stage_rows(c, i0, (int)arrays.size(), n_scalars, &i1, &words);
        PackArgs pa;
        pa.n_arrays = (int)arrays.size();
        pa.n = i1 - i0;
        pa.stride = mc;
        pa.total = (int)words;
        pa.rows = (const PackRow*)c->h_stage;
        uint32_t* body = c->h_stage + 4 * (size_t)(i1 - i0);
        if (first) {
            pa.scalars = body;
            pa.reward = (const uint32_t*)c->d_reward;
            pa.flag = c->d_nonfinite;
            pa.n_reward = n;
        }
        pa.out = body + n_scalars;
        for (size_t k = 0; k < arrays.size(); ++k) {
            pa.src[k] = (const uint32_t*)arrays[k].src;
            pa.after_prompt[k] = arrays[k].after_prompt;
        }
        HIPCK(c, launch_pack_results(c->sd, pa));
        HIPCK(c, hipStreamSynchronize(c->sd));
        if (first) {
            if (out->reward && n) memcpy(out->reward, body, (size_t)n * 4);
            bad = (int)body[n];
        }
        for (size_t k = 0; k < arrays.size(); ++k)
            memcpy((uint32_t*)arrays[k].dst + done, pa.out + k * (size_t)words, (size_t)words * 4);
        done += words;
        i0 = i1;
    }
    // The 16-bit activation path has no scaling: a model whose activations leave IEEE half's range
    // (|x| > 65504) produces infinities and then NaNs.  Every kernel that writes a result raises
    // this flag when the value is not finite; the outputs above are still delivered.
    if (bad)
        return c->fail(RLHF_ENONFINITE, "rlhf_get_results: a log-prob, value or reward of this stage is not finite "
                                        "(activations outside the range of the 16-bit path?)");
    return RLHF_OK;
}

extern "C" int rlhf_debug_snapshot(rlhf_ctx* c, rlhf_snapshot* o) {
    if (!c) return RLHF_EINVAL;
    if (!o) return c->fail(RLHF_EINVAL, "rlhf_debug_snapshot: NULL");
    const int n = c->N;
    o->step = c->step;
    o->n_samples = n;
    o->n_waiting = (int)c->waiting.size();
    o->n_active = (int)c->active.size();
    o->n_retired = (int)c->retired.size();
    o->n_batches = (int)c->batch_step.size();
    o->n_free = (int)c->free_list.size();
    o->reserved_pages = c->reserved;
    o->pool_pages = c->pool_pages;
    o->max_pages = c->max_pages;
    if (o->cap_samples < n || o->cap_max_pages < c->max_pages ||
        (o->free_list && o->cap_pool_pages < c->pool_pages))
        return c->fail(RLHF_EINVAL, "rlhf_debug_snapshot: capacities too small (need %d samples, %d pages/sample, %d pool pages)",
                       n, c->max_pages, c->pool_pages);
    if (o->active) std::copy(c->active.begin(), c->active.end(), o->active);
    for (int i = 0; i < n; ++i) {
        const Sample& s = c->smp[i];
        if (o->ctx) o->ctx[i] = s.ctx;
        if (o->gen_len) o->gen_len[i] = s.gen_len;
        if (o->n_pages) o->n_pages[i] = (int)s.pages.size();
        if (o->page_table) {
            int* row = o->page_table + (size_t)i * o->cap_max_pages;
            std::fill(row, row + o->cap_max_pages, -1);
            std::copy(s.pages.begin(), s.pages.end(), row);
        }
    }
    if (o->free_list) std::copy(c->free_list.begin(), c->free_list.end(), o->free_list);
    if (o->retired) std::copy(c->retired.begin(), c->retired.end(), o->retired);
    if (o->batch_offsets) std::copy(c->batch_offsets.begin(), c->batch_offsets.end(), o->batch_offsets);
    if (o->batch_step) std::copy(c->batch_step.begin(), c->batch_step.end(), o->batch_step);
    return RLHF_OK;
}

// ====================================================================================== GAE

extern "C" int rlhf_compute_gae(rlhf_ctx* c, float gamma, float lam, float kl_coef, float* advantages,
                                float* returns, int64_t packed_capacity) {
    if (!c) return RLHF_EINVAL;
    if (!(gamma >= 0.f && gamma <= 1.f) || !(lam >= 0.f && lam <= 1.f))
        return c->fail(RLHF_EINVAL, "rlhf_compute_gae: gamma and lam must be in [0, 1]");
    int rc = rlhf_sync(c);
    if (rc) return rc;
    const int n = c->N, mc = c->ec.max_ctx;
    int64_t total = 0;
    for (int i = 0; i < n; ++i) {
        const Sample& s = c->smp[i];
        if (!sample_done(s) || s.gen_len < 1) return c->fail(RLHF_ESTATE, "rlhf_compute_gae: sample %d is not finished", i);
        total += s.gen_len;
    }
    if ((advantages || returns) && packed_capacity < total)
        return c->fail(RLHF_EINVAL, "rlhf_compute_gae: packed_capacity %lld < %lld", (long long)packed_capacity, (long long)total);
    GaePowers pw;
    pw.gl = (float)((double)gamma * (double)lam);
    for (int k = 0; k <= 64; ++k) pw.lanes[k] = (float)std::pow((double)gamma * (double)lam, 8.0 * k);
    int64_t done = 0;
    for (int i0 = 0; i0 < n;) {
        int i1;
        int64_t words;
        stage_rows(c, i0, 2, 0, &i1, &words);
        float* body = (float*)(c->h_stage + 4 * (size_t)(i1 - i0));
        HIPCK(c, launch_gae(c->sd, c->d_lp_actor, c->d_lp_ref, c->d_values, c->d_reward, (const PackRow*)c->h_stage, i1 - i0,
                            mc, gamma, kl_coef, pw, advantages ? body : nullptr, returns ? body + words : nullptr));
        HIPCK(c, hipStreamSynchronize(c->sd));
        if (advantages) memcpy(advantages + done, body, (size_t)words * 4);
        if (returns) memcpy(returns + done, body + words, (size_t)words * 4);
        done += words;
        i0 = i1;
    }
    return RLHF_OK;
}

// ================================================================================ profiling

extern "C" int rlhf_profile_begin(rlhf_ctx* c, int32_t sample_every) {
    if (!c) return RLHF_EINVAL;
    if (sample_every < 1) return c->fail(RLHF_EINVAL, "rlhf_profile_begin: sample_every must be >= 1");
    int rc = rlhf_sync(c);
    if (rc) return rc;
    Profiler& p = c->prof;
    p.on = true;
    p.every = sample_every;
    p.n_used = 0;
    for (int k = 0; k < kClassCount; ++k) {
        p.launches[k] = p.sampled[k] = p.dropped[k] = 0;
        p.tot_bytes[k] = p.tot_flops[k] = p.s_ms[k] = p.s_bytes[k] = p.s_flops[k] = 0;
    }
    {   // What a bracket costs beyond the kernels inside it.  A bracket around one empty kernel takes
        // overhead + d, around two of them overhead + 2 d (d = an empty kernel with its dispatch gap), so
        // overhead = 2 t1 - t2, from the medians of 33 brackets of each kind, taken alternately.
        constexpr int kCal = 33;
        hipEvent_t ev[4 * kCal];
        for (hipEvent_t& e : ev) HIPCK(c, hipEventCreate(&e));
        for (int i = 0; i < 2 * kCal; ++i) {
            HIPCK(c, hipEventRecord(ev[2 * i], c->sd));
            HIPCK(c, launch_noop(c->sd));
            if (i & 1) HIPCK(c, launch_noop(c->sd));
            HIPCK(c, hipEventRecord(ev[2 * i + 1], c->sd));
        }
        HIPCK(c, hipStreamSynchronize(c->sd));
        float one[kCal], two[kCal];
        for (int i = 0; i < 2 * kCal; ++i)
            HIPCK(c, hipEventElapsedTime((i & 1) ? &two[i / 2] : &one[i / 2], ev[2 * i], ev[2 * i + 1]));
        std::sort(one, one + kCal);
        std::sort(two, two + kCal);
        p.bracket_overhead_ms = std::max(0.0, 2.0 * one[kCal / 2] - two[kCal / 2]);
        for (hipEvent_t e : ev) (void)hipEventDestroy(e);
    }
    return RLHF_OK;
}

extern "C" int rlhf_profile_end(rlhf_ctx* c, rlhf_kernel_profile* out) {
    if (!c) return RLHF_EINVAL;
    if (!out) return c->fail(RLHF_EINVAL, "rlhf_profile_end: NULL");
    int rc = rlhf_sync(c);
    if (rc) return rc;
    Profiler& p = c->prof;
    p.on = false;
    HIPCK(c, profiler_fold(p));
    for (int k = 0; k < kClassCount; ++k) {
        memset(&out[k], 0, sizeof out[k]);
        out[k].launches = p.launches[k];
        out[k].total_bytes = p.tot_bytes[k];
        out[k].total_flops = p.tot_flops[k];
        out[k].sampled = p.sampled[k];
        out[k].sampled_ms = p.s_ms[k];
        out[k].sampled_bytes = p.s_bytes[k];
        out[k].sampled_flops = p.s_flops[k];
        out[k].dropped = p.dropped[k];
        out[k].bracket_overhead_ms = p.bracket_overhead_ms;
    }
    return RLHF_OK;
}
