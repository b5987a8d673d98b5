// Host-callable launchers of the HIP kernels.  Every launcher validates nothing: the engine
// checks shapes and bounds on the host before it launches (see engine.cpp).  All pointers are
// device pointers.  "nsplit / sstride": a float input that is the sum of nsplit partial
// buffers, partial s at x + s * sstride (split-K GEMM output consumed without a reduce pass).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace rlhf {

// Storage types.  Weights are kF32 or kBF16.  With bf16 weights every activation fed to the
// matrix units and the KV pool are kF16: IEEE half keeps 11 significant bits against bf16's 8,
// and the bf16 weights convert to half exactly on their way into LDS.  (The kernels also accept
// bf16 activations and a bf16 pool; the engine does not use them.)
enum DType { kF32 = 0, kBF16 = 1, kF16 = 2 };

struct Dims {
    int n_layers, d_model, n_q_heads, n_kv_heads, head_dim, ffn, vocab;
    int page_tokens;
};

// Where element (m, k) of a 16-bit activation matrix lies: m * row + (k / 8) * chunk + k % 8.  Row-major
// is {K, 8}.  Between the kernels of a decode step it is {8, 8 M}: the same 16-byte chunk of all rows is
// contiguous, which is how a matrix operand is read (M = 16, 7B gate||up + QKV: 52.5 us against 56.3 with
// row-major activations; M = 64: 76 against 95).  row == 0 stands for row-major.
struct ActLayout { int row = 0, chunk = 8; };
__host__ __device__ inline size_t act_index(const ActLayout& l, int m, int k) {
    return (size_t)m * l.row + (size_t)(k >> 3) * l.chunk + (k & 7);
}

// ---- GEMM: C[s][m][n] = sum over k in split s of A[m][k] * W[n][k];  C float, split stride M*N
// (wdt, adt) in {(kF32,kF32), (kBF16,kBF16), (kBF16,kF16)}
int gemm_choose_nsplit(int wdt, int M, int N, int K, int max_split);
// wdt == kF16 (with adt == kF16, K a multiple of 64): W is a half copy of a bf16 matrix, made with
// launch_bf16_to_half; the 256 x 256 tiling then loads both operands global -> LDS directly.  The
// fused-epilogue launchers below accept it too.  gemm_is_tall: the shapes launch_gemm runs with that tiling.
bool gemm_is_tall(int M, int N, int K, int nsplit);
int gemm_tall_grid(int tiles_m, int tiles_n);                                  // workgroups launched for a tile grid
bool gemm_tall_tile(int bid, int tiles_m, int tiles_n, int* tm, int* tn);      // false: the workgroup has no tile
hipError_t launch_bf16_to_half(hipStream_t st, const void* src, void* dst, size_t n_elements);
// variant 0 = the tiling chosen from M; > 0 forces one (tuning / benchmarks).
hipError_t launch_gemm(hipStream_t st, int wdt, int adt, const void* A, const void* W, float* C,
                       int M, int N, int K, int nsplit, int variant = 0);

// wdt == kF16: the matrix is a half copy of bf16 weights, for half activations.  The entry points promise such calls for
// operands below 4 GiB only; k_gemm_tall itself takes a 64-bit base per tile and needs 256 rows of K below 4 GiB.
inline bool half_weights_ok(int wdt, int adt, int K) { return wdt != kF16 || (adt == kF16 && K % 64 == 0); }
inline bool half_operands_ok(int wdt, long M, long N, long K) { return wdt != kF16 || (M > N ? M : N) * K * 2 < (1L << 32); }

// The compute-bound kernel behind them (gemm_tall.hip), K a multiple of 64.
bool gemm_tall_supported(int wdt, int adt, int K);
hipError_t launch_gemm_tall(hipStream_t st, int wdt, int adt, const void* A, const void* W, float* C, int M, int N, int K,
                            int nsplit);
// h [M, N] += A W^T, N a multiple of 4, half activations
hipError_t launch_gemm_tall_add(hipStream_t st, int wdt, int adt, const void* A, const void* W, float* h, int M, int N, int K);
hipError_t launch_gemm_tall_swiglu(hipStream_t st, int wdt, int adt, const void* A, const void* W, void* act, int M, int ffn,
                                   int K);

// Gate||up projection with SwiGLU fused into the epilogue (tall passes of bf16 models):
// act[m][c] = silu(<A[m], W[c]>) * <A[m], W[ffn + c]>, written as adt [M, ffn].
bool gemm_swiglu_supported(int wdt, int adt, int M, int ffn, int K);
hipError_t launch_gemm_swiglu(hipStream_t st, int wdt, int adt, const void* A, const void* W_gate_up,
                              void* act, int M, int ffn, int K);

// QKV projection of a tall pass with rotary embedding, type conversion and the scatter to q / k / v
// (and to the paged pool, if given) in the epilogue: replaces launch_gemm + launch_rope_kv there.
// Element type of q, k, v, pool = adt.  k, v may be NULL (nothing but the pool wants them).
struct RopeOut {
    const int* pos = nullptr;       // [M] rotary position of each row
    const int* kv_dst = nullptr;    // [M] page * page_tokens + offset (needed with pool)
    const float* table = nullptr;   // [max_pos][head_dim/2][cos, sin]
    void* q = nullptr;              // [M, Hq*hd]
    void* k = nullptr;              // [M, Hkv*hd] or NULL
    void* v = nullptr;
    void* pool = nullptr;           // paged KV pool or NULL
    int layer = 0, n_layers = 0, n_q_heads = 0, n_kv_heads = 0, head_dim = 0, page_tokens = 16;
};
bool gemm_rope_supported(int wdt, int adt, int M, int K, const Dims& dm);
hipError_t launch_gemm_rope(hipStream_t st, int wdt, int adt, const void* A, const void* Wqkv, int M, int K,
                            const RopeOut& ro);

// Few rows (gemm_stream.hip): workgroups walk the whole K range, so that the step that
// consumes the projection rides in its epilogue and needs no launch of its own.
// mode 0: C float [M, N]; mode 1: gate||up with SwiGLU, act [M, ffn] of type adt (N = 2 ffn);
// mode 2: QKV with rotary embedding and the q / k / v / paged-pool scatter (ep.ro as in launch_gemm_rope);
// mode 3: residual: h += result, and the unscaled input of the next norm (ep.res).
// Half activations: 1..kStreamMaxRows rows; bf16 activations: 1..16; K a multiple of 64.  Float weights and
// activations (row-major): 1..kStreamF32Rows rows, K a multiple of 4.
constexpr int kStreamMaxRows = 64;
constexpr int kStreamF32Rows = 448;   // beyond, other kernels are level or ahead at nearly every width
constexpr int kSsqStride = 512; // floats per row of the partial sums of squares (d_model <= 8192, 16 columns each)
struct NormIn {                 // modes 0..2: A holds x = h * gain * s_in; result of row m times (1/rms) / s_in[m]
    const float* ssq = nullptr;     // [M, kSsqStride] partial sums of h^2 (n_ssq used, the others zero), or NULL: A is used as it is
                                    // sign bit set: an x among those columns left half's range
    const float* h = nullptr;       // [M, K] residual stream and
    const float* g = nullptr;       // [K] gain: half models take the norm from these where x will not do
    int n_ssq = 0;
    const float* s_in = nullptr;    // [M]
    float* s_out = nullptr;         // [M] receives the power of two below 1/rms (may be NULL)
    float eps = 0.f;
};
struct ResidOut {               // mode 3
    float* h = nullptr;             // [M, N] residual stream, updated
    const float* g = nullptr;       // [N] gain of the norm that follows
    void* x = nullptr;              // [M, N] in the activation type: h * g * s
    const float* s = nullptr;       // [M] scale that keeps x in half's range (power of two below the row's previous 1/rms)
    float* ssq = nullptr;           // [M, kSsqStride] partial sums of h^2, one per 16 columns (sign as in NormIn)
};
struct RowsEpi {
    ActLayout a, out;          // layout of A; of act (mode 1) or x (mode 3)
    void* act = nullptr;       // mode 1
    int ffn = 0;
    RopeOut ro;                // mode 2
    NormIn nrm;
    ResidOut res;
};
bool gemm_stream_supported(int wdt, int adt, int M, int K);
// Estimated time of a float launch, which reads the matrix once per 16 rows.
double stream_f32_us(int M, int N, int K);
constexpr int kStreamResidRows = 16;
// Whether a pass over a residual stream of d columns runs on mode 3 and NormIn: any up to kStreamResidRows
// rows; half activations of up to 64 partial sums (n_ssq, a column block of 16 each) at any row count here,
// but not into mode 0; float ones always.
bool stream_resid(int wdt, int M, int d);
// Mode 0 may split K into nsplit planes C [nsplit][M][N]; the split for O and down projections otherwise:
int gemm_stream_nsplit(int M, int N, int K, int max_split);
hipError_t launch_gemm_stream(hipStream_t st, int wdt, int adt, int mode, const void* A, const void* W, float* C,
                              int M, int N, int K, const RowsEpi& ep, int nsplit = 1, bool rows = false);
// The same for more rows (gemm_rows.hip; launch_gemm_stream hands over calls with rows set): modes 0..2 without
// norms, up to kRowsMaxRows rows, half activations, bf16 weights or their half copy (wdt == kF16).
constexpr int kRowsMaxRows = 256;
bool gemm_rows_supported(int wdt, int adt, int M, int K);
int gemm_rows_nsplit(int N, int K, int max_split);
// Whether a pass over a residual stream of d columns takes this kernel, with bf16 weights or their half copy alike (the two
// give the same bits; k_gemm_stream, whose waves share K, gives others).  Beyond 64 rows; from 33 on where the stream is
// wide (not stream_resid), but not at 8192 columns.  The four projections of a layer, 40 / 64 rows, weights cold, us, this
// kernel with half copies, with bf16 weights (every compute wave converts them), k_gemm_stream: d = 2048 30, 37, 34 / 33,
// 38, 39; 4096 75, 91, 82 / 81, 93, 94; 5120 113, 131, 122 / 123, 133, 131; 8192 302, 334, 286 / 315, 339, 310.  Up to 32
// rows k_gemm_stream is the faster one.
bool takes_gemm_rows(int M, int d);
hipError_t launch_gemm_rows(hipStream_t st, int wdt, int mode, const void* A, const void* W, float* C, int M, int N, int K,
                            const RowsEpi& ep, int nsplit);

// Many rows of float models (gemm_f32.hip), row-major, modes as in launch_gemm_stream without norms; mode 3: ep.res.h += result.
bool gemm_f32_tall_supported(int N, int K, int mode);
double gemm_f32_tall_us(int M, int N, int K);      // estimated time of a launch
double gemm_f32_us(int M, int N, int K);           // the same, or that of planes and their reading where gemm_choose_nsplit splits K
hipError_t launch_gemm_f32_tall(hipStream_t st, int mode, const float* A, const float* W, float* C, int M, int N, int K,
                                const RowsEpi& ep);

// LM head of a scoring pass fused with the log-softmax gather: the logits stay in registers.  Per
// row m the GEMM leaves n_part = gemm_lse_partials(N) pairs (max, sum of exp(z - max)), one per 128
// columns (a pair whose columns all lie beyond N is (-inf, 0)), and the logit of the row's target
// token tokens[target_idx[m]] in tgt[m]; launch_lse_merge finishes
// out[out_dst[m]] = tgt[m] - log sum_n exp(z[m][n]).
struct LseOut {
    const int* tokens = nullptr;       // token buffer
    const int* target_idx = nullptr;   // [M] index into tokens of each row's target
    float* part_max = nullptr;         // [M, n_part]
    float* part_sum = nullptr;         // [M, n_part]
    float* tgt = nullptr;              // [M]
    int n_part = 0;
};
bool gemm_lse_supported(int wdt, int adt, int K);
int gemm_lse_partials(int N);
hipError_t launch_gemm_lse(hipStream_t st, int wdt, int adt, const void* A, const void* W_head, int M, int N, int K,
                           const LseOut& lo);
hipError_t launch_lse_merge(hipStream_t st, const float* part_max, const float* part_sum, const float* tgt,
                            int n_part, int rows, float* out, const int* out_dst, int* nonfinite = nullptr);

// ---- elementwise / row kernels
hipError_t launch_embed(hipStream_t st, int dtype, const int* tokens, const int* tok_idx,
                        const void* table, float* h, int rows, int d, int vocab);
// The embedding row with the first norm applied, for the few-row projections of gemm_stream.hip: h, and
// x = h * s * g (activation type, layout x_layout), s[r] the power of two below 1/rms, ssq [rows, kSsqStride]: the sum of h^2, then zeros.
hipError_t launch_embed_norm(hipStream_t st, int dtype, const int* tokens, const int* tok_idx, const void* table,
                             float* h, const float* g, void* x, const ActLayout& x_layout, float* s, float* ssq,
                             int rows, int d, int vocab, float eps);
// v = h[src] + sum partials[src];  (row_idx == NULL: src = r and h[src] = v is written back)
// xn[r] = v * rsqrt(mean(v^2) + eps) * g
hipError_t launch_rmsnorm(hipStream_t st, int adt, float* h, const float* part, int nsplit,
                          size_t sstride, const int* row_idx, const float* g, void* xn, int rows,
                          int d, float eps, const ActLayout& xn_layout = ActLayout{});
// Rotary on Q and K heads of qkv rows.  q_out [rows, Hq*hd] and, if non-NULL, k_out/v_out
// [rows, Hkv*hd] have type qdt; if pool != NULL and kv_dst[r] >= 0, K/V of row r also go (as
// type pdt) to token slot kv_dst[r] (= page * page_tokens + offset) of `layer` in the paged pool.
// (qdt, pdt) in {(kF32,kF32), (kBF16,kBF16), (kF16,kF16)}.
hipError_t launch_rope_kv(hipStream_t st, int qdt, int pdt, const float* qkv, int nsplit, size_t sstride,
                          const int* pos, const int* kv_dst, const float* rope_table,
                          void* q_out, void* k_out, void* v_out, void* pool, int layer,
                          int rows, const Dims& dm);
hipError_t launch_swiglu(hipStream_t st, int adt, const float* gu, int nsplit, size_t sstride,
                         void* act, int rows, int ffn);
// Greedy choice per logit row (lowest id on ties), optional imposed token forced[r] >= 0;
// writes the emitted token to tokens[tok_dst[r]] and picked[r], its log-prob to lp[lp_dst[r]].
// nonfinite (here and below, may be NULL): *nonfinite is set to 1 when a written result is not finite.
// scratch: pick_scratch_floats(rows) floats.
hipError_t launch_pick(hipStream_t st, const float* logits, int nsplit, size_t sstride, int rows,
                       int vocab, const int* forced, int* tokens, const int* tok_dst, float* lp,
                       const int* lp_dst, int* picked, float* scratch, int* nonfinite = nullptr);
size_t pick_scratch_floats(int rows);
// lp[out_dst[r]] = log_softmax(logits[r])[tokens[target_idx[r]]]
hipError_t launch_gather_lp(hipStream_t st, const float* logits, int nsplit, size_t sstride,
                            int rows, int vocab, const int* tokens, const int* target_idx,
                            float* out, const int* out_dst, int* nonfinite = nullptr);
// out[out_dst[r]] = <xn[r], w>;  xn of type adt (or float), w of type wdt
hipError_t launch_head_dot(hipStream_t st, int adt, int wdt, const void* xn, const void* w, int rows,
                           int d, float* out, const int* out_dst, int* nonfinite = nullptr);
hipError_t launch_noop(hipStream_t st);   // empty kernel (calibrates event brackets)
// page_table[upd_idx[i]] = upd_val[i]
hipError_t launch_scatter_int(hipStream_t st, int* dst, const int* idx, const int* val, int n);

// ---- results to pinned host memory (pointers the device can write)
struct PackRow { int row, prompt, len, offset; };   // buffer row, prompt length, entries, place in the packed output
struct PackArgs {
    const uint32_t* src[5] = {};      // [max_samples][stride] buffers of 32-bit entries
    int after_prompt[5] = {};         // entries start behind the row's prompt (token buffer)
    int n_arrays = 0, n = 0, stride = 0, total = 0;
    const PackRow* rows = nullptr;    // [n]
    uint32_t* out = nullptr;          // [n_arrays][total]
    uint32_t* scalars = nullptr;      // [n_reward] rewards, then the flag; or NULL
    const uint32_t* reward = nullptr;
    const int* flag = nullptr;
    int n_reward = 0;
};
hipError_t launch_pack_results(hipStream_t st, const PackArgs& a);

// ---- GAE: advantages and returns of n samples (either may be NULL), packed by PackRow::offset
struct GaePowers { float gl, lanes[65]; };          // gamma*lam and its powers 8 * k, k = 0..64
hipError_t launch_gae(hipStream_t st, const float* lp_actor, const float* lp_ref, const float* values,
                      const float* reward, const PackRow* rows, int n, int stride, float gamma, float kl_coef,
                      const GaePowers& pw, float* adv, float* ret);

// ---- attention
// Decode: one query row per active sample against its paged K/V.  q [rows, Hq*hd]; out the same.
// row_sample[r] selects the page-table row; ctx_len[r] keys are visible.  part_* hold split
// partials when nsplit > 1 (sizes rows*Hq*nsplit*(hd or 1)).
// out_layout: row-major by default.  max_pages: pages of the longest context, 0 where the caller does not know.
hipError_t launch_decode_attn(hipStream_t st, int dtype, const void* q, const void* pool,
                              const int* page_table, int pt_stride, const int* row_sample,
                              const int* ctx_len, void* out, float* part_acc, float* part_ml,
                              int rows, int layer, int nsplit, const Dims& dm, const ActLayout& out_layout = ActLayout{},
                              int max_pages = 0);
// Splits of the contexts for a decode step of `rows` rows whose longest context has max_pages pages.
int decode_attn_nsplit(int rows, int max_pages, const Dims& dm, int max_split);
// Prefill / scoring: packed varlen causal attention over contiguous float q [T,Hq*hd], k, v
// [T,Hkv*hd]; out has type odt; row r belongs to the sequence starting at row_start[r] and sits at position
// row_pos[r] in it (sees keys row_start[r] .. row_start[r] + row_pos[r]).
hipError_t launch_prefill_attn(hipStream_t st, int odt, const float* q, const float* k,
                               const float* v, const int* row_start, const int* row_pos,
                               void* out, int rows, const Dims& dm);

// The same on the matrix units for bf16 models: q, k, v, out IEEE half.  The queries are cut
// into tiles of kFlashTile rows that never straddle a sequence: tile i covers rows
// tile_start[i] + tile_q0[i] .. of the sequence that starts at row tile_start[i] and has
// tile_len[i] rows.  T_total = rows of the packed buffers (loads are clamped to it).
constexpr int kFlashTile = 128;
hipError_t launch_flash_attn(hipStream_t st, const void* q, const void* k, const void* v,
                             const int* tile_start, const int* tile_q0, const int* tile_len, void* out,
                             int n_tiles, int T_total, const Dims& dm);

// The same in float; longest: rows of the longest sequence.
hipError_t launch_flash_attn_f32(hipStream_t st, const float* q, const float* k, const float* v, const int* tile_start,
                                 const int* tile_q0, const int* tile_len, float* out, int n_tiles, int longest, const Dims& dm);

size_t pool_page_elems(const Dims& dm);  // elements of one page over all layers

// Error text of a call without a context; rlhf_last_error(NULL) returns it (per thread).
void set_global_error(const char* msg);

}  // namespace rlhf
