// Row-wise and elementwise kernels of the decoder forward: embedding gather, RMSNorm (fused
// with the residual add of split-K partials), rotary + KV-cache append, SwiGLU, the greedy
// pick / log-softmax gather over the vocabulary, and the value / reward head.
// All are HBM-bound; each reads its input once and writes its output once.
#include "common.h"
#include "kernels.h"

namespace rlhf {

size_t pool_page_elems(const Dims& dm) {
    return (size_t)dm.n_layers * 2 * dm.n_kv_heads * dm.page_tokens * dm.head_dim;
}

// ------------------------------------------------------------------------------- embedding
template <typename T>
__global__ __launch_bounds__(256) void k_embed(const int* __restrict__ tokens,
                                               const int* __restrict__ tok_idx,
                                               const T* __restrict__ table, float* __restrict__ h,
                                               int d, int vocab) {
    const int r = blockIdx.x;
    int tok = tokens[tok_idx[r]];
    tok = min(max(tok, 0), vocab - 1);
    const T* src = table + (size_t)tok * d;
    float* dst = h + (size_t)r * d;
    for (int i = threadIdx.x * 8; i < d; i += 256 * 8) {
        float v[8];
        load8<T>(src + i, v);
        store8<float>(dst + i, v);
    }
}

hipError_t launch_embed(hipStream_t st, int dtype, const int* tokens, const int* tok_idx,
                        const void* table, float* h, int rows, int d, int vocab) {
    if (rows <= 0) return hipSuccess;
    if (dtype == kBF16)
        k_embed<bf16_t><<<rows, 256, 0, st>>>(tokens, tok_idx, (const bf16_t*)table, h, d, vocab);
    else
        k_embed<float><<<rows, 256, 0, st>>>(tokens, tok_idx, (const float*)table, h, d, vocab);
    return hipGetLastError();
}

// With the first norm (see gemm_stream.hip): one block per row, the row in registers between the passes.
constexpr int kEmbedIter = 4;
template <typename T, typename TX>
__global__ __launch_bounds__(256) void k_embed_norm(const int* __restrict__ tokens, const int* __restrict__ tok_idx,
                                                    const T* __restrict__ table, float* __restrict__ h,
                                                    const float* __restrict__ g, TX* __restrict__ x, ActLayout xl,
                                                    float* __restrict__ s_out, float* __restrict__ ssq_out, int d,
                                                    int vocab, float eps) {
    __shared__ float red[16];
    const int r = blockIdx.x;
    const int tok = min(max(tokens[tok_idx[r]], 0), vocab - 1);
    const T* src = table + (size_t)tok * d;
    float v[kEmbedIter][8], ss = 0.f;
#pragma unroll
    for (int it = 0; it < kEmbedIter; ++it) {
        const int i = (it * 256 + threadIdx.x) * 8;
        if (i < d) {
            load8<T>(src + i, v[it]);
            store8<float>(h + (size_t)r * d + i, v[it]);
#pragma unroll
            for (int e = 0; e < 8; ++e) ss += v[it][e] * v[it][e];
        }
    }
    const float tot = block_sum(ss, red);
    const float sc = pow2_below(rsqrtf(tot / (float)d + eps));
#pragma unroll
    for (int it = 0; it < kEmbedIter; ++it) {
        const int i = (it * 256 + threadIdx.x) * 8;
        if (i < d) {
            float gg[8];
            load8<float>(g + i, gg);
#pragma unroll
            for (int e = 0; e < 8; ++e) gg[e] *= v[it][e] * sc;
            store8<TX>(x + act_index(xl, r, i), gg);
        }
    }
    for (int i = threadIdx.x; i < kSsqStride; i += 256) ssq_out[(size_t)r * kSsqStride + i] = i == 0 ? tot : 0.f;
    if (threadIdx.x == 0) s_out[r] = sc;
}

hipError_t launch_embed_norm(hipStream_t st, int dtype, const int* tokens, const int* tok_idx, const void* table,
                             float* h, const float* g, void* x, const ActLayout& x_layout, float* s, float* ssq,
                             int rows, int d, int vocab, float eps) {
    if (rows <= 0) return hipSuccess;
    if (d % 8 || d > 256 * 8 * kEmbedIter) return hipErrorInvalidValue;
    ActLayout xl = x_layout;
    if (xl.row == 0) xl = ActLayout{d, 8};
    if (dtype == kBF16)
        k_embed_norm<bf16_t, f16_t><<<rows, 256, 0, st>>>(tokens, tok_idx, (const bf16_t*)table, h, g, (f16_t*)x, xl, s,
                                                          ssq, d, vocab, eps);
    else
        k_embed_norm<float, float><<<rows, 256, 0, st>>>(tokens, tok_idx, (const float*)table, h, g, (float*)x, xl, s, ssq,
                                                        d, vocab, eps);
    return hipGetLastError();
}

// --------------------------------------------------------------------------------- RMSNorm
// One block per output row, one float4 of the row per thread and iteration (up to
// kRmsMaxIter iterations).  The residual add of the split-K partial planes is fused in: all
// planes of a float4 are requested before any is used, so a row costs one memory round trip.
constexpr int kRmsMaxIter = 2;
constexpr int kMaxPlanes = 16;

template <typename T> __device__ __forceinline__ void store4(T* p, float4 v);
template <> __device__ __forceinline__ void store4<float>(float* p, float4 v) {
    *reinterpret_cast<float4*>(p) = v;
}
template <> __device__ __forceinline__ void store4<bf16_t>(bf16_t* p, float4 v) {
    uint2 r;
    r.x = (uint32_t)f32_to_bf16(v.x) | ((uint32_t)f32_to_bf16(v.y) << 16);
    r.y = (uint32_t)f32_to_bf16(v.z) | ((uint32_t)f32_to_bf16(v.w) << 16);
    *reinterpret_cast<uint2*>(p) = r;
}
template <> __device__ __forceinline__ void store4<f16_t>(f16_t* p, float4 v) {
    typedef _Float16 h4 __attribute__((ext_vector_type(4)));
    h4 r = {(f16_t)v.x, (f16_t)v.y, (f16_t)v.z, (f16_t)v.w};
    *reinterpret_cast<h4*>(p) = r;
}

// NS >= 0: exactly NS partial planes, all of them requested back to back (the usual counts are
// instantiated); NS < 0: `nsplit` planes in a loop.  Either way the planes are added in order.
template <typename T, int NS>
__global__ __launch_bounds__(1024) void k_rmsnorm(float* __restrict__ h, const float* __restrict__ part,
                                                  int nsplit, size_t sstride,
                                                  const int* __restrict__ row_idx,
                                                  const float* __restrict__ g, T* __restrict__ xn,
                                                  ActLayout xl, int d, float eps) {
    __shared__ float red[16];
    const int r = blockIdx.x;
    const int src = row_idx ? row_idx[r] : r;
    float* hrow = h + (size_t)src * d;
    float4 v[kRmsMaxIter], gg[kRmsMaxIter];
    float ss = 0.f;
#pragma unroll
    for (int it = 0; it < kRmsMaxIter; ++it) {
        const int i = (it * blockDim.x + threadIdx.x) * 4;
        v[it] = gg[it] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (i < d) {
            const float* pp = part + (size_t)src * d + i;
            float4 a = *reinterpret_cast<const float4*>(hrow + i);
            if constexpr (NS >= 0) {
                float4 p[NS > 0 ? NS : 1];
#pragma unroll
                for (int s = 0; s < NS; ++s) p[s] = *reinterpret_cast<const float4*>(pp + s * sstride);
                gg[it] = *reinterpret_cast<const float4*>(g + i);      // in flight with the planes
#pragma unroll
                for (int s = 0; s < NS; ++s) { a.x += p[s].x; a.y += p[s].y; a.z += p[s].z; a.w += p[s].w; }
            } else {
                gg[it] = *reinterpret_cast<const float4*>(g + i);
                for (int s = 0; s < nsplit; ++s) {
                    const float4 q = *reinterpret_cast<const float4*>(pp + s * sstride);
                    a.x += q.x; a.y += q.y; a.z += q.z; a.w += q.w;
                }
            }
            if (nsplit > 0 && !row_idx) *reinterpret_cast<float4*>(hrow + i) = a;
            v[it] = a;
            ss += a.x * a.x + a.y * a.y + a.z * a.z + a.w * a.w;
        }
    }
    const float tot = block_sum(ss, red);
    const float inv = rsqrtf(tot / (float)d + eps);
#pragma unroll
    for (int it = 0; it < kRmsMaxIter; ++it) {
        const int i = (it * blockDim.x + threadIdx.x) * 4;
        if (i < d)
            store4<T>(xn + act_index(xl, r, i),
                      make_float4(v[it].x * inv * gg[it].x, v[it].y * inv * gg[it].y, v[it].z * inv * gg[it].z,
                                  v[it].w * inv * gg[it].w));
    }
}

template <typename T>
static hipError_t rmsnorm_launch(hipStream_t st, float* h, const float* part, int nsplit, size_t sstride,
                                 const int* row_idx, const float* g, T* xn, const ActLayout& xl, int rows, int threads, int d,
                                 float eps) {
#define RLHF_RMS(NS) k_rmsnorm<T, NS><<<rows, threads, 0, st>>>(h, part, nsplit, sstride, row_idx, g, xn, xl, d, eps)
    switch (nsplit) {
        case 0: RLHF_RMS(0); break;
        case 1: RLHF_RMS(1); break;
        case 2: RLHF_RMS(2); break;
        case 3: RLHF_RMS(3); break;
        case 4: RLHF_RMS(4); break;
        case 5: RLHF_RMS(5); break;
        case 6: RLHF_RMS(6); break;
        case 7: RLHF_RMS(7); break;
        case 8: RLHF_RMS(8); break;
        case 16: RLHF_RMS(16); break;
        default: RLHF_RMS(-1); break;
    }
#undef RLHF_RMS
    return hipGetLastError();
}

hipError_t launch_rmsnorm(hipStream_t st, int adt, float* h, const float* part, int nsplit,
                          size_t sstride, const int* row_idx, const float* g, void* xn, int rows,
                          int d, float eps, const ActLayout& xn_layout) {
    if (rows <= 0) return hipSuccess;
    if (d > 1024 * 4 * kRmsMaxIter || d % 8 || nsplit < 0 || nsplit > kMaxPlanes) return hipErrorInvalidValue;
    ActLayout xl = xn_layout;
    if (xl.row == 0) xl = ActLayout{d, 8};
    const int quads = d / 4;
    const int iters = (quads + 1023) / 1024;
    const int threads = ((quads + iters - 1) / iters + 63) / 64 * 64;
    if (adt == kBF16) return rmsnorm_launch<bf16_t>(st, h, part, nsplit, sstride, row_idx, g, (bf16_t*)xn, xl, rows, threads, d, eps);
    if (adt == kF16) return rmsnorm_launch<f16_t>(st, h, part, nsplit, sstride, row_idx, g, (f16_t*)xn, xl, rows, threads, d, eps);
    return rmsnorm_launch<float>(st, h, part, nsplit, sstride, row_idx, g, (float*)xn, xl, rows, threads, d, eps);
}

// ---------------------------------------------------------------- rotary + KV-cache append
// rope_table: [max_pos][hd/2][2] = (cos, sin) of pos * base^(-2k/hd), computed in double on
// the host.  Pair (k, k + hd/2) is rotated.  One wave per (row, head): the Hq query heads, then
// the Hkv key heads, then the Hkv value heads (copied).  Split-K partials are summed four at a
// time so that their loads are in flight together.
__device__ __forceinline__ float sum_partials(const float* p, int nsplit, size_t sstride) {
    float a0 = p[0], a1 = 0.f, a2 = 0.f, a3 = 0.f;
    int s = 1;
    for (; s + 3 <= nsplit; s += 3) {
        a1 += p[s * sstride];
        a2 += p[(s + 1) * sstride];
        a3 += p[(s + 2) * sstride];
    }
    for (; s < nsplit; ++s) a1 += p[s * sstride];
    return (a0 + a1) + (a2 + a3);
}

template <typename T, typename TP>
__global__ __launch_bounds__(64) void k_rope_kv(const float* __restrict__ qkv, int nsplit,
                                                size_t sstride, const int* __restrict__ pos,
                                                const int* __restrict__ kv_dst,
                                                const float* __restrict__ rope_table,
                                                T* __restrict__ q_out, T* __restrict__ k_out,
                                                T* __restrict__ v_out, TP* __restrict__ pool,
                                                int layer, Dims dm) {
    const int r = blockIdx.x, hh = blockIdx.y;
    const int hd = dm.head_dim, half = hd >> 1;
    const int Hq = dm.n_q_heads, Hkv = dm.n_kv_heads;
    const int qkv_w = (Hq + 2 * Hkv) * hd;
    const float* x = qkv + (size_t)r * qkv_w + (size_t)hh * hd;
    const int slot = (pool && kv_dst) ? kv_dst[r] : -1;
    TP* pbase = nullptr;                       // K block of this layer at this token slot
    if (slot >= 0) {
        const int pt = dm.page_tokens;
        const size_t page = slot / pt, off = slot % pt;
        pbase = pool + (page * dm.n_layers + layer) * 2 * (size_t)Hkv * pt * hd + off * hd;
    }
    const size_t head_stride = (size_t)dm.page_tokens * hd;      // between KV heads inside a page
    if (hh < Hq + Hkv) {
        const float* tab = rope_table + (size_t)pos[r] * hd;
        for (int k = threadIdx.x; k < half; k += 64) {
            const float a = sum_partials(x + k, nsplit, sstride);
            const float b = sum_partials(x + k + half, nsplit, sstride);
            const float c = tab[2 * k], sn = tab[2 * k + 1];
            const float fa = a * c - b * sn, fb = a * sn + b * c;
            if (hh < Hq) {
                T* dst = q_out + ((size_t)r * Hq + hh) * hd;
                dst[k] = from_f32<T>(fa);
                dst[k + half] = from_f32<T>(fb);
            } else {
                const int kh = hh - Hq;
                if (k_out) {
                    T* dst = k_out + ((size_t)r * Hkv + kh) * hd;
                    dst[k] = from_f32<T>(fa);
                    dst[k + half] = from_f32<T>(fb);
                }
                if (pbase) {
                    TP* dst = pbase + kh * head_stride;
                    dst[k] = from_f32<TP>(fa);
                    dst[k + half] = from_f32<TP>(fb);
                }
            }
        }
    } else {
        const int kh = hh - Hq - Hkv;
        for (int e = threadIdx.x; e < hd; e += 64) {
            const float a = sum_partials(x + e, nsplit, sstride);
            if (v_out) v_out[((size_t)r * Hkv + kh) * hd + e] = from_f32<T>(a);
            if (pbase) pbase[(size_t)Hkv * head_stride + kh * head_stride + e] = from_f32<TP>(a);
        }
    }
}

hipError_t launch_rope_kv(hipStream_t st, int qdt, int pdt, const float* qkv, int nsplit,
                          size_t sstride, const int* pos, const int* kv_dst, const float* rope_table,
                          void* q_out, void* k_out, void* v_out, void* pool, int layer, int rows,
                          const Dims& dm) {
    if (rows <= 0) return hipSuccess;
    dim3 grid(rows, dm.n_q_heads + 2 * dm.n_kv_heads);
    if (qdt == kBF16 && pdt == kBF16)
        k_rope_kv<bf16_t, bf16_t><<<grid, 64, 0, st>>>(qkv, nsplit, sstride, pos, kv_dst, rope_table,
                                                       (bf16_t*)q_out, (bf16_t*)k_out, (bf16_t*)v_out,
                                                       (bf16_t*)pool, layer, dm);
    else if (qdt == kF16 && pdt == kF16)
        k_rope_kv<f16_t, f16_t><<<grid, 64, 0, st>>>(qkv, nsplit, sstride, pos, kv_dst, rope_table,
                                                     (f16_t*)q_out, (f16_t*)k_out, (f16_t*)v_out,
                                                     (f16_t*)pool, layer, dm);
    else if (qdt == kF32 && pdt == kF32)
        k_rope_kv<float, float><<<grid, 64, 0, st>>>(qkv, nsplit, sstride, pos, kv_dst, rope_table,
                                                     (float*)q_out, (float*)k_out, (float*)v_out,
                                                     (float*)pool, layer, dm);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------- SwiGLU
// gu rows are [gate (ffn) | up (ffn)]; act = silu(gate) * up.
template <typename T>
__global__ __launch_bounds__(256) void k_swiglu(const float* __restrict__ gu, int nsplit,
                                                size_t sstride, T* __restrict__ act, int rows,
                                                int ffn) {
    const size_t per_row = (size_t)(ffn >> 3);
    const size_t total = (size_t)rows * per_row;
    for (size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x; idx < total;
         idx += (size_t)gridDim.x * 256) {
        const size_t r = idx / per_row;
        const int c = (int)(idx - r * per_row) * 8;
        const float* row = gu + r * (size_t)(2 * ffn);
        float g[8], u[8], o[8];
        load8<float>(row + c, g);
        load8<float>(row + ffn + c, u);
        for (int s = 1; s < nsplit; ++s) {
            float pg[8], pu[8];
            load8<float>(row + s * sstride + c, pg);
            load8<float>(row + s * sstride + ffn + c, pu);
#pragma unroll
            for (int e = 0; e < 8; ++e) { g[e] += pg[e]; u[e] += pu[e]; }
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = g[e] / (1.f + __expf(-g[e])) * u[e];
        store8<T>(act + r * (size_t)ffn + c, o);
    }
}

hipError_t launch_swiglu(hipStream_t st, int adt, const float* gu, int nsplit, size_t sstride,
                         void* act, int rows, int ffn) {
    if (rows <= 0) return hipSuccess;
    if (ffn % 8) return hipErrorInvalidValue;
    const size_t total = (size_t)rows * (ffn / 8);
    const int grid = (int)((total + 255) / 256 < 65536 ? (total + 255) / 256 : 65536);
    if (adt == kBF16)
        k_swiglu<bf16_t><<<grid, 256, 0, st>>>(gu, nsplit, sstride, (bf16_t*)act, rows, ffn);
    else if (adt == kF16)
        k_swiglu<f16_t><<<grid, 256, 0, st>>>(gu, nsplit, sstride, (f16_t*)act, rows, ffn);
    else
        k_swiglu<float><<<grid, 256, 0, st>>>(gu, nsplit, sstride, (float*)act, rows, ffn);
    return hipGetLastError();
}

// ------------------------------------------------------- greedy pick / log-softmax gather
__device__ __forceinline__ float logit_at(const float* row, int nsplit, size_t sstride, int i) {
    float z = row[i];
    for (int s = 1; s < nsplit; ++s) z += row[s * sstride + i];
    return z;
}

// Block-wide (max value, lowest index attaining it) and sum of exp(z - max).
__device__ __forceinline__ void row_softmax_stats(const float* row, int nsplit, size_t sstride,
                                                  int vocab, float& out_max, int& out_arg,
                                                  float& out_sum) {
    __shared__ float s_val[4];
    __shared__ int s_idx[4];
    __shared__ float s_red[16];
    float best = -INFINITY;
    int arg = 0x7FFFFFFF;
    for (int i = threadIdx.x; i < vocab; i += 256) {
        const float z = logit_at(row, nsplit, sstride, i);
        if (z > best) { best = z; arg = i; }   // ascending i: the first maximum is kept
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const float ov = __shfl_xor(best, o, kWave);
        const int oi = __shfl_xor(arg, o, kWave);
        if (ov > best || (ov == best && oi < arg)) { best = ov; arg = oi; }
    }
    if ((threadIdx.x & 63) == 0) { s_val[threadIdx.x >> 6] = best; s_idx[threadIdx.x >> 6] = arg; }
    __syncthreads();
    best = s_val[0]; arg = s_idx[0];
    for (int w = 1; w < 4; ++w)
        if (s_val[w] > best || (s_val[w] == best && s_idx[w] < arg)) { best = s_val[w]; arg = s_idx[w]; }
    float se = 0.f;
    for (int i = threadIdx.x; i < vocab; i += 256)
        se += expf(logit_at(row, nsplit, sstride, i) - best);
    out_sum = block_sum(se, s_red);
    out_max = best;
    out_arg = arg;
}

// Greedy pick of wide or split rows in two stages, so that a handful of rows still spreads over the chip: stage 1,
// one block per (row, column chunk), leaves (max, argmax, sum exp(z - max)) of its chunk;
// stage 2, one wave per row, merges the chunks in ascending order (so the lowest id wins a
// tie), applies an imposed token and writes token and log-prob.
constexpr int kPickChunks = 32;

__global__ __launch_bounds__(256) void k_pick_stage1(const float* __restrict__ logits, int nsplit,
                                                     size_t sstride, int vocab,
                                                     float* __restrict__ scratch) {
    const int r = blockIdx.x, c = blockIdx.y;
    const int per = (vocab + kPickChunks - 1) / kPickChunks;
    const int lo = c * per, n = max(0, min(vocab, lo + per) - lo);
    float mx = -INFINITY, se = 0.f;
    int arg = 0x7FFFFFFF;
    if (n > 0) row_softmax_stats(logits + (size_t)r * vocab + lo, nsplit, sstride, n, mx, arg, se);
    if (threadIdx.x == 0) {
        float* o = scratch + ((size_t)r * kPickChunks + c) * 3;
        o[0] = mx;
        o[1] = __int_as_float(n > 0 ? arg + lo : 0x7FFFFFFF);
        o[2] = se;
    }
}

// The emitted token (the maximum at `arg`, or the imposed one) and its log-prob, by one thread.
__device__ __forceinline__ void pick_finish(const float* row, int nsplit, size_t sstride, int vocab, float best, int arg, float tot, int r,
                                            const int* forced, int* tokens, const int* tok_dst, float* lp, const int* lp_dst,
                                            int* picked, int* nonfinite) {
    int y = arg;
    const int f = forced ? forced[r] : -1;
    if (f >= 0 && f < vocab) y = f;
    if ((unsigned)y >= (unsigned)vocab) y = 0;   // a row of NaNs has no maximum: stay in bounds, the log-prob below flags it
    const float z = logit_at(row, nsplit, sstride, y);
    tokens[tok_dst[r]] = y;
    const float v = z - best - logf(tot);
    lp[lp_dst[r]] = v;
    if (picked) picked[r] = y;
    if (nonfinite && !isfinite(v)) *nonfinite = 1;
}

__global__ __launch_bounds__(64) void k_pick_stage2(const float* __restrict__ logits, int nsplit,
                                                    size_t sstride, int vocab,
                                                    const float* __restrict__ scratch,
                                                    const int* __restrict__ forced,
                                                    int* __restrict__ tokens,
                                                    const int* __restrict__ tok_dst,
                                                    float* __restrict__ lp,
                                                    const int* __restrict__ lp_dst,
                                                    int* __restrict__ picked, int* __restrict__ nonfinite) {
    const int r = blockIdx.x, lane = threadIdx.x;
    const float* sc = scratch + (size_t)r * kPickChunks * 3;
    float mx = -INFINITY, se = 0.f;
    int arg = 0x7FFFFFFF;
    if (lane < kPickChunks) { mx = sc[lane * 3]; arg = __float_as_int(sc[lane * 3 + 1]); se = sc[lane * 3 + 2]; }
    float best = mx;
    int barg = arg;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const float ov = __shfl_xor(best, o, kWave);
        const int oi = __shfl_xor(barg, o, kWave);
        if (ov > best || (ov == best && oi < barg)) { best = ov; barg = oi; }
    }
    const float tot = wave_sum(mx > -INFINITY ? se * expf(mx - best) : 0.f);
    if (lane == 0)
        pick_finish(logits + (size_t)r * vocab, nsplit, sstride, vocab, best, barg, tot, r, forced, tokens, tok_dst, lp, lp_dst, picked,
                    nonfinite);
}

// The same in one kernel, for one plane of up to 32 * 1024 columns: a block of 1024 threads per row, up to 32 logits a
// thread, all requested at once and kept for the second pass (32000 columns, us, two kernels / one: 1 row 9.7 8.8, 64 rows
// 11.5 9.7, 256 rows 25.5 13.0).  512 threads up to 4096 columns, fewer waves to start and to merge (two kernels / 1024 threads /
// 512: 8 rows of 4096 6.3 4.6 3.9, 448 rows 21.3 6.2 4.6).
constexpr int kPickRowMax = 32 * 1024;
template <int IT, int THREADS>
__global__ __launch_bounds__(THREADS) void k_pick_row(const float* __restrict__ logits, int vocab,
                                                              const int* __restrict__ forced, int* __restrict__ tokens,
                                                              const int* __restrict__ tok_dst, float* __restrict__ lp,
                                                              const int* __restrict__ lp_dst, int* __restrict__ picked,
                                                              int* __restrict__ nonfinite) {
    __shared__ float s_val[16], s_red[16];
    __shared__ int s_idx[16];
    const int r = blockIdx.x, t = threadIdx.x;
    const float* row = logits + (size_t)r * vocab;
    float z[IT];
#pragma unroll
    for (int i = 0; i < IT; ++i) z[i] = row[min(t + i * THREADS, vocab - 1)];
    float best = -INFINITY;
    int arg = 0x7FFFFFFF;
#pragma unroll
    for (int i = 0; i < IT; ++i) {
        const int n = t + i * THREADS;
        if (n < vocab && z[i] > best) { best = z[i]; arg = n; }    // ascending: the first maximum is kept
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const float ov = __shfl_xor(best, o, kWave);
        const int oi = __shfl_xor(arg, o, kWave);
        if (ov > best || (ov == best && oi < arg)) { best = ov; arg = oi; }
    }
    if ((t & 63) == 0) { s_val[t >> 6] = best; s_idx[t >> 6] = arg; }
    __syncthreads();
    best = s_val[0]; arg = s_idx[0];
#pragma unroll
    for (int w = 1; w < THREADS / 64; ++w)
        if (s_val[w] > best || (s_val[w] == best && s_idx[w] < arg)) { best = s_val[w]; arg = s_idx[w]; }
    float se = 0.f;
#pragma unroll
    for (int i = 0; i < IT; ++i)
        if (t + i * THREADS < vocab) se += expf(z[i] - best);
    const float tot = block_sum(se, s_red);
    if (t == 0) pick_finish(row, 1, 0, vocab, best, arg, tot, r, forced, tokens, tok_dst, lp, lp_dst, picked, nonfinite);
}

hipError_t launch_pick(hipStream_t st, const float* logits, int nsplit, size_t sstride, int rows,
                       int vocab, const int* forced, int* tokens, const int* tok_dst, float* lp,
                       const int* lp_dst, int* picked, float* scratch, int* nonfinite) {
    if (rows <= 0) return hipSuccess;
    if (nsplit == 1 && vocab <= kPickRowMax) {
#define RLHF_PICK(IT, THREADS) k_pick_row<IT, THREADS><<<rows, THREADS, 0, st>>>(logits, vocab, forced, tokens, tok_dst, lp, lp_dst, picked, nonfinite)
        if (vocab <= 4096) RLHF_PICK(8, 512);
        else if (vocab <= 16384) RLHF_PICK(16, 1024);
        else RLHF_PICK(32, 1024);
#undef RLHF_PICK
        return hipGetLastError();
    }
    k_pick_stage1<<<dim3(rows, kPickChunks), 256, 0, st>>>(logits, nsplit, sstride, vocab, scratch);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    k_pick_stage2<<<rows, 64, 0, st>>>(logits, nsplit, sstride, vocab, scratch, forced, tokens, tok_dst, lp,
                                       lp_dst, picked, nonfinite);
    return hipGetLastError();
}

size_t pick_scratch_floats(int rows) { return (size_t)rows * kPickChunks * 3; }

__global__ __launch_bounds__(256) void k_gather_lp(const float* __restrict__ logits, int nsplit,
                                                   size_t sstride, int vocab,
                                                   const int* __restrict__ tokens,
                                                   const int* __restrict__ target_idx,
                                                   float* __restrict__ out,
                                                   const int* __restrict__ out_dst, int* __restrict__ nonfinite) {
    const int r = blockIdx.x;
    const float* row = logits + (size_t)r * vocab;
    float mx, se;
    int arg;
    row_softmax_stats(row, nsplit, sstride, vocab, mx, arg, se);
    if (threadIdx.x == 0) {
        int y = tokens[target_idx[r]];
        y = min(max(y, 0), vocab - 1);
        const float v = logit_at(row, nsplit, sstride, y) - mx - logf(se);
        out[out_dst[r]] = v;
        if (nonfinite && !isfinite(v)) *nonfinite = 1;
    }
}

hipError_t launch_gather_lp(hipStream_t st, const float* logits, int nsplit, size_t sstride,
                            int rows, int vocab, const int* tokens, const int* target_idx,
                            float* out, const int* out_dst, int* nonfinite) {
    if (rows <= 0) return hipSuccess;
    k_gather_lp<<<rows, 256, 0, st>>>(logits, nsplit, sstride, vocab, tokens, target_idx, out,
                                      out_dst, nonfinite);
    return hipGetLastError();
}

// Merge of the per-128-column (max, sum exp) partials left by the LM-head GEMM of a scoring pass:
// one wave per row; out[out_dst[r]] = tgt[r] - (max + log sum).
__global__ __launch_bounds__(256) void k_lse_merge(const float* __restrict__ part_max,
                                                   const float* __restrict__ part_sum,
                                                   const float* __restrict__ tgt, int n_part, int rows,
                                                   float* __restrict__ out, const int* __restrict__ out_dst,
                                                   int* __restrict__ nonfinite) {
    const int r = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (r >= rows) return;
    const int lane = threadIdx.x & 63;
    const float* pm = part_max + (size_t)r * n_part;
    const float* ps = part_sum + (size_t)r * n_part;
    float mx = -INFINITY;
    for (int i = lane; i < n_part; i += 64) mx = fmaxf(mx, pm[i]);
    mx = wave_max(mx);
    float se = 0.f;
    for (int i = lane; i < n_part; i += 64) {
        const float m = pm[i];
        if (m > -INFINITY) se += ps[i] * __expf(m - mx);
    }
    se = wave_sum(se);
    if (lane == 0) {
        const float v = tgt[r] - mx - logf(se);
        out[out_dst[r]] = v;
        if (nonfinite && !isfinite(v)) *nonfinite = 1;
    }
}

hipError_t launch_lse_merge(hipStream_t st, const float* part_max, const float* part_sum, const float* tgt,
                            int n_part, int rows, float* out, const int* out_dst, int* nonfinite) {
    if (rows <= 0) return hipSuccess;
    k_lse_merge<<<(rows + 3) / 4, 256, 0, st>>>(part_max, part_sum, tgt, n_part, rows, out, out_dst, nonfinite);
    return hipGetLastError();
}

// ------------------------------------------------------------------- value / reward head
// One wave per row: out[out_dst[r]] = <xn[r], w>.
template <typename T, typename TW>
__global__ __launch_bounds__(256) void k_head_dot(const T* __restrict__ xn, const TW* __restrict__ w,
                                                  int rows, int d, float* __restrict__ out,
                                                  const int* __restrict__ out_dst, int* __restrict__ nonfinite) {
    const int r = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (r >= rows) return;
    const int lane = threadIdx.x & 63;
    float acc = 0.f;
    for (int i = lane * 8; i < d; i += 64 * 8) {
        float a[8], b[8];
        load8<T>(xn + (size_t)r * d + i, a);
        load8<TW>(w + i, b);
#pragma unroll
        for (int e = 0; e < 8; ++e) acc += a[e] * b[e];
    }
    acc = wave_sum(acc);
    if (lane == 0) {
        out[out_dst[r]] = acc;
        if (nonfinite && !isfinite(acc)) *nonfinite = 1;
    }
}

hipError_t launch_head_dot(hipStream_t st, int adt, int wdt, const void* xn, const void* w,
                           int rows, int d, float* out, const int* out_dst, int* nonfinite) {
    if (rows <= 0) return hipSuccess;
    const int grid = (rows + 3) / 4;
    if (adt == kBF16 && wdt == kBF16)
        k_head_dot<bf16_t, bf16_t><<<grid, 256, 0, st>>>((const bf16_t*)xn, (const bf16_t*)w, rows, d, out, out_dst, nonfinite);
    else if (adt == kF16 && wdt == kBF16)
        k_head_dot<f16_t, bf16_t><<<grid, 256, 0, st>>>((const f16_t*)xn, (const bf16_t*)w, rows, d, out, out_dst, nonfinite);
    else if (adt == kF32 && wdt == kBF16)
        k_head_dot<float, bf16_t><<<grid, 256, 0, st>>>((const float*)xn, (const bf16_t*)w, rows, d, out, out_dst, nonfinite);
    else if (adt == kF32 && wdt == kF32)
        k_head_dot<float, float><<<grid, 256, 0, st>>>((const float*)xn, (const float*)w, rows, d, out, out_dst, nonfinite);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

// -------------------------------------------------------------------------- small scatter
__global__ void k_scatter_int(int* __restrict__ dst, const int* __restrict__ idx,
                              const int* __restrict__ val, int n) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) dst[idx[i]] = val[i];
}

hipError_t launch_scatter_int(hipStream_t st, int* dst, const int* idx, const int* val, int n) {
    if (n <= 0) return hipSuccess;
    k_scatter_int<<<(n + 255) / 256, 256, 0, st>>>(dst, idx, val, n);
    return hipGetLastError();
}

// An empty kernel: what two events around a launch measure beyond the kernel itself.
__global__ void k_noop() {}
hipError_t launch_noop(hipStream_t st) {
    k_noop<<<1, 64, 0, st>>>();
    return hipGetLastError();
}

// ------------------------------------------------- results on their way to the host
// Ragged rows of the stage's result buffers, packed back to back into pinned host memory: one kernel and
// one wait instead of a copy of the whole padded buffer per array (8 samples: 5 copies of about 12 us each).
__global__ __launch_bounds__(256) void k_pack_results(PackArgs a) {
    const int i = blockIdx.x, k = blockIdx.y;
    if (i == a.n) {                                        // the scalars: rewards, the non-finite flag
        if (k > 0) return;
        for (int j = threadIdx.x; j < a.n_reward; j += 256) a.scalars[j] = a.reward[j];
        if (threadIdx.x == 0) a.scalars[a.n_reward] = (uint32_t)*a.flag;
        return;
    }
    const PackRow r = a.rows[i];
    const uint32_t* src = a.src[k] + (size_t)r.row * a.stride + (a.after_prompt[k] ? r.prompt : 0);
    uint32_t* dst = a.out + (size_t)k * a.total + r.offset;
    for (int t = threadIdx.x; t < r.len; t += 256) dst[t] = src[t];
}

hipError_t launch_pack_results(hipStream_t st, const PackArgs& a) {
    if (a.n_arrays <= 0 && !a.scalars) return hipSuccess;
    k_pack_results<<<dim3(a.n + (a.scalars ? 1 : 0), a.n_arrays > 0 ? a.n_arrays : 1), 256, 0, st>>>(a);
    return hipGetLastError();
}

// ------------------------------------------------- Generalized Advantage Estimation
// The recursion A_t = delta_t + gamma*lam*A_{t+1}, unrolled: A_t = sum over s >= t of (gamma*lam)^(s-t) delta_s,
//   delta_t = r_t + gamma*V_{t+1} - V_t,  V_{L+1} = 0,
//   r_t = -kl_coef*(lp_actor_t - lp_ref_t) + [t == L] * reward
// As a matrix product (D times the triangular matrix of the powers) this is 2 n L^2 flops and an L x L matrix
// for L outputs of 2 flops each; a workgroup per sample evaluates the same sums as a suffix scan instead,
// in tiles of 2048 tokens from the end: a thread sums 8 tokens, six lane exchanges weighted by
// (gamma*lam)^(8 * 2^k) cover a wave, LDS the four waves and the carry between tiles.  What is left is
// latency: 256 samples with up to 2048 tokens take about 25 us, most of it stores to host memory.
constexpr int kGaeE = 8, kGaeTile = 256 * kGaeE;

__global__ __launch_bounds__(256) void k_gae(const float* __restrict__ lp_actor, const float* __restrict__ lp_ref,
                                             const float* __restrict__ values, const float* __restrict__ reward,
                                             const PackRow* __restrict__ rows, int stride, float gamma, float kl_coef,
                                             GaePowers pw, float* __restrict__ adv, float* __restrict__ ret) {
    // token i of a tile sits at i + i / 32: the 8-token stride of the scan then spreads over the banks
    __shared__ float sd[kGaeTile + kGaeTile / 32], sv[kGaeTile + kGaeTile / 32];
    __shared__ float s_tot[4], s_carry;
    const PackRow r = rows[blockIdx.x];
    const int L = r.len, t = threadIdx.x, lane = t & 63, w = t >> 6;
    const size_t base = (size_t)r.row * stride;
    auto at = [](int i) { return i + (i >> 5); };
    if (t == 0) s_carry = 0.f;
    for (int tile = (L - 1) / kGaeTile; tile >= 0; --tile) {
        const int t0 = tile * kGaeTile;
#pragma unroll
        for (int e = 0; e < kGaeE; ++e) {
            const int i = e * 256 + t, k = t0 + i;
            float d = 0.f, v = 0.f;
            if (k < L) {
                v = values[base + k];
                d = -kl_coef * (lp_actor[base + k] - lp_ref[base + k]);
                if (k == L - 1) d += reward[r.row];
                else d += gamma * values[base + k + 1];
                d -= v;
            }
            sd[at(i)] = d;
            sv[at(i)] = v;
        }
        __syncthreads();
        float a = 0.f;
#pragma unroll
        for (int e = kGaeE - 1; e >= 0; --e) a = sd[at(t * kGaeE + e)] + pw.gl * a;
#pragma unroll
        for (int k = 0; k < 6; ++k) {                      // suffix sums over the wave's lanes
            const float x = __shfl_down(a, 1 << k, kWave);
            if (lane + (1 << k) < 64) a += pw.lanes[1 << k] * x;
        }
        if (lane == 0) s_tot[w] = a;
        __syncthreads();
        float c = s_carry;                                 // the advantage right after this wave's tokens
        for (int x = 3; x > w; --x) c = s_tot[x] + pw.lanes[64] * c;
        float x = __shfl_down(a, 1, kWave);
        if (lane == 63) x = 0.f;
        a = x + pw.lanes[63 - lane] * c;
        float o[kGaeE];
#pragma unroll
        for (int e = kGaeE - 1; e >= 0; --e) { a = sd[at(t * kGaeE + e)] + pw.gl * a; o[e] = a; }
        __syncthreads();
#pragma unroll
        for (int e = 0; e < kGaeE; ++e) sd[at(t * kGaeE + e)] = o[e];
        if (t == 0) s_carry = o[0];
        __syncthreads();
        for (int i = t; i < kGaeTile && t0 + i < L; i += 256) {
            const float x = sd[at(i)];
            if (adv) adv[r.offset + t0 + i] = x;
            if (ret) ret[r.offset + t0 + i] = x + sv[at(i)];
        }
        __syncthreads();
    }
}

hipError_t launch_gae(hipStream_t st, const float* lp_actor, const float* lp_ref, const float* values,
                      const float* reward, const PackRow* rows, int n, int stride, float gamma, float kl_coef,
                      const GaePowers& pw, float* adv, float* ret) {
    if (n <= 0) return hipSuccess;
    k_gae<<<n, 256, 0, st>>>(lp_actor, lp_ref, values, reward, rows, stride, gamma, kl_coef, pw, adv, ret);
    return hipGetLastError();
}

}  // namespace rlhf
