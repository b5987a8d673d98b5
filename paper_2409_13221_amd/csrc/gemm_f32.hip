// Float models, many rows: projections and packed causal attention on float matrix instructions (v_mfma_f32_16x16x4:
// products and sums in float), with everything the decoder block does to a projection's result in its epilogue.
//
// What bounds the projections is the matrix unit (256 flop per cycle and compute unit) if the operands come in time.
// These matrices are a few MB, so both operands come out of the L2 straight into matrix-operand registers, no LDS: a
// wave owns 16 * MBW activation rows and 64 weight rows, and a chunk of 16 k is (MBW + 4) loads of 16 bytes a lane for
// 16 * MBW matrix instructions of 32 cycles; two to four chunks are in flight.  The four waves of a workgroup lie below each
// other and read the same weight rows out of the L1.
// M = 8192, K = 256, us and TFLOP/s: N = 1376 65, 88; N = 4096 166, 104; N = 256 15, 73 (a register-only loop of these
// instructions 154, in long runs 123; 64 x 64 tiles of vector code in gemm.hip about 25).  Asking for the next chunk before
// working on the present one, two in flight, ran at 71 and 82 where this order ran at 83 and 103.
#include "common.h"
#include "kernels.h"
#include <algorithm>
#include <type_traits>

namespace rlhf {

// First weight row of block b (16 rows) of column tile ct.  MODE 0 and 3: 64 consecutive rows.  MODE 1 (SwiGLU): 32 gate
// rows, then the matching up rows.  MODE 2 (rotary): 32 dims of a head's first half, then their partners: a lane holds both
// members of its pairs.
template <int MODE> __device__ __forceinline__ int f32_wrow(const RowsEpi& ep, int ct, int b) {
    if (MODE == 1) return (b >> 1) * ep.ffn + ct * 32 + (b & 1) * 16;
    if (MODE == 2) {
        const int hd = ep.ro.head_dim, half = hd >> 1, per_head = half / 32;
        return ct / per_head * hd + (b >> 1) * half + (ct % per_head) * 32 + (b & 1) * 16;
    }
    return ct * 64 + b * 16;
}

// Modes as in launch_gemm_stream, but mode 3 is h += result only (ep.res.h): the norm that follows reads whole rows.
template <int MBW, int MODE>
__global__ __launch_bounds__(256) void k_gemm_f32_tall(const float* __restrict__ A, const float* __restrict__ W,
                                                       float* __restrict__ C, int M, int N, int K, const RowsEpi ep) {
    const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6), fr = lane & 15, fq = lane >> 4;
    const int ct = blockIdx.x, m0 = (blockIdx.y * 4 + w) * (16 * MBW);
    if (m0 >= M) return;
    const float *pw[4], *pa[MBW];
#pragma unroll
    for (int b = 0; b < 4; ++b) {                          // rows past a matrix' end: clamped, computed and never stored
        const int last = MODE == 1 ? (b >> 1) * ep.ffn + ep.ffn - 1 : N - 1;
        pw[b] = W + (size_t)min(f32_wrow<MODE>(ep, ct, b) + fr, last) * K + fq * 4;
    }
#pragma unroll
    for (int mb = 0; mb < MBW; ++mb) pa[mb] = A + (size_t)min(m0 + mb * 16 + fr, M - 1) * K + fq * 4;
    f32x4_t acc[4][MBW];
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int mb = 0; mb < MBW; ++mb) acc[b][mb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    constexpr int D = MBW == 1 ? 4 : MBW == 2 ? 3 : 2;     // chunks in flight
    float4 fw[D][4], fa[D][MBW];
    auto fetch = [&](int c, int u) {
        const int k = c * 16;
#pragma unroll
        for (int b = 0; b < 4; ++b) fw[u][b] = *reinterpret_cast<const float4*>(pw[b] + k);
#pragma unroll
        for (int mb = 0; mb < MBW; ++mb) fa[u][mb] = *reinterpret_cast<const float4*>(pa[mb] + k);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto step = [&](int u) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int b = 0; b < 4; ++b)
#pragma unroll
                for (int mb = 0; mb < MBW; ++mb)
                    acc[b][mb] = __builtin_amdgcn_mfma_f32_16x16x4f32((&fw[u][b].x)[e], (&fa[u][mb].x)[e], acc[b][mb], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    };
    const int n = K >> 4;                                  // whole chunks
    if (n > 0) {
#pragma unroll
        for (int j = 0; j < D; ++j) fetch(min(j, n - 1), j);
        int c = 0;
        for (; c + 2 * D <= n; c += D) {                   // successors for certain: no branches, exact waits
#pragma unroll
            for (int j = 0; j < D; ++j) {
                step(j);
                fetch(c + j + D, j);
            }
        }
        if (c + D <= n) {
#pragma unroll
            for (int j = 0; j < D; ++j) {
                step(j);
                if (c + j + D < n) fetch(c + j + D, j);
            }
            c += D;
        }
#pragma unroll
        for (int j = 0; j < D - 1; ++j)
            if (c + j < n) step(j);
    }
    if (K & 15) {                                          // 4, 8 or 12 k are left
        const bool in = n * 16 + fq * 4 < K;
        const int k = in ? n * 16 : K - 4 - fq * 4;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            fw[0][b] = *reinterpret_cast<const float4*>(pw[b] + k);
            if (!in) fw[0][b] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
#pragma unroll
        for (int mb = 0; mb < MBW; ++mb) {
            fa[0][mb] = *reinterpret_cast<const float4*>(pa[mb] + k);
            if (!in) fa[0][mb] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
        step(0);
    }

    // acc[b][mb][e]: row m0 + mb * 16 + fr, weight row fq * 4 + e of block b
#pragma unroll
    for (int mb = 0; mb < MBW; ++mb) {
        const int m = m0 + mb * 16 + fr;
        if (m >= M) continue;
        if constexpr (MODE == 0) {
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                const int c = ct * 64 + b * 16 + fq * 4;
                const f32x4_t v = acc[b][mb];
                float* dst = C + (size_t)m * N + c;
                if (c + 3 < N && (N & 3) == 0) {
                    *reinterpret_cast<float4*>(dst) = make_float4(v[0], v[1], v[2], v[3]);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (c + e < N) dst[e] = v[e];
                }
            }
        }
        if constexpr (MODE == 1) {
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const int c = ct * 32 + p * 16 + fq * 4;
                float o[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float g = acc[p][mb][e];
                    o[e] = g / (1.f + __expf(-g)) * acc[2 + p][mb][e];
                }
                if (c < ep.ffn) *reinterpret_cast<float4*>((float*)ep.act + (size_t)m * ep.ffn + c) = make_float4(o[0], o[1], o[2], o[3]);   // ffn % 4 == 0
            }
        }
        if constexpr (MODE == 2) {
            const RopeOut& ro = ep.ro;
            const int hd = ro.head_dim, half = hd >> 1, per_head = half / 32, Hq = ro.n_q_heads, Hkv = ro.n_kv_heads;
            const int head = ct / per_head, slot = ro.pool ? ro.kv_dst[m] : 0, pt = ro.page_tokens;
            const float* table = ro.table + (size_t)ro.pos[m] * hd;
            const bool rot = head < Hq + Hkv, is_q = head < Hq;
            const int kh = is_q ? 0 : rot ? head - Hq : head - Hq - Hkv;
            float* lin = is_q ? (float*)ro.q + ((size_t)m * Hq + head) * hd
                              : (rot ? (float*)ro.k : (float*)ro.v) ? (rot ? (float*)ro.k : (float*)ro.v) + ((size_t)m * Hkv + kh) * hd : nullptr;
            float* prow = is_q || !ro.pool ? nullptr
                                           : (float*)ro.pool + ((size_t)(slot / pt) * ro.n_layers + ro.layer) * 2 * (size_t)Hkv * pt * hd +
                                                 ((size_t)(rot ? 0 : Hkv) + kh) * pt * hd + (size_t)(slot % pt) * hd;
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const int c = (ct % per_head) * 32 + p * 16 + fq * 4;
                const float4 t0 = *reinterpret_cast<const float4*>(table + 2 * c), t1 = *reinterpret_cast<const float4*>(table + 2 * c + 4);
                const float cs[4] = {t0.x, t0.z, t1.x, t1.z}, sn[4] = {t0.y, t0.w, t1.y, t1.w};
                float a[4], b[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float x = acc[p][mb][e], y = acc[2 + p][mb][e];
                    a[e] = rot ? x * cs[e] - y * sn[e] : x;
                    b[e] = rot ? x * sn[e] + y * cs[e] : y;
                }
                for (float* dst : {lin, prow})
                    if (dst) {
                        *reinterpret_cast<float4*>(dst + c) = make_float4(a[0], a[1], a[2], a[3]);
                        *reinterpret_cast<float4*>(dst + half + c) = make_float4(b[0], b[1], b[2], b[3]);
                    }
            }
        }
        if constexpr (MODE == 3) {
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                const int c = ct * 64 + b * 16 + fq * 4;
                if (c >= N) continue;                      // N % 4 == 0
                float4* dst = reinterpret_cast<float4*>(ep.res.h + (size_t)m * N + c);
                const float4 o = *dst;
                const f32x4_t v = acc[b][mb];
                *dst = make_float4(o.x + v[0], o.y + v[1], o.z + v[2], o.w + v[3]);
            }
        }
    }
}

// Packed varlen causal attention, float: a wave owns 16 consecutive queries of one sequence and head and walks the keys 16 at
// a time: S^T[key][q] = K Q^T, softmax along the keys (a lane holds four of one query; its lanes meet by two xor-shuffles),
// O^T[d][q] += V^T P^T.  The lane's own four probabilities are the second product's right operand, and with dim d of
// block b taken as 4 * row + b its left one is four rows of V read 16 bytes a lane.  K and V come from the caches (the waves
// of a workgroup read the same ones), V requested before the first product, the next K before the second; no LDS and no
// barriers, so waves past the end of their sequence just end.
// SPLIT: the four waves of a workgroup own the same 16 queries and every fourth tile of keys, and meet in LDS.  With few
// tiles the time is that of the longest sequence's chain, 0.85 us for 16 keys (1.4 with heads of 128).  us, a wave per 16 queries / SPLIT / a
// workgroup per query (k_prefill_attn): one sequence, 4 heads of 64, 64 tokens 8 / 6 / 6, 300 20 / 10 / 11, 1200 63 / 28 / 74, 4800 357 /
// 195 / 961; 8 heads of 128 300 tokens 31 / 14 / 37, 1200 104 / 68 / 340.  Where every SIMD has work the shares cost more than they
// save: tiles times heads, 128 of 64 tokens 9 / 8, 180 of 64 9 / 9 (64; heads of 128 192 13 / 18), 192 of 300 24 / 21 (128: 41 / 40), 320 of
// 600 69 / 55 (128: 113 / 115), 360 of 100 21 / 27, 640 of 1200 181 / 209.
template <int HD, bool SPLIT>
__global__ __launch_bounds__(256) void k_flash_attn_f32(const float* __restrict__ q, const float* __restrict__ k,
                                                        const float* __restrict__ v, const int* __restrict__ tile_start,
                                                        const int* __restrict__ tile_q0, const int* __restrict__ tile_len,
                                                        float* __restrict__ out, int Hq, int Hkv) {
    constexpr int KC = HD / 16, VC = HD / 64, STEP = SPLIT ? 4 : 1;
    const int tile = blockIdx.x, h = blockIdx.y, kh = h / (Hq / Hkv);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), fr = lane & 15, fq = lane >> 4;
    const int s0 = tile_start[tile], L = tile_len[tile], q0 = tile_q0[tile] + (SPLIT ? (int)blockIdx.z : (int)blockIdx.z * 4 + wave) * 16;
    if (q0 >= L) return;
    const int qrow = q0 + fr;
    const size_t qstride = (size_t)Hq * HD, kstride = (size_t)Hkv * HD;
    const float scale = rsqrtf((float)HD);
    float4 qf[KC];
#pragma unroll
    for (int c = 0; c < KC; ++c) {
        qf[c] = *reinterpret_cast<const float4*>(q + (size_t)(s0 + min(qrow, L - 1)) * qstride + (size_t)h * HD + c * 16 + fq * 4);
        qf[c].x *= scale; qf[c].y *= scale; qf[c].z *= scale; qf[c].w *= scale;
    }
    const float* kb = k + (size_t)s0 * kstride + (size_t)kh * HD + fq * 4;
    const float* vb = v + (size_t)s0 * kstride + (size_t)kh * HD + fr * 4;
    const int n_kt = min(q0 + 15, L - 1) / 16 + 1;
    float4 kf[KC], vf[4][VC];
    auto fetch_k = [&](int kt) {
        const float* src = kb + (size_t)min(kt * 16 + fr, L - 1) * kstride;
#pragma unroll
        for (int c = 0; c < KC; ++c) kf[c] = *reinterpret_cast<const float4*>(src + c * 16);
    };
    f32x4_t o[VC * 4];
#pragma unroll
    for (int b = 0; b < VC * 4; ++b) o[b] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    float m = -INFINITY, l = 0.f, p[4];
    bool redo = false;
    auto attend = [&](int kt, auto last) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float* src = vb + (size_t)min(kt * 16 + fq * 4 + i, L - 1) * kstride;
#pragma unroll
            for (int x = 0; x < VC; ++x) vf[i][x] = *reinterpret_cast<const float4*>(src + x * 64);
        }
        __builtin_amdgcn_sched_barrier(0);
        f32x4_t s = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < KC; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e) s = __builtin_amdgcn_mfma_f32_16x16x4f32((&kf[c].x)[e], (&qf[c].x)[e], s, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        fetch_k(min(kt + STEP, n_kt - 1));
        __builtin_amdgcn_sched_barrier(0);
        float mx = -INFINITY;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (kt * 16 + fq * 4 + e > qrow) s[e] = -INFINITY;
            mx = fmaxf(mx, s[e]);
        }
        mx = fmaxf(mx, __shfl_xor(mx, 16, kWave));
        mx = fmaxf(mx, __shfl_xor(mx, 32, kWave));
        const float m_new = fmaxf(m, mx);                  // finite: every query sees the first key of every tile
        const float alpha = __expf(m - m_new);             // exp(-inf) = 0 on the first tile
        m = m_new;
        float ls = 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            p[e] = __expf(s[e] - m_new);
            ls += p[e];
        }
        l = l * alpha + ls;                                // this lane's keys; the lanes of a query meet at the end
#pragma unroll
        for (int b = 0; b < VC * 4; ++b) o[b] *= alpha;
        if constexpr (decltype(last)::value) {             // the tile with keys that some queries do not see
            bool bad = false;
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int x = 0; x < VC; ++x) bad |= !isfinite(vf[i][x].x + vf[i][x].y + vf[i][x].z + vf[i][x].w);
            redo = __any(bad);
            if (redo) return;                              // 0 * inf would reach them
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int x = 0; x < VC; ++x)
#pragma unroll
                for (int b = 0; b < 4; ++b)
                    o[x * 4 + b] = __builtin_amdgcn_mfma_f32_16x16x4f32((&vf[i][x].x)[b], p[i], o[x * 4 + b], 0, 0, 0);
    };
    const int kt0 = SPLIT ? wave : 0;
    fetch_k(min(kt0, n_kt - 1));
    for (int kt = kt0; kt < n_kt - 1; kt += STEP) attend(kt, std::false_type{});
    if (!SPLIT || (n_kt - 1) % STEP == wave) attend(n_kt - 1, std::true_type{});
    if (__builtin_expect(redo, 0)) {                       // the last tile key by key, for the queries that see it
#pragma unroll 1
        for (int j = 0; j < 16; ++j) {
            const int key = (n_kt - 1) * 16 + j;
            const float pe = (j & 3) == 0 ? p[0] : (j & 3) == 1 ? p[1] : (j & 3) == 2 ? p[2] : p[3];
            const float pj = __shfl(pe, (j >> 2) * 16 + fr, kWave);
            const float* src = vb + (fq * 16 - fr * 4) + (size_t)min(key, L - 1) * kstride;
            if (key > qrow) continue;
#pragma unroll
            for (int x = 0; x < VC; ++x)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float4 w = *reinterpret_cast<const float4*>(src + x * 64 + e * 4);
#pragma unroll
                    for (int b = 0; b < 4; ++b) o[x * 4 + b][e] += pj * (&w.x)[b];
                }
        }
    }
    l += __shfl_xor(l, 16, kWave);
    l += __shfl_xor(l, 32, kWave);
    if constexpr (SPLIT) {                                 // the waves' shares of the keys meet (none: m = -inf, l = 0)
        __shared__ float s_m[4][16], s_l[4][16];
        __shared__ __align__(16) float s_o[4][16][HD + 4];
        if (fq == 0) { s_m[wave][fr] = m; s_l[wave][fr] = l; }
        __syncthreads();
        const float w = __expf(m - fmaxf(fmaxf(s_m[0][fr], s_m[1][fr]), fmaxf(s_m[2][fr], s_m[3][fr])));
#pragma unroll
        for (int x = 0; x < VC; ++x)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                *reinterpret_cast<float4*>(&s_o[wave][fr][x * 64 + (fq * 4 + e) * 4]) =
                    make_float4(o[x * 4][e] * w, o[x * 4 + 1][e] * w, o[x * 4 + 2][e] * w, o[x * 4 + 3][e] * w);
        __syncthreads();
        for (int i = threadIdx.x; i < 16 * (HD / 4); i += 256) {
            const int r = i / (HD / 4), c = i % (HD / 4) * 4;
            if (q0 + r >= L) continue;
            const float mr = fmaxf(fmaxf(s_m[0][r], s_m[1][r]), fmaxf(s_m[2][r], s_m[3][r]));
            float lt = 0.f;
            float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
            for (int k4 = 0; k4 < 4; ++k4) {
                lt += s_l[k4][r] * __expf(s_m[k4][r] - mr);
                const float4 b = *reinterpret_cast<const float4*>(&s_o[k4][r][c]);
                a.x += b.x; a.y += b.y; a.z += b.z; a.w += b.w;
            }
            const float inv = 1.f / lt;
            *reinterpret_cast<float4*>(out + (size_t)(s0 + q0 + r) * qstride + (size_t)h * HD + c) =
                make_float4(a.x * inv, a.y * inv, a.z * inv, a.w * inv);
        }
        return;
    }
    if (qrow >= L) return;
    const float inv = 1.f / l;
    float* dst = out + (size_t)(s0 + qrow) * qstride + (size_t)h * HD;
#pragma unroll
    for (int x = 0; x < VC; ++x)
#pragma unroll
        for (int e = 0; e < 4; ++e)                        // dims 4 * (fq * 4 + e) .. + 3
            *reinterpret_cast<float4*>(dst + x * 64 + (fq * 4 + e) * 4) =
                make_float4(o[x * 4][e] * inv, o[x * 4 + 1][e] * inv, o[x * 4 + 2][e] * inv, o[x * 4 + 3][e] * inv);
}

// Rows per wave (16 * mbw) with the least time.  A workgroup's chunk of 16 k takes its matrix instructions, 512 * mbw cycles, or
// its four waves' loads, 66 cycles each (mbw + 4 of them a wave), whichever is more, and workgroups share a compute unit's
// time: rounds of 256 of them.  More rows a wave need fewer loads a product but fill the chip later.  us, 16 / 32 / 64
// rows a wave: N = K = 4096 64 rows 141 / 120 / 234, 512 rows 281 / 174 / 240, 1024 rows 560 / 344 / 242, 2048 rows 1115 / 688 / 567;
// N = 22016, K = 4096 64 rows 302 / 246 / 238; N = K = 768 1024 rows 29 / 34 / 49.  (By the number of workgroups alone, from 512
// of them on, the choice was up to 2.3 times the best one, and up to 1.22 times the kernel of gemm.hip.)  A second round
// of 64 rows takes a sixth more than the first.  The choice is within 3 % of the best one from 64 rows on (N = 256 .. 32000, K =
// 256 .. 11008, up to 4096 rows), and below 0.94 times the kernel of gemm.hip.
struct F32Shape { int mbw; double us; };
static F32Shape f32_shape(int M, int N, int K) {
    F32Shape best{1, 0.};
    for (int b = 1; b <= 4; b *= 2) {
        const int waves = std::min(4, (M + 16 * b - 1) / (16 * b));
        const long rounds = ((long)((N + 63) / 64) * ((M + 64 * b - 1) / (64 * b)) + 255) / 256;
        const double chunk = b == 4 && rounds > 1 ? 37. : std::max(8 * b, waves * (b + 4));       // in 64 cycles
        const double us = 3. + (K + 15) / 16 * 0.0272 * (double)rounds * chunk;
        if (b == 1 || us < 0.97 * best.us) best = F32Shape{b, us};
    }
    return best;
}
double gemm_f32_tall_us(int M, int N, int K) { return f32_shape(M, N, K).us; }

bool gemm_f32_tall_supported(int N, int K, int mode) { return K >= 4 && K % 4 == 0 && (mode == 0 || N % 8 == 0); }

hipError_t launch_gemm_f32_tall(hipStream_t st, int mode, const float* A, const float* W, float* C, int M, int N, int K,
                                const RowsEpi& ep) {
    if (M <= 0 || N <= 0) return hipSuccess;
    if (mode < 0 || mode > 3 || !gemm_f32_tall_supported(N, K, mode) || (long)M > 65535L * 64) return hipErrorInvalidValue;
    if (mode == 0 ? !C : mode == 1 ? !ep.act || N != 2 * ep.ffn || ep.ffn % 4 : mode == 3 ? !ep.res.h : false) return hipErrorInvalidValue;
    if (mode == 2) {
        const RopeOut& ro = ep.ro;
        if ((ro.head_dim != 64 && ro.head_dim != 128) || !ro.pos || !ro.table || !ro.q || (ro.pool && !ro.kv_dst) ||
            N != (ro.n_q_heads + 2 * ro.n_kv_heads) * ro.head_dim)
            return hipErrorInvalidValue;
    }
    const int cols = mode == 1 ? (ep.ffn + 31) / 32 : (N + 63) / 64;
    const int mbw = f32_shape(M, N, K).mbw;
    const dim3 grid(cols, (M + 64 * mbw - 1) / (64 * mbw));
#define RLHF_F32(MODE)                                                                                    \
    case MODE:                                                                                            \
        if (mbw == 4) k_gemm_f32_tall<4, MODE><<<grid, 256, 0, st>>>(A, W, C, M, N, K, ep);               \
        else if (mbw == 2) k_gemm_f32_tall<2, MODE><<<grid, 256, 0, st>>>(A, W, C, M, N, K, ep);          \
        else k_gemm_f32_tall<1, MODE><<<grid, 256, 0, st>>>(A, W, C, M, N, K, ep);                        \
        break
    switch (mode) { RLHF_F32(0); RLHF_F32(1); RLHF_F32(2); RLHF_F32(3); }
#undef RLHF_F32
    return hipGetLastError();
}

hipError_t launch_flash_attn_f32(hipStream_t st, const float* q, const float* k, const float* v, const int* tile_start,
                                 const int* tile_q0, const int* tile_len, float* out, int n_tiles, int longest, const Dims& dm) {
    if (n_tiles <= 0) return hipSuccess;
    const bool split = (long)n_tiles * dm.n_q_heads <= std::min(384, longest / 2 + 32);
    const dim3 grid(n_tiles, dm.n_q_heads, split ? kFlashTile / 16 : kFlashTile / 64);
#define RLHF_FLASH_F32(HD, SPLIT) \
    k_flash_attn_f32<HD, SPLIT><<<grid, 256, 0, st>>>(q, k, v, tile_start, tile_q0, tile_len, out, dm.n_q_heads, dm.n_kv_heads)
    if (dm.head_dim == 64) { if (split) RLHF_FLASH_F32(64, true); else RLHF_FLASH_F32(64, false); }
    else if (dm.head_dim == 128) { if (split) RLHF_FLASH_F32(128, true); else RLHF_FLASH_F32(128, false); }
    else return hipErrorInvalidValue;
#undef RLHF_FLASH_F32
    return hipGetLastError();
}

}  // namespace rlhf
