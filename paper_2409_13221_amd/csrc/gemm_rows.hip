// Projections of decode steps of up to 256 rows (and of passes as short): every weight is read once, by one
// workgroup that holds all activation rows, and what the decoder block does to the result rides in the epilogue.
//
// What bounds it is the weight stream from HBM, and close behind it the activations that every compute unit
// takes from the L2 (256 rows: 32 KB per 64 k beside 8-16 KB of weights, at 64 bytes a cycle).  Loads complete
// in order within a wave, so a wave that waits for activations out of the L2 would also wait for the weights
// it has requested before them, and the weight stream would be no deeper than the activations'.  Hence two
// kinds of waves: four loaders keep a ring of D steps (64 k) of the workgroup's 16 * NB weight rows coming,
// global -> LDS directly; CW compute waves own 16 * MBW activation rows each, which nobody shares and
// which therefore go from the L2 straight into matrix-operand registers, DA steps ahead.  One barrier a step.
//
// Measured on the 7B shapes, half copies, weights cold, us: 64 rows QKV / O / gate||up / down / head 23.9 / 9 / 30.7 / 18.0 / 41
// (workgroups in step along K: 25.2 / 9 / 37.5 / 18.3 / 58.6; k_gemm_stream 22.6 / 10.6 / 34.6 / 21.8 / 47); 128 rows 32.6 / 12.3 / 43.7 / 25.5 / 60
// (128 x 128 tiles with rotary and SwiGLU kernels behind them: 42 / 18 / 63 / 29); 256 rows 47 / 18 / 54 / 34 / 70
// (256 x 256 tiles with K split: 53 / 27 / 70 / 43 / 83).  From 128 rows on it is the activations: about 75 KB
// per us and compute unit arrive, whatever their prefetch distance (5 or 8 steps) and the ring's depth (6, 10, 16).
#include "common.h"
#include "kernels.h"

namespace rlhf {

namespace {

typedef __attribute__((address_space(3))) void* lds_ptr_t;
typedef uint32_t u32x4r_t __attribute__((ext_vector_type(4)));
typedef _Float16 f16x4r_t __attribute__((ext_vector_type(4)));
constexpr int kLoaders = 4;

// s_waitcnt vmcnt(LPW * steps), steps <= MAX
template <int LPW, int MAX> __device__ __forceinline__ void wait_steps(int steps) {
    if constexpr (MAX > 0) {
        if (steps < MAX) return wait_steps<LPW, MAX - 1>(steps);
    }
    asm volatile("s_waitcnt vmcnt(%0)" : : "n"(LPW * MAX) : "memory");
}

[[maybe_unused]] __device__ __forceinline__ f16x4r_t half4(const float (&o)[4]) { return f16x4r_t{(f16_t)o[0], (f16_t)o[1], (f16_t)o[2], (f16_t)o[3]}; }

}  // namespace

// First of the 16 weight rows of block b, and the last row there is (rows past it are clamped, computed and
// never stored).  MODE 0: consecutive rows.  MODE 1 (SwiGLU) and 2 (rotary): blocks come in pairs, 16 gate rows and the
// matching up rows, or dims c .. c + 15 of a head and c + hd/2 .., so that a lane holds both members.
template <int MODE> __device__ __forceinline__ int rows_wrow(const RowsEpi& ep, int N, int b, int* last) {
    if (MODE == 1) {
        *last = (b & 1) * ep.ffn + ep.ffn - 1;
        return (b & 1) * ep.ffn + min((b >> 1) * 16, ep.ffn - 1);
    }
    *last = N - 1;
    if (MODE == 2) {
        const int hd = ep.ro.head_dim, half = hd >> 1, per_head = half / 16;
        return min((b >> 1) / per_head, N / hd - 1) * hd + (b & 1) * half + ((b >> 1) % per_head) * 16;
    }
    return min(b * 16, N - 1);
}

// A: half activations; W: bf16 (CVT, converted after the LDS read) or its half copy.  Modes as in launch_gemm_stream.
template <int MBW, int CW, int NB, int D, int MODE, bool CVT>
__global__ __launch_bounds__((CW + kLoaders) * 64) void k_gemm_rows(const f16_t* __restrict__ A, const bf16_t* __restrict__ W,
                                                                    float* __restrict__ C, int M, int N, int K, int kchunk,
                                                                    const RowsEpi ep) {
#if defined(__HIP_DEVICE_COMPILE__)                        // buffer resources exist in the device pass only
    constexpr int LPW = NB * 2 / kLoaders;                 // loads (8 rows x 128 bytes) per loader and step
    constexpr int kSlot = NB * 2048;
    constexpr int DA = MBW == 1 ? 8 : NB <= 4 ? 5 : 3;      // as many as registers allow
    static_assert(NB % 2 == 0 && LPW >= 1 && (D - 2) * LPW < 64, "blocks in pairs, whole loads per loader, six bits of vmcnt");
    __shared__ __attribute__((aligned(16))) uint8_t ring[D * kSlot];
    const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int blk = blockIdx.x;
    const int kbeg = MODE == 0 ? (int)blockIdx.y * kchunk : 0;
    const int n = (MODE == 0 ? min(K, kbeg + kchunk) - kbeg : K) >> 6;
    // workgroups start at different steps, as in gemm_stream.hip
    const int rot = (blk >> 3) % n;
    auto step_at = [&](int i) { return i + rot >= n ? i + rot - n : i + rot; };
#define RLHF_R_BAR                                                     \
    do {                                                               \
        __builtin_amdgcn_sched_barrier(0);                             \
        asm volatile("s_barrier" : : : "memory");                      \
        __builtin_amdgcn_sched_barrier(0);                             \
    } while (0)
    if (w >= CW) {                                         // ---- loaders
        const int lw = w - CW;
        __amdgpu_buffer_rsrc_t rs[LPW];
        uint32_t vo[LPW];
#pragma unroll
        for (int i = 0; i < LPW; ++i) {
            const int q = lw * LPW + i;                    // piece: rows (q & 1) * 8 .. of block q / 2
            int last;
            const int first = rows_wrow<MODE>(ep, N, blk * NB + (q >> 1), &last);
            const int base = __builtin_amdgcn_readfirstlane(first), lim = last - base, r = (q & 1) * 8 + (lane >> 3);
            rs[i] = __builtin_amdgcn_make_buffer_rsrc((void*)(W + (size_t)base * K + kbeg), 0, -1, 0x00020000);
            // LDS position p of row r holds chunk p ^ r (mod 8): the fragment reads then spread over the banks
            vo[i] = (uint32_t)(min(r, lim) * K * 2 + ((lane & 7) ^ (r & 7)) * 16);
        }
        auto issue = [&](int step, int slot) {
#pragma unroll
            for (int i = 0; i < LPW; ++i)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rs[i], (lds_ptr_t)(ring + slot * kSlot + (lw * LPW + i) * 1024), 16, vo[i],
                                                         step_at(step) * 128, 0, 2);
        };
        for (int j = 0; j < D - 1 && j < n; ++j) issue(j, j);
        int slot = D - 1;                                  // of step k + D - 1, which is that of step k - 1
        for (int k = 0; k < n; ++k) {
            wait_steps<LPW, D - 2>(min(n - 1 - k, D - 2)); // step k has landed
            RLHF_R_BAR;                                    // ... and everybody has read step k - 1
            if (k + D - 1 < n) issue(k + D - 1, slot);
            slot = slot + 1 == D ? 0 : slot + 1;
        }
        return;
    }
    // ---- compute waves: row blocks w, w + CW
    const int fr = lane & 15, fq = lane >> 4;
    const f16_t* pa[MBW];
#pragma unroll
    for (int mb = 0; mb < MBW; ++mb) pa[mb] = A + act_index(ep.a, min((w + mb * CW) * 16 + fr, M - 1), kbeg + fq * 8);
    const size_t a_half = (size_t)4 * ep.a.chunk;          // elements from one 32-k half of a step to the next
    f16x8_t fa[DA][MBW][2];
    auto fetch = [&](int i, int j) {
        const int step = step_at(i);
#pragma unroll
        for (int mb = 0; mb < MBW; ++mb) {                 // rows past the end: the last one again (no branch, the
            fa[j][mb][0] = *reinterpret_cast<const f16x8_t*>(pa[mb] + (size_t)step * 2 * a_half);  // waits stay exact)
            fa[j][mb][1] = *reinterpret_cast<const f16x8_t*>(pa[mb] + (size_t)step * 2 * a_half + a_half);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    f32x4_t acc[NB][MBW];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int mb = 0; mb < MBW; ++mb) acc[nb][mb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < DA; ++j) fetch(min(j, n - 1), j);
    // fragment reads: row fr of a block, chunk s * 4 + fq, in groups of GS blocks, one group ahead of its use
    constexpr int GS = NB <= 4 ? NB : NB / 2, GPS = NB / GS, NG = 2 * GPS;
    const uint32_t lb = (uint32_t)(size_t)(lds_ptr_t)ring + fr * 128;
    const uint32_t l_off[2] = {lb + ((uint32_t)fq ^ (fr & 7)) * 16, lb + ((uint32_t)(4 + fq) ^ (fr & 7)) * 16};
    u32x4r_t wf[2][GS];
#define RLHF_R_READ(G)                                                                                               \
    do {                                                                                                             \
        _Pragma("unroll") for (int i = 0; i < GS; ++i)                                                               \
            asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(wf[(G) & 1][i])                                      \
                         : "v"(l_off[(G) / GPS] + so), "n"((((G) % GPS) * GS + i) * 2048) : "memory");               \
    } while (0)
    int slot = 0;
#define RLHF_R_STEP(J)                                                                                               \
    do {                                                                                                             \
        RLHF_R_BAR;                                                                                                  \
        const uint32_t so = (uint32_t)slot * kSlot;                                                                  \
        slot = slot + 1 == D ? 0 : slot + 1;                                                                         \
        RLHF_R_READ(0);                                                                                              \
        _Pragma("unroll") for (int g = 0; g < NG; ++g) {                                                             \
            if (g + 1 < NG) {                                                                                        \
                RLHF_R_READ(g + 1);                                                                                  \
                asm volatile("s_waitcnt lgkmcnt(%0)" : : "n"(GS) : "memory");                                        \
            } else {                                                                                                 \
                asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");                                                 \
            }                                                                                                        \
            _Pragma("unroll") for (int i = 0; i < GS; ++i) asm volatile("" : "+v"(wf[g & 1][i])); /* tied to the wait */ \
            _Pragma("unroll") for (int i = 0; i < GS; ++i) {                                                         \
                u32x4r_t x = wf[g & 1][i];                                                                           \
                if (CVT) {                                                                                           \
                    _Pragma("unroll") for (int e = 0; e < 4; ++e) x[e] = bf16x2_to_f16x2(x[e]);                      \
                }                                                                                                    \
                const f16x8_t wv = *reinterpret_cast<const f16x8_t*>(&x);                                            \
                _Pragma("unroll") for (int mb = 0; mb < MBW; ++mb)                                                   \
                    acc[(g % GPS) * GS + i][mb] =                                                                    \
                        __builtin_amdgcn_mfma_f32_16x16x32_f16(wv, fa[J][mb][g / GPS], acc[(g % GPS) * GS + i][mb], 0, 0, 0); \
            }                                                                                                        \
            __builtin_amdgcn_sched_barrier(0);                                                                       \
        }                                                                                                            \
    } while (0)
    int k0 = 0;
    for (; k0 + DA <= n; k0 += DA) {
#pragma unroll
        for (int j = 0; j < DA; ++j) {
            RLHF_R_STEP(j);
            fetch(min(k0 + j + DA, n - 1), j);
        }
    }
#pragma unroll
    for (int j = 0; j < DA - 1; ++j)
        if (k0 + j < n) RLHF_R_STEP(j);
#undef RLHF_R_STEP
#undef RLHF_R_READ
#undef RLHF_R_BAR

    // ---- epilogues.  acc[nb][mb][e]: activation row (w + mb * CW) * 16 + fr, weight row fq * 4 + e of block nb
#pragma unroll
    for (int mb = 0; mb < MBW; ++mb) {
        const int m = (w + mb * CW) * 16 + fr;
        if (m >= M) continue;
        if constexpr (MODE == 0) {
            float* dst = C + (size_t)blockIdx.y * M * N + (size_t)m * N;
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                const int c = (blk * NB + nb) * 16 + fq * 4;
                const f32x4_t v = acc[nb][mb];
                if (c + 3 < N && (N & 3) == 0) {
                    *reinterpret_cast<float4*>(dst + c) = make_float4(v[0], v[1], v[2], v[3]);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (c + e < N) dst[c + e] = v[e];
                }
            }
        }
        if constexpr (MODE == 1) {
            f16_t* act = reinterpret_cast<f16_t*>(ep.act);
#pragma unroll
            for (int p = 0; p < NB / 2; ++p) {
                const int c = (blk * (NB / 2) + p) * 16 + fq * 4;
                float o[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float g = acc[2 * p][mb][e];
                    o[e] = g / (1.f + __expf(-g)) * acc[2 * p + 1][mb][e];
                }
                if (c < ep.ffn) *reinterpret_cast<f16x4r_t*>(act + act_index(ep.out, m, c)) = half4(o);    // ffn % 16 == 0
            }
        }
        if constexpr (MODE == 2) {
            const RopeOut& ro = ep.ro;
            const int hd = ro.head_dim, half = hd >> 1, per_head = half / 16, Hq = ro.n_q_heads, Hkv = ro.n_kv_heads;
            const int slot_m = ro.pool ? ro.kv_dst[m] : 0, pt = ro.page_tokens;
            const float* row_table = ro.table + (size_t)ro.pos[m] * hd;
            f16_t* prow = nullptr;                         // this token's K row of head 0 in the pool
            if (ro.pool)
                prow = (f16_t*)ro.pool + ((size_t)(slot_m / pt) * ro.n_layers + ro.layer) * 2 * (size_t)Hkv * pt * hd +
                       (size_t)(slot_m % pt) * hd;
            float4 tb[NB / 2][2];
#pragma unroll
            for (int p = 0; p < NB / 2; ++p) {
                const int c = ((blk * (NB / 2) + p) % per_head) * 16 + fq * 4;
                tb[p][0] = *reinterpret_cast<const float4*>(row_table + 2 * c);
                tb[p][1] = *reinterpret_cast<const float4*>(row_table + 2 * c + 4);
            }
#pragma unroll
            for (int p = 0; p < NB / 2; ++p) {
                const int pi = blk * (NB / 2) + p, head = pi / per_head, c = (pi % per_head) * 16 + fq * 4;
                if (head >= Hq + 2 * Hkv) continue;
                const float cs[4] = {tb[p][0].x, tb[p][0].z, tb[p][1].x, tb[p][1].z};
                const float sn[4] = {tb[p][0].y, tb[p][0].w, tb[p][1].y, tb[p][1].w};
                float a[4], b[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float x = acc[2 * p][mb][e], y = acc[2 * p + 1][mb][e];
                    const bool rot = head < Hq + Hkv;
                    a[e] = rot ? x * cs[e] - y * sn[e] : x;
                    b[e] = rot ? x * sn[e] + y * cs[e] : y;
                }
                const f16x4r_t ha = half4(a), hb = half4(b);
                auto put = [&](f16_t* dst) {
                    *reinterpret_cast<f16x4r_t*>(dst + c) = ha;
                    *reinterpret_cast<f16x4r_t*>(dst + c + half) = hb;
                };
                if (head < Hq) {
                    put((f16_t*)ro.q + ((size_t)m * Hq + head) * hd);
                } else {
                    const bool is_k = head < Hq + Hkv;
                    const int kh = is_k ? head - Hq : head - Hq - Hkv;
                    f16_t* lin = (f16_t*)(is_k ? ro.k : ro.v);
                    if (lin) put(lin + ((size_t)m * Hkv + kh) * hd);
                    if (prow) put(prow + ((size_t)(is_k ? 0 : Hkv) + kh) * pt * hd);
                }
            }
        }
    }
#endif
}

namespace {

// Weight blocks per workgroup: as few as leave one round of workgroups (256 compute units, one each): every workgroup
// reads all activations (7B gate||up, 256 rows: 58 us with 6, 86 with 4).  Eight at most (registers).
int rows_nb(int N) {
    const int blocks = (N + 15) / 16;
    for (int nb = 2; nb < 8; nb += 2)
        if ((blocks + nb - 1) / nb <= 256) return nb;
    return 8;
}

template <int MBW, int CW, int NB, int D, bool CVT>
hipError_t rows_launch3(hipStream_t st, int mode, const f16_t* a, const bf16_t* w, float* C, int M, int N, int K, int nsplit,
                        const RowsEpi& ep) {
    const int blocks = ((N + 15) / 16 + NB - 1) / NB, kchunk = ((K + nsplit - 1) / nsplit + 63) / 64 * 64;
    if ((long)(nsplit - 1) * kchunk >= K) return hipErrorInvalidValue;        // a split without a K range
    const dim3 grid(blocks, nsplit), threads((CW + kLoaders) * 64);
    switch (mode) {
        case 0: k_gemm_rows<MBW, CW, NB, D, 0, CVT><<<grid, threads, 0, st>>>(a, w, C, M, N, K, kchunk, ep); break;
        case 1: k_gemm_rows<MBW, CW, NB, D, 1, CVT><<<grid, threads, 0, st>>>(a, w, C, M, N, K, kchunk, ep); break;
        case 2: k_gemm_rows<MBW, CW, NB, D, 2, CVT><<<grid, threads, 0, st>>>(a, w, C, M, N, K, kchunk, ep); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}
template <int MBW, int CW, bool CVT>
hipError_t rows_launch2(hipStream_t st, int mode, int nb, const f16_t* a, const bf16_t* w, float* C, int M, int N, int K,
                        int nsplit, const RowsEpi& ep) {
    switch (nb) {
        case 2: return rows_launch3<MBW, CW, 2, 16, CVT>(st, mode, a, w, C, M, N, K, nsplit, ep);
        case 4: return rows_launch3<MBW, CW, 4, 6, CVT>(st, mode, a, w, C, M, N, K, nsplit, ep);
        case 6: return rows_launch3<MBW, CW, 6, 8, CVT>(st, mode, a, w, C, M, N, K, nsplit, ep);
        default: return rows_launch3<MBW, CW, 8, 6, CVT>(st, mode, a, w, C, M, N, K, nsplit, ep);
    }
}
template <bool CVT>
hipError_t rows_launch1(hipStream_t st, int mode, int nb, const f16_t* a, const bf16_t* w, float* C, int M, int N, int K,
                        int nsplit, const RowsEpi& ep) {
    if (M <= 64) return rows_launch2<1, 4, CVT>(st, mode, nb, a, w, C, M, N, K, nsplit, ep);
    if (M <= 128) return rows_launch2<1, 8, CVT>(st, mode, nb, a, w, C, M, N, K, nsplit, ep);
    return rows_launch2<2, 8, CVT>(st, mode, nb, a, w, C, M, N, K, nsplit, ep);
}

}  // namespace

bool gemm_rows_supported(int wdt, int adt, int M, int K) {
    return (wdt == kBF16 || wdt == kF16) && adt == kF16 && M >= 1 && M <= kRowsMaxRows && K > 0 && K % 64 == 0;
}

// K split of O and down projections: four weight blocks per workgroup, workgroups for every compute unit, at
// least four steps each, eight planes at most.  (7B down, 256 rows: 35 us with four blocks and four planes, 33 with
// eight and eight, which the norm that reads them pays for; 51 with two and two.)
constexpr int kPlaneBlocks = 4;
int gemm_rows_nsplit(int N, int K, int max_split) {
    const int blocks = ((N + 15) / 16 + kPlaneBlocks - 1) / kPlaneBlocks;
    int ns = 256 / blocks;
    ns = ns < (K >> 6) / 4 ? ns : (K >> 6) / 4;
    ns = ns < 8 ? ns : 8;
    ns = ns < max_split ? ns : max_split;
    if (ns < 1) ns = 1;
    while (ns > 1 && (long)(ns - 1) * (((K + ns - 1) / ns + 63) / 64 * 64) >= K) --ns;     // every split gets a K range
    return ns;
}

hipError_t launch_gemm_rows(hipStream_t st, int wdt, int mode, const void* A, const void* W, float* C, int M, int N, int K,
                            const RowsEpi& ep, int nsplit) {
    if ((long)16 * K * 2 >= (1L << 31)) return hipErrorInvalidValue;          // offsets inside a block are 32-bit
    const int nb = nsplit > 1 ? kPlaneBlocks : rows_nb(N);
    return wdt == kF16 ? rows_launch1<false>(st, mode, nb, (const f16_t*)A, (const bf16_t*)W, C, M, N, K, nsplit, ep)
                       : rows_launch1<true>(st, mode, nb, (const f16_t*)A, (const bf16_t*)W, C, M, N, K, nsplit, ep);
}

}  // namespace rlhf
