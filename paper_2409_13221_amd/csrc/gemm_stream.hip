// Projections of decode steps (and of very short passes): up to 64 activation rows against a bf16
// weight matrix that is read once, with everything the decoder block does to the result in the
// epilogue.
//
// What bounds it is how fast the weights come in.  A workgroup owns 16 * NB weight rows and the WHOLE
// K range, its waves a contiguous share of K each, so that nothing is left to a consumer to sum (no
// split-K planes) and the waves never wait for one another before the epilogue.  Weights go global ->
// LDS directly into a ring that belongs to one wave (no barrier, no registers), D steps of 64 k ahead,
// as buffer loads of 8 rows x 128 bytes: whole cache lines per instruction, which the matrix-operand
// layout itself (16 rows x 64 bytes per load) would not give.  Measured on the 7B shapes, weights
// cold, loads alone: 16.9 / 6.7 / 30.2 / 16.9 us (QKV, O, gate||up, down) this way, 17.9 / 7.3 / 32.8
// / 21.3 us with loads in operand layout straight to registers; a linear read of the same bytes takes
// 15.4 / 6.0 / 27.6 / 14.1 us.  A deeper ring (128 KB in flight per workgroup) is slower: 19.6 us QKV.
// Activations are a few KB per step, shared by all workgroups, and come from the L2 straight into
// matrix-operand registers.
//
// Up to 16 rows RMSNorm costs no kernel of its own.  The projection that finishes the residual stream (O, down)
// adds its result to h, and writes x = h * g * s (half; g the next norm's gain, s the power of two below
// the row's previous 1/rms, which rounds nothing by itself) and the partial sums of h^2 of its 16 * NB columns; the
// projection that consumes the normed row multiplies x by W as it is and scales the result of row m by
// (1/rms_m) / s_m in its epilogue.
// x has the size of a normed row as long as one projection does not change the row's rms much.  A row that
// grows may leave half's range (the producer marks it in the sign of its partial sum), one that shrinks sinks
// into half's subnormals ((1/rms) / s > kMaxShrink shows it).  Then the consuming workgroups drop what they
// have summed and take their share of K again from h itself, normalised before the rounding to half: any
// stream that RMSNorm as a kernel can take is taken here, and ordinary rows pay one test.
#include "common.h"
#include "kernels.h"
#include <algorithm>
#include <type_traits>

namespace rlhf {

namespace {

template <bool AF16> struct StreamMfma;
template <> struct StreamMfma<false> {
    typedef bf16x8_t frag;
    static __device__ __forceinline__ f32x4_t run(frag a, frag b, f32x4_t c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
    }
};
template <> struct StreamMfma<true> {
    typedef f16x8_t frag;
    static __device__ __forceinline__ f32x4_t run(frag a, frag b, f32x4_t c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
    }
};

typedef __attribute__((address_space(3))) void* lds_ptr_t;
typedef uint32_t u32x4s_t __attribute__((ext_vector_type(4)));

// Largest (1/rms) / s at which x is used: an entry of x is then at least 1/64 of the normed one, and half's
// subnormal grid (2^-24) still 256 times finer than the rounding of an entry of average size.
constexpr float kMaxShrink = 64.f;

template <int N> __device__ __forceinline__ void wait_vmem() { asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory"); }

}  // namespace

// First weight row of half `hi` (8 rows) of row block b; rows past the end are clamped, computed and never
// stored.  MODE 0 plain, 3 residual: 16 consecutive rows.  MODE 1 (SwiGLU): 8 gate rows and the matching 8
// up rows.  MODE 2 (rotary): dims c .. c+7 and c + hd/2 .. of one head.  So the members of every pair meet
// in one workgroup.
template <int MODE> __device__ __forceinline__ int stream_wrow(const RowsEpi& ep, int N, int b, int hi) {
    if (MODE == 1) return hi * ep.ffn + min(b * 8, ep.ffn - 1);
    if (MODE == 2) {
        const int hd = ep.ro.head_dim, half = hd >> 1, per_head = half / 8;
        const int head = min(b / per_head, N / hd - 1), c = (b % per_head) * 8;
        return head * hd + hi * half + c;
    }
    return min(b * 16 + hi * 8, N - 1);
}
// last row of that half that exists
template <int MODE> __device__ __forceinline__ int stream_last_row(const RowsEpi& ep, int N, int hi) {
    return (MODE == 1 ? (hi + 1) * ep.ffn : N) - 1;
}

// 1/rms of the rows of an unscaled norm input, RPW rows per wave: kSsqStride partial sums of squares each
// (unused ones are zero), a float4 per lane and 256 of them.  FEW: at most 64 are used, one per lane; with 64
// rows the float4 form would take 128 registers.
template <int RPW, bool FEW> struct StreamNorm {
    float4 q0[FEW ? 1 : RPW], q1[FEW ? 1 : RPW];
    float q[RPW], s_in;
    __device__ __forceinline__ void request(const NormIn& ni, int M, int w, int lane) {
        s_in = ni.s_in[min(w * RPW + lane / (64 / RPW), M - 1)];
        if constexpr (FEW) {
#pragma unroll
            for (int i = 0; i < RPW; ++i) q[i] = ni.ssq[(size_t)min(w * RPW + i, M - 1) * kSsqStride + lane];
            return;
        }
        const bool two = ni.n_ssq > 256;
#pragma unroll
        for (int i = 0; i < (FEW ? 1 : RPW); ++i) {
            const float* src = ni.ssq + (size_t)min(w * RPW + i, M - 1) * kSsqStride + lane * 4;
            q0[i] = *reinterpret_cast<const float4*>(src);
            q1[i] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (two) q1[i] = *reinterpret_cast<const float4*>(src + 256);
        }
    }
    // s_scale[m]: factor of row m's result; s_inv[m]: 1/rms.  Returns whether a row of this wave asks for h itself.
    __device__ __forceinline__ bool reduce(const NormIn& ni, int M, int K, int w, int lane, bool first_block, float* s_scale,
                                           float* s_inv) {
        float v[RPW];
        uint32_t sign = 0;
        auto sum = [&](const float4& a, const float4& b) {
            sign |= (__float_as_uint(a.x) | __float_as_uint(a.y)) | (__float_as_uint(a.z) | __float_as_uint(a.w)) |
                    (__float_as_uint(b.x) | __float_as_uint(b.y)) | (__float_as_uint(b.z) | __float_as_uint(b.w));
            return ((fabsf(a.x) + fabsf(b.x)) + (fabsf(a.y) + fabsf(b.y))) + ((fabsf(a.z) + fabsf(b.z)) + (fabsf(a.w) + fabsf(b.w)));
        };
#pragma unroll
        for (int i = 0; i < RPW; ++i)
            if constexpr (FEW) { v[i] = fabsf(q[i]); sign |= __float_as_uint(q[i]); }
            else v[i] = sum(q0[i], q1[i]);
        // all rows at once: every exchange halves the rows a lane still carries, row lane / (64 / RPW) in the end
        int o = 32;
#pragma unroll
        for (int nn = RPW; nn > 1; nn >>= 1, o >>= 1)
#pragma unroll
            for (int i = 0; i < nn / 2; ++i) {
                const bool up = lane & o;
                const float give = up ? v[i] : v[i + nn / 2], keep = up ? v[i + nn / 2] : v[i];
                v[i] = keep + __shfl_xor(give, o, kWave);
            }
#pragma unroll
        for (; o > 0; o >>= 1) v[0] += __shfl_xor(v[0], o, kWave);
        constexpr int LPR = 64 / RPW;
        const int m = w * RPW + lane / LPR;
        bool redo = sign >> 31;
        if (m < M && lane % LPR == 0) {
            const float inv = rsqrtf(v[0] / (float)K + ni.eps), sc = inv / s_in;
            s_scale[m] = sc;
            s_inv[m] = inv;
            redo |= !(sc <= kMaxShrink);                   // NaN too
            if (first_block && ni.s_out) ni.s_out[m] = pow2_below(inv);
        }
        return __any(redo);
    }
};

// What becomes of the result.  The waves' shares of K lie in red[wave][weight row][activation row] (row pitch
// MB * 16 + 1); a thread owns OUT_IT outputs (pairs, in MODE 1 and 2) and asks for what it needs of other
// arrays before the weights come, so that it does not wait at the end.  TO: type of activations and pool.
template <int MB, int NB, int WAVES, int MODE, typename TO> struct StreamEpilogue {
    static constexpr int NT = WAVES * 64, R16 = NB * 16, R8 = NB * 8, MP = MB * 16 + 1;
    static constexpr int OUT_IT = ((MODE == 1 || MODE == 2 ? R8 : R16) * MB * 16 + NT - 1) / NT;
    float pre_a[OUT_IT], pre_b[OUT_IT];                    // MODE 3: h, g * s;  MODE 2: cos, sin
    int pre_i[OUT_IT];                                     // MODE 2: position, then pool slot

    __device__ __forceinline__ void request(const RowsEpi& ep, int M, int N, int blk, int t) {
        if (MODE == 2) {
#pragma unroll
            for (int i = 0; i < OUT_IT; ++i) pre_i[i] = ep.ro.pos[min((t + i * NT) / R8, M - 1)];
        }
        if (MODE == 3) {
#pragma unroll
            for (int i = 0; i < OUT_IT; ++i) {
                const int o = t + i * NT, m = min(o / R16, M - 1), nn = min(blk * R16 + o % R16, N - 1);
                pre_a[i] = ep.res.h[(size_t)m * N + nn];
                pre_b[i] = ep.res.g[nn] * ep.res.s[m];
            }
        }
    }
    __device__ __forceinline__ void request_table(const RowsEpi& ep, int M, int blk, int t) {     // after the first weights
        if (MODE == 2) {
            const int half = ep.ro.head_dim >> 1, per_head = half / 8;
#pragma unroll
            for (int i = 0; i < OUT_IT; ++i) {
                const int o = t + i * NT, r = o % R8, d0 = ((blk * NB + (r >> 3)) % per_head) * 8 + (r & 7);
                const float2 cs = *reinterpret_cast<const float2*>(ep.ro.table + ((size_t)pre_i[i] * half + d0) * 2);
                pre_a[i] = cs.x;
                pre_b[i] = cs.y;
                pre_i[i] = ep.ro.kv_dst ? ep.ro.kv_dst[min(o / R8, M - 1)] : 0;
            }
        }
    }
    __device__ __forceinline__ void finish(const RowsEpi& ep, const float* red, const float* s_scale, bool normed, float* C,
                                           int M, int N, int blk, int t) {
        auto total = [&](int row, int m) {
            float v = 0.f;
#pragma unroll
            for (int x = 0; x < WAVES; ++x) v += red[(x * NB * 16 + row) * MP + m];
            return v;
        };
        if (MODE == 0) {
            for (int i = t; i < R16 * M; i += NT) {
                const int m = i / R16, r = i % R16, nn = blk * R16 + r;
                if (nn < N) C[(size_t)m * N + nn] = total(r, m) * (normed ? s_scale[m] : 1.f);
            }
        }
        if (MODE == 1) {
            TO* act = reinterpret_cast<TO*>(ep.act);
            for (int i = t; i < R8 * M; i += NT) {
                const int m = i / R8, r = i % R8, oc = blk * R8 + r, lr = (r >> 3) * 16 + (r & 7);
                if (oc < ep.ffn) {
                    const float sc = normed ? s_scale[m] : 1.f;
                    const float g = total(lr, m) * sc, u = total(lr + 8, m) * sc;
                    act[act_index(ep.out, m, oc)] = from_f32<TO>(g / (1.f + __expf(-g)) * u);
                }
            }
        }
        if (MODE == 2) {
            const RopeOut& ro = ep.ro;
            const int hd = ro.head_dim, half = hd >> 1, per_head = half / 8;
            const int Hq = ro.n_q_heads, Hkv = ro.n_kv_heads;
            TO* q_out = reinterpret_cast<TO*>(ro.q);
            TO* k_out = reinterpret_cast<TO*>(ro.k);
            TO* v_out = reinterpret_cast<TO*>(ro.v);
            TO* pool = reinterpret_cast<TO*>(ro.pool);
#pragma unroll
            for (int it = 0; it < OUT_IT; ++it) {
                const int i = t + it * NT, m = i / R8, r = i % R8, lr = (r >> 3) * 16 + (r & 7);
                const int b = blk * NB + (r >> 3), head = b / per_head;
                if (m >= M || head >= Hq + 2 * Hkv) continue;
                const int d0 = (b % per_head) * 8 + (r & 7), d1 = d0 + half;
                const float sc = normed ? s_scale[m] : 1.f;
                float a = total(lr, m) * sc, c = total(lr + 8, m) * sc;
                if (head < Hq + Hkv) {
                    const float ra = a * pre_a[it] - c * pre_b[it], rc = a * pre_b[it] + c * pre_a[it];
                    a = ra; c = rc;
                }
                if (head < Hq) {
                    TO* dst = q_out + ((size_t)m * Hq + head) * hd;
                    dst[d0] = from_f32<TO>(a);
                    dst[d1] = from_f32<TO>(c);
                } else {
                    const bool is_k = head < Hq + Hkv;
                    const int kh = is_k ? head - Hq : head - Hq - Hkv;
                    TO* lin = is_k ? k_out : v_out;
                    if (lin) {
                        lin[((size_t)m * Hkv + kh) * hd + d0] = from_f32<TO>(a);
                        lin[((size_t)m * Hkv + kh) * hd + d1] = from_f32<TO>(c);
                    }
                    if (pool) {
                        const int slot = pre_i[it], pt = ro.page_tokens;
                        TO* dst = pool + ((size_t)(slot / pt) * ro.n_layers + ro.layer) * 2 * (size_t)Hkv * pt * hd +
                                  (size_t)(is_k ? 0 : Hkv) * pt * hd + (size_t)kh * pt * hd + (size_t)(slot % pt) * hd;
                        dst[d0] = from_f32<TO>(a);
                        dst[d1] = from_f32<TO>(c);
                    }
                }
            }
        }
        if (MODE == 3) {
            const ResidOut& rz = ep.res;
            TO* x = reinterpret_cast<TO*>(rz.x);
#pragma unroll
            for (int it = 0; it < OUT_IT; ++it) {          // whole waves take part: the sums below are lane shuffles
                const int i = t + it * NT, m = i / R16, r = i % R16, nn = blk * R16 + r;
                float v = 0.f;
                bool over = false;
                if (m < M && nn < N) {
                    v = pre_a[it] + total(r, m);
                    const float xv = v * pre_b[it];
                    over = sizeof(TO) == 2 && fabsf(xv) > 65504.f;
                    rz.h[(size_t)m * N + nn] = v;
                    x[act_index(ep.out, m, nn)] = from_f32<TO>(xv);
                }
                float q = v * v;
#pragma unroll
                for (int o = 1; o < 16; o <<= 1) q += __shfl_xor(q, o, kWave);     // 16 columns of a row: 16 neighbouring lanes
                if (__ballot(over) >> (t & 48) & 0xFFFF) q = -q;
                if (m < M && r % 16 == 0 && nn < N) rz.ssq[(size_t)m * kSsqStride + nn / 16] = q;
            }
        }
    }
};

// MB: 16-row blocks of activations; NB: 16-row blocks of weights per workgroup; WAVES share K; D: ring depth
// in steps of 64 k; NORM: A may be an unscaled norm input (above 16 rows of at most 64 partial sums).
template <int MB, int NB, int WAVES, int D, int MODE, bool AF16, bool NORM>
__global__ __launch_bounds__(WAVES * 64) void k_gemm_stream(const bf16_t* __restrict__ A, const bf16_t* __restrict__ W,
                                                            float* __restrict__ C, int M, int N, int K,
                                                            const RowsEpi ep_in) {
#if defined(__HIP_DEVICE_COMPILE__)                        // buffer resources exist in the device pass only
    constexpr int OPS = 2 * NB + 2 * MB;                   // vector memory operations per step
    constexpr int kRing = WAVES * D * NB * 1024;           // halves (2 KB per step and weight block)
    constexpr int MP = MB * 16 + 1;
    constexpr int kRed = WAVES * NB * 16 * MP;             // floats
    __shared__ __attribute__((aligned(16))) uint8_t smem[kRing * 2 > kRed * 4 ? kRing * 2 : kRed * 4];
    __shared__ float s_scale[MB * 16], s_inv[MB * 16];
    __shared__ int s_redo[WAVES];
    const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int fr = lane & 15, fq = lane >> 4;
    const int blk = blockIdx.x;
    RowsEpi ep = ep_in;
    typedef typename std::conditional<AF16, f16_t, bf16_t>::type TO;
    if (MODE == 0) C += (size_t)blockIdx.y * M * N;        // K range blockIdx.y of gridDim.y: a plane of its own

    if (MODE == 3) {                                       // row group blockIdx.z: everything that goes by rows moves along
        const int m0 = blockIdx.z * (MB * 16);
        M = min(M - m0, MB * 16);
        A += act_index(ep.a, m0, 0);
        ep.res.h += (size_t)m0 * N;
        ep.res.x = (TO*)ep.res.x + act_index(ep.out, m0, 0);
        ep.res.s += m0;
        ep.res.ssq += (size_t)m0 * kSsqStride;
    }

    // this wave's steps; the count is rounded up to whole rings, surplus steps re-read the last one against zeros
    const int steps = K >> 6, parts = WAVES * (MODE == 0 ? gridDim.y : 1);
    const int per = (steps + parts - 1) / parts;
    const int s0 = min(((MODE == 0 ? (int)blockIdx.y * WAVES : 0) + w) * per, steps), n_real = min(steps - s0, per);
    const int n = (per + D - 1) / D * D;
    // Workgroups start at different places of their shares, the ones of an XCD one step apart: in step with each other
    // they would all ask for the same offset within a row of W at a time, and where the rows lie a multiple of 16 KB
    // apart, or 2752 k, that keeps part of the memory channels waiting (us, in step / rotated: N = 4096, 13 rows, K = 8192
    // 14.8 / 13.0, 11008 18.5 / 16.7, 16384 26.8 / 22.4, 22016 40.8 / 35.1; N = 12288, 32 rows, K = 8192 42.9 / 33.0; the
    // other K between 1024 and 28672 are the same within 2 %; but for the LM head, N = 32000, K = 4096, 1 row 38.6 / 40.8: one plane
    // of mode 0 is rotated for the first reason only)
    const int rot = n_real > 0 && (MODE != 0 || gridDim.y > 1 || K % 8192 == 0) ? (blk >> 3) % n_real : 0;

    __amdgpu_buffer_rsrc_t rs[NB][2];
    uint32_t vo[NB][2];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int hi = 0; hi < 2; ++hi) {
            const int base = __builtin_amdgcn_readfirstlane(stream_wrow<MODE>(ep, N, blk * NB + nb, hi));
            rs[nb][hi] = __builtin_amdgcn_make_buffer_rsrc((void*)(W + (size_t)base * K), 0, -1, 0x00020000);
            const int r = lane >> 3;
            const int lim = stream_last_row<MODE>(ep, N, hi) - base;
            // LDS position p of row r holds chunk p ^ r: the fragment reads below then spread over the banks
            vo[nb][hi] = (uint32_t)(min(r, max(lim, 0)) * K * 2 + ((lane & 7) ^ r) * 16);
        }
    bf16_t* ring = reinterpret_cast<bf16_t*>(smem) + w * (D * NB * 1024);
    typedef typename StreamMfma<AF16>::frag frag_t;
    const bf16_t* pa[MB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) pa[mb] = A + act_index(ep.a, min(mb * 16 + fr, M - 1), fq * 8);
    const size_t a_half = (size_t)4 * ep.a.chunk;          // elements from one 32-k half of a step to the next

    // requested before everything else
    bool normed = NORM && ep.nrm.ssq != nullptr;
    StreamNorm<MB * 16 / WAVES, (MB > 1)> norm;
    if (normed) norm.request(ep.nrm, M, w, lane);
    StreamEpilogue<MB, NB, WAVES, MODE, TO> epi;
    epi.request(ep, M, N, blk, t);

    frag_t fa[D][2 * MB];
#define RLHF_ST_ISSUE(STEP, J)                                                                                     \
    do {                                                                                                           \
        int ix_ = min((STEP), n_real - 1) + rot;                                                                   \
        ix_ -= ix_ >= n_real ? n_real : 0;                                                                         \
        const int st_ = s0 + max(ix_, 0);                                                                          \
        const int sc_ = min(st_, steps - 1);                                                                       \
        _Pragma("unroll") for (int nb = 0; nb < NB; ++nb) {                                                        \
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs[nb][0], (lds_ptr_t)(ring + ((J) * NB + nb) * 1024), 16,    \
                                                     vo[nb][0], sc_ * 128, 0, 2);                                  \
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs[nb][1], (lds_ptr_t)(ring + ((J) * NB + nb) * 1024 + 512), 16, \
                                                     vo[nb][1], sc_ * 128, 0, 2);                                  \
        }                                                                                                          \
        __builtin_amdgcn_sched_barrier(0);                                                                         \
        _Pragma("unroll") for (int mb = 0; mb < MB; ++mb) {                                                        \
            fa[J][2 * mb] = *reinterpret_cast<const frag_t*>(pa[mb] + (size_t)sc_ * 2 * a_half);                           \
            fa[J][2 * mb + 1] = *reinterpret_cast<const frag_t*>(pa[mb] + (size_t)sc_ * 2 * a_half + a_half);                  \
        }                                                                                                          \
        __builtin_amdgcn_sched_barrier(0);                                                                         \
    } while (0)
    f32x4_t acc[NB][MB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) acc[nb][mb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    // fragment reads: row fr of the block, chunk s * 4 + fq; rows 8.. of a block sit 1 KB further (128 bytes a row)
    const uint32_t lb = (uint32_t)(size_t)(lds_ptr_t)ring + fr * 128;
    const uint32_t l0 = lb + ((uint32_t)fq ^ (fr & 7)) * 16, l1 = lb + ((uint32_t)(4 + fq) ^ (fr & 7)) * 16;
#define RLHF_ST_CONSUME(STEP, J)                                                                                   \
    do {                                                                                                           \
        u32x4s_t wr_[NB][2];                                                                                       \
        _Pragma("unroll") for (int nb = 0; nb < NB; ++nb) {                                                        \
            asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(wr_[nb][0]) : "v"(l0), "n"(((J) * NB + nb) * 2048) : "memory"); \
            asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(wr_[nb][1]) : "v"(l1), "n"(((J) * NB + nb) * 2048) : "memory"); \
        }                                                                                                          \
        _Pragma("unroll") for (int nb = 0; nb < NB; ++nb)   /* the first one waits, the others only tie their registers to it */ \
            asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(wr_[nb][0]), "+v"(wr_[nb][1]) : : "memory");                \
        const bool live_ = (STEP) < n_real;                                                                        \
        _Pragma("unroll") for (int s = 0; s < 2; ++s)                                                              \
        _Pragma("unroll") for (int nb = 0; nb < NB; ++nb) {                                                        \
            u32x4s_t x_ = wr_[nb][s];                                                                              \
            if (AF16) {                                                                                            \
                x_[0] = bf16x2_to_f16x2(x_[0]); x_[1] = bf16x2_to_f16x2(x_[1]);                                    \
                x_[2] = bf16x2_to_f16x2(x_[2]); x_[3] = bf16x2_to_f16x2(x_[3]);                                    \
            }                                                                                                      \
            if (!live_) x_ = u32x4s_t{0, 0, 0, 0};                                                                 \
            const frag_t wf_ = *reinterpret_cast<const frag_t*>(&x_);                                              \
            _Pragma("unroll") for (int mb = 0; mb < MB; ++mb)                                                      \
                acc[nb][mb] = StreamMfma<AF16>::run(wf_, fa[J][2 * mb + s], acc[nb][mb]);                          \
        }                                                                                                          \
        __builtin_amdgcn_sched_barrier(0);                                                                         \
    } while (0)

#pragma unroll
    for (int j = 0; j < D; ++j) RLHF_ST_ISSUE(j, j);
    epi.request_table(ep, M, blk, t);
    if (normed) {
        const bool redo = norm.reduce(ep.nrm, M, K, w, lane, blk == 0, s_scale, s_inv);
        if (lane == 0) s_redo[w] = redo;
    }
    int k = 0;
    for (; k + D < n; k += D) {
#pragma unroll
        for (int j = 0; j < D; ++j) {
            wait_vmem<(D - 1) * OPS>();
            RLHF_ST_CONSUME(k + j, j);
            RLHF_ST_ISSUE(k + j + D, j);
        }
    }
#pragma unroll
    for (int j = 0; j < D; ++j) {                          // the last ring: nothing left to request
        if (j == D - 1) wait_vmem<0>();
        else if (j == D - 2) wait_vmem<OPS>();
        else if (j == D - 3) wait_vmem<2 * OPS>();
        else wait_vmem<3 * OPS>();
        RLHF_ST_CONSUME(k + j, j);
    }
    static_assert(D >= 2 && D <= 4 && (D - 1) * OPS < 64, "waits written out for up to four steps; vmcnt has six bits");
#undef RLHF_ST_ISSUE
#undef RLHF_ST_CONSUME

    // ---- the waves' shares of K meet in LDS: red[wave][weight row][activation row]
    float* red = reinterpret_cast<float*>(smem);
    auto put = [&] {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    red[(w * NB * 16 + nb * 16 + fq * 4 + e) * MP + mb * 16 + fr] = acc[nb][mb][e];
    };
    __syncthreads();
    [[maybe_unused]] const bool redo = NORM && AF16 && normed && lane < WAVES && s_redo[lane];
    put();
    if constexpr (NORM && AF16) {
        if (__builtin_expect(__any(redo), 0)) {            // all rows of the workgroup, from the residual stream
            normed = false;
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int mb = 0; mb < MB; ++mb) acc[nb][mb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
            for (int k32 = 0; k32 < 2 * n_real; ++k32) {
                const int kk = s0 * 64 + k32 * 32 + fq * 8;
                frag_t fx[MB];
#pragma unroll
                for (int mb = 0; mb < MB; ++mb) {
                    const int m = min(mb * 16 + fr, M - 1);
                    float hv[8], gv[8];
                    load8<float>(ep.nrm.h + (size_t)m * K + kk, hv);
                    load8<float>(ep.nrm.g + kk, gv);
#pragma unroll
                    for (int e = 0; e < 8; ++e) fx[mb][e] = (f16_t)(hv[e] * s_inv[m] * gv[e]);
                }
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    const int base = stream_wrow<MODE>(ep, N, blk * NB + nb, fr >> 3);
                    const int row = base + min(fr & 7, max(stream_last_row<MODE>(ep, N, fr >> 3) - base, 0));
                    u32x4s_t x = *reinterpret_cast<const u32x4s_t*>(W + (size_t)row * K + kk);
#pragma unroll
                    for (int e = 0; e < 4; ++e) x[e] = bf16x2_to_f16x2(x[e]);
#pragma unroll
                    for (int mb = 0; mb < MB; ++mb)
                        acc[nb][mb] = StreamMfma<AF16>::run(*reinterpret_cast<const frag_t*>(&x), fx[mb], acc[nb][mb]);
                }
            }
            put();
        }
    }
    __syncthreads();
    epi.finish(ep, red, s_scale, normed, C, M, N, blk, t);
#endif
}

// Float models: the same split and epilogues on float matrix instructions (16x16x4: products and sums in float), 16
// rows at a time (blockIdx.y).  These matrices fit the caches, so the time is that of one dependent chain: eight
// waves share K, a lane takes four consecutive k of its row and of its activation row per 16 k, four such
// loads ahead.  (8 rows of 256 x 256 .. 1376 weights: 2.5-3 us a launch, where 64 x 64 tiles took 6.9 us and
// left planes to rotary, SwiGLU and norm kernels of 3 us each.)  FEW: at most 64 partial sums of squares a row.
// GROUPS: more than 16 rows, so that pointers move by blockIdx.y; without it the 2-layer model of d = 256 generates 1 % faster.
template <int MODE, bool FEW, bool GROUPS>
__global__ __launch_bounds__(512) void k_gemm_stream_f32(const float* __restrict__ A, const float* __restrict__ W,
                                                         float* __restrict__ C, int M, int N, int K, const RowsEpi ep_in) {
    constexpr int WAVES = 8, U = 4, MP = 17;
    __shared__ float red[WAVES * 16 * MP];
    __shared__ float s_scale[16], s_inv[16];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6, fr = lane & 15, fq = lane >> 4, blk = blockIdx.x;
    RowsEpi ep = ep_in;
    if constexpr (GROUPS) {                                // everything that goes by rows moves along
        const int m0 = blockIdx.y * 16;
        M = min(M - m0, 16);
        A += (size_t)m0 * K;
        if (MODE == 0) C += (size_t)m0 * N;
        if (MODE == 1) ep.act = (float*)ep.act + (size_t)m0 * ep.ffn;
        if (MODE == 2) {
            RopeOut& ro = ep.ro;
            ro.pos += m0;
            if (ro.kv_dst) ro.kv_dst += m0;
            ro.q = (float*)ro.q + (size_t)m0 * ro.n_q_heads * ro.head_dim;
            if (ro.k) ro.k = (float*)ro.k + (size_t)m0 * ro.n_kv_heads * ro.head_dim;
            if (ro.v) ro.v = (float*)ro.v + (size_t)m0 * ro.n_kv_heads * ro.head_dim;
        }
        if (MODE == 3) {
            ep.res.h += (size_t)m0 * N;
            ep.res.x = (float*)ep.res.x + (size_t)m0 * N;
            ep.res.s += m0;
            ep.res.ssq += (size_t)m0 * kSsqStride;
        } else if (ep.nrm.ssq) {
            ep.nrm.ssq += (size_t)m0 * kSsqStride;
            ep.nrm.s_in += m0;
            if (ep.nrm.s_out) ep.nrm.s_out += m0;
        }
    }
    const bool normed = MODE != 3 && ep.nrm.ssq != nullptr;
    StreamNorm<2, FEW> norm;
    if (normed) norm.request(ep.nrm, M, w, lane);
    StreamEpilogue<1, 1, WAVES, MODE, float> epi;
    epi.request(ep, M, N, blk, t);
    const int hi = fr >> 3;
    const float* pw = W + (size_t)min(stream_wrow<MODE>(ep, N, blk, hi) + (fr & 7), stream_last_row<MODE>(ep, N, hi)) * K;
    const float* pa = A + (size_t)min(fr, M - 1) * K;
    const int chunks = (K + 15) / 16, per = (chunks + WAVES - 1) / WAVES;
    const int c0 = w * per, c1 = min(chunks, c0 + per);
    f32x4_t acc = f32x4_t{0.f, 0.f, 0.f, 0.f};
    for (int c = c0; c < c1; c += U) {
        float4 fw[U], fa[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {                      // past the share or past K: read in bounds, count as zero
            const int k = (c + u) * 16 + fq * 4, kc = min(k, K - 4);
            const float z = c + u < c1 && k < K ? 1.f : 0.f;
            fw[u] = *reinterpret_cast<const float4*>(pw + kc);
            fa[u] = *reinterpret_cast<const float4*>(pa + kc);
            if (z == 0.f) { fw[u] = make_float4(0.f, 0.f, 0.f, 0.f); fa[u] = fw[u]; }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(fw[u].x, fa[u].x, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(fw[u].y, fa[u].y, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(fw[u].z, fa[u].z, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(fw[u].w, fa[u].w, acc, 0, 0, 0);
        }
    }
    epi.request_table(ep, M, blk, t);
    if (normed) norm.reduce(ep.nrm, M, K, w, lane, blk == 0, s_scale, s_inv);     // float x: any jump fits
#pragma unroll
    for (int e = 0; e < 4; ++e) red[(w * 16 + fq * 4 + e) * MP + fr] = acc[e];
    __syncthreads();
    epi.finish(ep, red, s_scale, normed, C, M, N, blk, t);
}

namespace {

template <int MB, int NB, int WAVES, int D, bool AF16, bool NORM>
hipError_t stream_launch(hipStream_t st, int mode, int blocks, int nsplit, const bf16_t* a, const bf16_t* w, float* C,
                         int M, int N, int K, const RowsEpi& ep) {
    const dim3 grid(blocks, nsplit);
    switch (mode) {
        case 0: k_gemm_stream<MB, NB, WAVES, D, 0, AF16, NORM><<<grid, WAVES * 64, 0, st>>>(a, w, C, M, N, K, ep); break;
        case 1: k_gemm_stream<MB, NB, WAVES, D, 1, AF16, NORM><<<grid, WAVES * 64, 0, st>>>(a, w, C, M, N, K, ep); break;
        case 2: k_gemm_stream<MB, NB, WAVES, D, 2, AF16, NORM><<<grid, WAVES * 64, 0, st>>>(a, w, C, M, N, K, ep); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}
// mode 3: groups of 16 rows, each against the whole matrix
template <int NB, int WAVES, int D>
hipError_t stream_resid_launch(hipStream_t st, const bf16_t* a, const bf16_t* w, int M, int N, int K, const RowsEpi& ep) {
    k_gemm_stream<1, NB, WAVES, D, 3, true, false><<<dim3((N + 16 * NB - 1) / (16 * NB), 1, (M + 15) / 16), WAVES * 64, 0, st>>>(a, w, nullptr, M, N, K, ep);
    return hipGetLastError();
}
// modes 1 and 2 with the norm of 17..64 rows: one weight block per workgroup, eight waves share K
template <int MB>
hipError_t stream_norm_launch(hipStream_t st, int mode, const bf16_t* a, const bf16_t* w, int M, int N, int K, const RowsEpi& ep) {
    const int blocks = (N + 15) / 16;
    if (mode == 1) k_gemm_stream<MB, 1, 8, 2, 1, true, true><<<blocks, 512, 0, st>>>(a, w, nullptr, M, N, K, ep);
    else k_gemm_stream<MB, 1, 8, 2, 2, true, true><<<blocks, 512, 0, st>>>(a, w, nullptr, M, N, K, ep);
    return hipGetLastError();
}

}  // namespace

bool gemm_stream_supported(int wdt, int adt, int M, int K) {
    if (wdt == kF32) return adt == kF32 && M >= 1 && M <= kStreamF32Rows && K >= 4 && K % 4 == 0;
    return wdt == kBF16 && (adt == kF16 || (adt == kBF16 && M <= 16)) && M >= 1 && M <= kStreamMaxRows && K > 0 && K % 64 == 0;
}

// Every workgroup of 16 columns and 16 rows takes 0.0069 us of the chip per 512 k, and the launch at least a round trip of about
// 1.7 us for each 512 k of a wave's chain.  us, estimate / measured: N = 4096, K = 256 48 rows 8.3 / 7.7, 200 rows 26 / 26, 448 52 /
// 53; N = 32000, K = 768 32 rows 58 / 58, 448 776 / 767; N = 4096, K = 1024 33 rows 13.6 / 11.9, 300 70 / 68; N = 515, K = 256 448
// rows 9.4 / 9.7.
double stream_f32_us(int M, int N, int K) {
    const double its = (K + 511) / 512;
    return std::max(3. + 0.0069 * ((N + 15) / 16) * ((M + 15) / 16) * its, 2. + 1.7 * its);
}

// Shape of a launch: 16-row blocks of activations, of weights per workgroup (nb), ring depth (four waves throughout).
// Every workgroup reads all activation rows of its K range, from the L2, and the loads of a compute unit share one
// queue.  A compute unit's time goes with the 16 * nb weight rows of its workgroup plus about half the activation
// rows, which every workgroup reads again, and the launch takes as many rounds of 256 workgroups as it has: the
// least rounds * (2 nb + activation blocks) is the best shape, or within 4 % of it, for N = 2048 .. 57344 at K =
// 2048 .. 28672 and 13, 32, 64 rows (us, the former shape, now the one chosen: 32 rows N = 15360, K = 5120 38.4 28.1; N
// = 27648, K = 5120 60.5 46.7; N = 10240, K = 8192 41.7 30.9; N = 32000, K = 4096 47.8 43.1; 64 rows N = 57344, K = 8192
// 180.7 151.3, N = 32000, K = 8192 115.1 86.8; 13 rows N = 12288, K = 4096 17.8 17.1, N = 27648, K = 5120 50.1 44.8; N =
// 10240, K = 8192 32.1 27.8).  Among shapes a tenth apart the one with fewer blocks keeps the chip evenly loaded (13 rows
// N = 32000, K = 4096 two blocks 40.0, four 40.7, eight 41.2).  Up to 8 rows activations cost next to nothing and any
// shape that gives every compute unit its share reads at the rate of HBM (1 row, N = 12288 one, two, three blocks 16.3,
// 18.1, 16.8; N = 22016 28.8, 27.6, 28.7).
// With more than 16 rows O and down split K and leave planes to the norm that follows where that pays for the planes
// (32 rows: N = 5120, K = 13824 unsplit 37.0, three planes of four blocks 25.6; N = 4096, K = 4096 12.2, 8.5 as two of two;
// N = 8192, K = 28672 84.7, 77.9 as two of four).
// Four steps in flight where that does not add more than an eighth of surplus steps (one or two blocks, us, depth 2
// and 4: 1 row N = 12288 17.0 and 16.3; K = 1536, six steps a wave, 5.2 and 5.9), else two.
//
// 17..64 rows of a narrow residual stream (stream_resid: d_model <= 1024): the matrices come from the
// caches and a kernel's time is mostly its start and its chain of loads, so the five kernels of the norm
// form win over seven, with one weight block per workgroup and O and down in groups of 16 rows (d = 768,
// ffn = 2048, 64 rows, us: QKV 6.3 -> 6.7, O 4.5 -> 3.8, gate||up 7.9 -> 6.4, down 5.1 -> 4.9, two RMSNorms of
// 4.3 gone; O and down as one group of 64 rows 5.1 and 8.0).  Wider streams keep planes and RMSNorm: their
// time is weight traffic, which groups of 16 rows would repeat.  The head stays with the norm kernel (32000
// columns: 25 us against 19.6 + 4.3, and more registers).
constexpr int kStreamMaxBlocks = 8;
static int stream_rounds(int N, int nb, int ns) { return (((N + 16 * nb - 1) / (16 * nb)) * ns + 255) / 256; }
struct StreamShape { int mb, nb, depth; };
static StreamShape stream_shape(int M, int N, int K, int ns) {
    StreamShape sh{M <= 16 ? 1 : M <= 32 ? 2 : 4, 1, 2};
    auto cost = [&](int nb) { return stream_rounds(N, nb, ns) * (2 * nb + sh.mb); };
    if (M <= 8) {
        sh.nb = N >= 19200 ? 2 : 1;
    } else {
        int least = cost(1);
        for (int nb = 2; nb <= kStreamMaxBlocks; ++nb) least = least < cost(nb) ? least : cost(nb);
        while (cost(sh.nb) * 10 > least * 11) ++sh.nb;
    }
    const int per = ((K >> 6) + 4 * ns - 1) / (4 * ns);    // steps of a wave
    if ((sh.nb == 1 || (sh.nb == 2 && sh.mb == 1)) && (per <= 4 || (per + 3) / 4 * 4 * 8 <= per * 9)) sh.depth = 4;
    return sh;
}
bool takes_gemm_rows(int M, int d) { return M > kStreamMaxRows || (M > 32 && !stream_resid(kBF16, M, d) && d < 8192); }
bool stream_resid(int wdt, int M, int d) { return wdt == kF32 || M <= kStreamResidRows || (M <= kStreamMaxRows && d <= 1024); }
// The split with the least time, in steps of a compute unit as above; a plane more costs its write, and its read by
// the norm (about 1.3 us at 32 rows of 4096).
int gemm_stream_nsplit(int M, int N, int K, int max_split) {
    const int steps = K >> 6;
    int best = 1;
    long least = 0;
    for (int ns = 1; ns <= 8 && ns <= max_split && (ns == 1 || ns * 8 <= steps); ++ns) {
        const StreamShape sh = stream_shape(M, N, K, ns);
        const long c = (long)stream_rounds(N, sh.nb, ns) * (2 * sh.nb + sh.mb) * ((steps + ns - 1) / ns) + (ns - 1) * ((long)M * N >> 11);
        if (ns == 1 || c < least) { best = ns; least = c; }
    }
    return best;
}

hipError_t launch_gemm_stream(hipStream_t st, int wdt, int adt, int mode, const void* A, const void* W, float* C, int M,
                              int N, int K, const RowsEpi& ep_in, int nsplit, bool rows) {
    RowsEpi ep = ep_in;
    if (ep.a.row == 0) ep.a = ActLayout{K, 8};             // row-major unless the caller says otherwise
    if (ep.out.row == 0) ep.out = ActLayout{mode == 1 ? ep.ffn : N, 8};
    if (!(rows ? gemm_rows_supported(wdt, adt, M, K) : gemm_stream_supported(wdt, adt, M, K)) || N <= 0 || mode < 0 || mode > 3) return hipErrorInvalidValue;
    if (rows && (mode == 3 || ep.nrm.ssq)) return hipErrorInvalidValue;
    if ((long)8 * K * 2 >= (1L << 31)) return hipErrorInvalidValue;
    if (nsplit < 1 || (mode == 0 ? !C : nsplit != 1) || (nsplit > 1 && ep.nrm.ssq)) return hipErrorInvalidValue;
    if (mode == 1 && (!ep.act || ep.ffn <= 0 || N != 2 * ep.ffn || ep.ffn % 8)) return hipErrorInvalidValue;
    if (mode == 2) {
        const RopeOut& ro = ep.ro;
        if ((ro.head_dim != 64 && ro.head_dim != 128) || !ro.pos || !ro.table || !ro.q || (ro.pool && !ro.kv_dst) ||
            N != (ro.n_q_heads + 2 * ro.n_kv_heads) * ro.head_dim)
            return hipErrorInvalidValue;
    }
    if (ep.nrm.ssq && wdt == kBF16 && (adt != kF16 || !ep.nrm.h || !ep.nrm.g)) return hipErrorInvalidValue;
    if (ep.nrm.ssq && M > 16 && wdt != kF32 && (ep.nrm.n_ssq > 64 || mode == 0)) return hipErrorInvalidValue;
    if (rows) return mode == 1 && ep.ffn % 16 ? hipErrorInvalidValue : launch_gemm_rows(st, wdt, mode, A, W, C, M, N, K, ep, nsplit);
    if (mode == 3 && (adt == kBF16 || N % 16 || N > 16 * kSsqStride || !ep.res.h || !ep.res.g || !ep.res.x || !ep.res.s || !ep.res.ssq))
        return hipErrorInvalidValue;
    if (wdt == kF32) {
        if (nsplit != 1 || ep.a.row != K || (mode == 1 && ep.out.row != ep.ffn) || (mode == 3 && ep.out.row != N))
            return hipErrorInvalidValue;                   // row-major only
        const float *af = (const float*)A, *wf = (const float*)W;
        const dim3 grid((N + 15) / 16, (M + 15) / 16);
        const bool few = ep.nrm.ssq && ep.nrm.n_ssq <= 64;
#define RLHF_STREAM_F32(MODE, FEW)                                                                       \
    do {                                                                                                 \
        if (M <= 16) k_gemm_stream_f32<MODE, FEW, false><<<grid, 512, 0, st>>>(af, wf, C, M, N, K, ep);  \
        else k_gemm_stream_f32<MODE, FEW, true><<<grid, 512, 0, st>>>(af, wf, C, M, N, K, ep);           \
    } while (0)
        switch (mode) {
            case 0: if (few) RLHF_STREAM_F32(0, true); else RLHF_STREAM_F32(0, false); break;
            case 1: if (few) RLHF_STREAM_F32(1, true); else RLHF_STREAM_F32(1, false); break;
            case 2: if (few) RLHF_STREAM_F32(2, true); else RLHF_STREAM_F32(2, false); break;
            default: RLHF_STREAM_F32(3, false);
        }
#undef RLHF_STREAM_F32
        return hipGetLastError();
    }
    const bf16_t* a = (const bf16_t*)A;
    const bf16_t* w = (const bf16_t*)W;
    if (adt == kBF16) return stream_launch<1, 1, 4, 4, false, false>(st, mode, (N + 15) / 16, nsplit, a, w, C, M, N, K, ep);
    if (mode == 3) {
        if (M > 16) return stream_resid_launch<1, 8, 2>(st, a, w, M, N, K, ep);
        // two weight blocks where that saves a round (13 rows: N = 5120, K = 5120 12.7 us against 14.8, K = 13824 29.9 against 35.5)
        return stream_rounds(N, 2, 1) * 5 < stream_rounds(N, 1, 1) * 3 ? stream_resid_launch<2, 4, 4>(st, a, w, M, N, K, ep)
                                                                      : stream_resid_launch<1, 4, 4>(st, a, w, M, N, K, ep);
    }
    if (ep.nrm.ssq && M > 16)
        return M <= 32 ? stream_norm_launch<2>(st, mode, a, w, M, N, K, ep) : stream_norm_launch<4>(st, mode, a, w, M, N, K, ep);
    const StreamShape sh = stream_shape(M, N, K, nsplit);
    const int blocks = (N + 16 * sh.nb - 1) / (16 * sh.nb);
#define RLHF_STREAM(MB, NB, D)                       \
    if (sh.mb == MB && sh.nb == NB && sh.depth == D) \
        return stream_launch<MB, NB, 4, D, true, MB == 1>(st, mode, blocks, nsplit, a, w, C, M, N, K, ep)
#define RLHF_STREAM_MB(MB)                                                                                               \
    RLHF_STREAM(MB, 1, 4); RLHF_STREAM(MB, 1, 2); RLHF_STREAM(MB, 2, 2); RLHF_STREAM(MB, 3, 2); RLHF_STREAM(MB, 4, 2); \
    RLHF_STREAM(MB, 5, 2); RLHF_STREAM(MB, 6, 2); RLHF_STREAM(MB, 7, 2); RLHF_STREAM(MB, 8, 2)
    RLHF_STREAM_MB(1);
    RLHF_STREAM(1, 2, 4);
    RLHF_STREAM_MB(2);
    RLHF_STREAM_MB(4);
#undef RLHF_STREAM_MB
#undef RLHF_STREAM
    return hipErrorInvalidValue;
}

}  // namespace rlhf
