// The compute-bound GEMM of prefill and scoring passes: 256 x 256 output tiles, K in tiles of 64, both
// operands global -> LDS directly, eight waves in two groups that take turns on the matrix units.
//
// What bounds it is keeping the matrix units fed: a K tile is 2048 cycles of MFMA per SIMD, and the LDS
// reads (192 KB) and direct loads (64 KB, at most 59 bytes per cycle and compute unit) it takes would
// stop them for half as long again if the two waves of a SIMD did them at the same time, which is what a
// kernel with one barrier per K tile drifts into (1.06-1.20 PFLOP/s at 8192 rows of the 7B shapes).
// Here a K tile is four phases, one per quadrant of the wave's output, each a memory part (fragment
// reads, two direct loads, the waits) and a matrix part (16 MFMAs), with a barrier after either; waves
// 4..7 (on the same SIMDs as 0..3) run one part behind, so that on every SIMD one wave computes while
// the other fetches.  Without that offset the same code is 17 % slower (1.39 -> 1.18 PFLOP/s on QKV).
// A tile's operands lie in LDS as halves of 128 rows (A0, A1, W0, W1), two tiles deep.  Half h of tile
// t + 2 is requested in the phase after that half of tile t has been read, so that six halves (12
// loads per wave) stay in flight: "vmcnt(12)" at the end of every memory part covers what the next
// phase reads, and the count never drops to zero before the last tile.  Every quadrant needs one new
// half, because the order of W's halves alternates from tile to tile: (A0,Wf) (A0,Ws) (A1,Ws) (A1,Wf).
// Measured, M = 8192, half weights: QKV 1.16 -> 1.39, O 1.24 -> 1.41, gate||up 1.13 -> 1.32, down 1.17 ->
// 1.47 PFLOP/s (float output); random operands and this power budget cap a register-only MFMA loop at
// 1.8.  Requesting before reading is 2-4 % slower; wave priorities, and waiting for the fragments after
// the barrier instead of before, change nothing.
//
// The order of accumulation over K is that of a plain loop, 32 at a time.
#include "common.h"
#include "kernels.h"
#include "tile_walk.h"
#include <type_traits>

namespace rlhf {

namespace {

template <bool AF16> struct TallMfma;
template <> struct TallMfma<false> {
    typedef bf16x8_t frag;
    static __device__ __forceinline__ f32x4_t run(frag a, frag b, f32x4_t c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
    }
};
template <> struct TallMfma<true> {
    typedef f16x8_t frag;
    static __device__ __forceinline__ f32x4_t run(frag a, frag b, f32x4_t c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
    }
};

typedef __attribute__((address_space(3))) void* lds_ptr_t;
typedef uint32_t u32x4t_t __attribute__((ext_vector_type(4)));

// s_waitcnt vmcnt(N) lgkmcnt(0), at the end of a memory part
template <int N> __device__ __forceinline__ void wait_part() { asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" : : "n"(N) : "memory"); }

// Neighbouring quarter waves swap one packed fragment each: p0 and p1 are four consecutive 16-bit
// columns each, 16 apart; afterwards an even quarter holds eight consecutive columns of the first group,
// an odd one of the second.
[[maybe_unused]] __device__ __forceinline__ uint4 swap_quarters(uint2 p0, uint2 p1, bool odd) {
    const uint2 give = odd ? p0 : p1;
    uint2 got;
    got.x = (uint32_t)__shfl_xor((int)give.x, 16, kWave);
    got.y = (uint32_t)__shfl_xor((int)give.y, 16, kWave);
    return odd ? make_uint4(got.x, got.y, p1.x, p1.y) : make_uint4(p0.x, p0.y, got.x, got.y);
}

template <bool AF16> __device__ __forceinline__ uint2 pack4(const float (&o)[4]) {
    uint2 pk;
    if (AF16) {
        fp16x2_t a = {(__fp16)o[0], (__fp16)o[1]}, b = {(__fp16)o[2], (__fp16)o[3]};
        pk.x = *reinterpret_cast<uint32_t*>(&a);
        pk.y = *reinterpret_cast<uint32_t*>(&b);
    } else {
        pk.x = (uint32_t)f32_to_bf16(o[0]) | ((uint32_t)f32_to_bf16(o[1]) << 16);
        pk.y = (uint32_t)f32_to_bf16(o[2]) | ((uint32_t)f32_to_bf16(o[3]) << 16);
    }
    return pk;
}

}  // namespace

// AF16: half activations (else bf16).  CVT: W is bf16 and the activations half: weight fragments are
// converted after their LDS read, one phase ahead of their use, under the reads of the next A half.
// EPI: what becomes of the tile.
//   kTallPlain   C float [M, N] (plane blockIdx.y when K is split)
//   kTallAdd     C float [M, N] += the tile: O and down projections finish the residual stream, and RMSNorm reads
//                one array instead of two and writes none back (8000 x 4096: RMSNorm 73 -> 38 us, O and down +5 to +15 us)
//   kTallSwiglu  W = gate||up [2f, K], N = 2f; W0 holds 128 gate rows, W1 the matching up rows;
//                C = act [M, f], 16-bit
//   kTallRope64, kTallRope128  W = QKV; W0 holds the first halves of the tile's heads, W1 the second, so a
//                lane has both members of its rotary pairs; q, k, v and the paged pool are written
//   kTallLse     W = LM head; per row two (max, sum of exp) partials a tile and the target's logit
enum TallEpi { kTallPlain, kTallAdd, kTallSwiglu, kTallRope64, kTallRope128, kTallLse };

template <bool AF16, bool CVT, TallEpi EPI>
__global__ __launch_bounds__(512, 2) void k_gemm_tall(const bf16_t* __restrict__ A, const bf16_t* __restrict__ W,
                                                      float* __restrict__ C, int M, int N, int K, int kchunk,
                                                      int tiles_m, int tiles_n, const RopeOut ro, const LseOut lo) {
#if defined(__HIP_DEVICE_COMPILE__)                        // buffer resources exist in the device pass only
    static_assert(!CVT || AF16, "conversion is for half activations");
    constexpr int HD = EPI == kTallRope128 ? 128 : 64, HALF = HD / 2;
    constexpr bool ROPE = EPI == kTallRope64 || EPI == kTallRope128;
    __shared__ __attribute__((aligned(16))) bf16_t sA[2][2][128 * 64];
    __shared__ __attribute__((aligned(16))) bf16_t sB[2][2][128 * 64];
    int tm, tn;
    if (!xcd_tile_of(blockIdx.x, tiles_m, tiles_n, tm, tn)) return;
    const int m0 = tm * 256, n0 = tn * 256;
    const int kbeg = blockIdx.y * kchunk, nk = (min(K, kbeg + kchunk) - kbeg) >> 6;
    const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wm = w >> 2, wn = w & 3, fr = lane & 15, fq = lane >> 4;

    // operand bases of this tile (64-bit); a lane's byte offsets below them fit 32 bits, rows past the end clamped
    const int f = N >> 1, oc0 = tn * 128;
    __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc((void*)(A + (size_t)m0 * K + kbeg), 0, -1, 0x00020000);
    __amdgpu_buffer_rsrc_t rb[2];
    uint32_t oa[2][2], ob[2][2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int b_row = EPI == kTallSwiglu ? h * f + oc0 : n0;
        rb[h] = __builtin_amdgcn_make_buffer_rsrc((void*)(W + (size_t)b_row * K + kbeg), 0, -1, 0x00020000);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            // a load fills 8 LDS rows of 64; position p of a row holds chunk p ^ (row / 2 % 8), so that the
            // fragment reads (16 rows, one chunk) spread over the banks
            const int r = (w * 2 + i) * 8 + (lane >> 3), c = (lane & 7) ^ ((r >> 1) & 7);
            const int br = EPI == kTallSwiglu ? min(r, f - 1 - oc0)
                           : ROPE ? min((r / HALF) * HD + h * HALF + r % HALF, N - 1 - n0)
                                  : min(h * 128 + r, N - 1 - n0);
            oa[h][i] = (uint32_t)((min(h * 128 + r, M - 1 - m0) * K + c * 8) * 2);
            ob[h][i] = (uint32_t)((br * K + c * 8) * 2);
        }
    }
#define RLHF_T_ISSUE_A(H, BUF, T)                                                                                     \
    do {                                                                                                              \
        _Pragma("unroll") for (int i = 0; i < 2; ++i) __builtin_amdgcn_raw_ptr_buffer_load_lds(                       \
            ra, (lds_ptr_t)&sA[BUF][H][(w * 2 + i) * 512], 16, oa[H][i], (T) * 128, 0, 0);                            \
    } while (0)
#define RLHF_T_ISSUE_B(H, BUF, T)                                                                                     \
    do {                                                                                                              \
        _Pragma("unroll") for (int i = 0; i < 2; ++i) __builtin_amdgcn_raw_ptr_buffer_load_lds(                       \
            rb[H], (lds_ptr_t)&sB[BUF][H][(w * 2 + i) * 512], 16, ob[H][i], (T) * 128, 0, 0);                         \
    } while (0)
    // fragment reads: wave (wm, wn) takes rows wm * 64 .. of an A half and wn * 32 .. of a W half
    const uint32_t xr = (fr >> 1) & 7;
    const uint32_t pa0 = (uint32_t)(size_t)(lds_ptr_t)&sA[0][0][0] + (wm * 64 + fr) * 128;
    const uint32_t pb0 = (uint32_t)(size_t)(lds_ptr_t)&sB[0][0][0] + (wn * 32 + fr) * 128;
    const uint32_t pa[2] = {pa0 + ((uint32_t)fq ^ xr) * 16, pa0 + ((uint32_t)(4 + fq) ^ xr) * 16};
    const uint32_t pb[2] = {pb0 + ((uint32_t)fq ^ xr) * 16, pb0 + ((uint32_t)(4 + fq) ^ xr) * 16};
    typedef typename TallMfma<AF16>::frag frag;
    u32x4t_t fa[2][4], fb[2][2][2];                        // [32-k step][16 rows], [half][step][16 rows]
    f32x4_t acc[2][2][4][2];                               // [A half][W half][16 rows][16 columns]
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int m = 0; m < 4; ++m)
#pragma unroll
                for (int n = 0; n < 2; ++n) acc[i][j][m][n] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    // reads and waits are written out: the compiler, seeing an LDS read after a direct load, waits for all of them
#define RLHF_T_READ(DST, ADDR, OFF) asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(DST) : "v"(ADDR), "n"(OFF) : "memory")
#define RLHF_T_READ_A(H, BUF)                                                                                         \
    do {                                                                                                              \
        _Pragma("unroll") for (int s = 0; s < 2; ++s) _Pragma("unroll") for (int m = 0; m < 4; ++m)                   \
            RLHF_T_READ(fa[s][m], pa[s], (BUF) * 32768 + (H) * 16384 + m * 2048);                                     \
    } while (0)
#define RLHF_T_READ_B(H, BUF)                                                                                         \
    do {                                                                                                              \
        _Pragma("unroll") for (int s = 0; s < 2; ++s) _Pragma("unroll") for (int n = 0; n < 2; ++n)                   \
            RLHF_T_READ(fb[H][s][n], pb[s], (BUF) * 32768 + (H) * 16384 + n * 2048);                                  \
    } while (0)
    // ties fragment registers to the wait in front of it
#define RLHF_T_TIE_A                                                                                                  \
    asm volatile("" : "+v"(fa[0][0]), "+v"(fa[0][1]), "+v"(fa[0][2]), "+v"(fa[0][3]), "+v"(fa[1][0]), "+v"(fa[1][1]), \
                 "+v"(fa[1][2]), "+v"(fa[1][3]))
#define RLHF_T_TIE_B(H) asm volatile("" : "+v"(fb[H][0][0]), "+v"(fb[H][0][1]), "+v"(fb[H][1][0]), "+v"(fb[H][1][1]))
#define RLHF_T_CVT_B(H)                                                                                               \
    do {                                                                                                              \
        if (CVT) {                                                                                                    \
            _Pragma("unroll") for (int s = 0; s < 2; ++s) _Pragma("unroll") for (int n = 0; n < 2; ++n)               \
            _Pragma("unroll") for (int e = 0; e < 4; ++e) fb[H][s][n][e] = bf16x2_to_f16x2(fb[H][s][n][e]);           \
            RLHF_T_TIE_B(H);                                                                                          \
        }                                                                                                             \
    } while (0)
#define RLHF_T_MMA(I, J)                                                                                              \
    do {                                                                                                              \
        _Pragma("unroll") for (int s = 0; s < 2; ++s) _Pragma("unroll") for (int m = 0; m < 4; ++m)                   \
        _Pragma("unroll") for (int n = 0; n < 2; ++n)                                                                 \
            acc[I][J][m][n] = TallMfma<AF16>::run(*reinterpret_cast<const frag*>(&fb[J][s][n]),                       \
                                                  *reinterpret_cast<const frag*>(&fa[s][m]), acc[I][J][m][n]);        \
        __builtin_amdgcn_sched_barrier(0);                                                                            \
    } while (0)
#define RLHF_T_BAR                                                                                                    \
    do {                                                                                                              \
        __builtin_amdgcn_sched_barrier(0);                                                                            \
        __builtin_amdgcn_s_barrier();                                                                                 \
        __builtin_amdgcn_sched_barrier(0);                                                                            \
    } while (0)
    // end of a memory part: loads of the last two tiles are requested without successors, so fewer may stay in flight
#define RLHF_T_WAIT(N_BEFORE_LAST, N_LAST)                                                                            \
    do {                                                                                                              \
        if (more) wait_part<12>();                                                                                    \
        else if (kt + 1 < nk) wait_part<N_BEFORE_LAST>();                                                             \
        else wait_part<N_LAST>();                                                                                     \
    } while (0)
    // One K tile.  BF: W half of the first quadrant (the tile's parity).  With CVT the second W half is read along
    // with A0 (so it has to be there one part earlier) and converted in the second part.  The fourth part reads the
    // next tile's first W half (after the last tile: something that nobody uses).
#define RLHF_T_TILE(BF, MORE)                                                                                         \
    do {                                                                                                              \
        constexpr int BUF = BF, BS = 1 - BF;                                                                          \
        const bool more = MORE;                                                                                       \
        RLHF_T_READ_A(0, BUF);                                                                                        \
        if (CVT) RLHF_T_READ_B(BS, BUF);                                                                              \
        if (more) RLHF_T_ISSUE_B(BF, BUF, kt + 2);                                                                    \
        RLHF_T_CVT_B(BF);                                                                                             \
        RLHF_T_WAIT(10, 2); RLHF_T_TIE_A; if (CVT) RLHF_T_TIE_B(BS);                                                  \
        RLHF_T_BAR; RLHF_T_MMA(0, BF); RLHF_T_BAR;                                                                    \
        if (!CVT) RLHF_T_READ_B(BS, BUF);                                                                             \
        if (more) RLHF_T_ISSUE_A(0, BUF, kt + 2);                                                                     \
        RLHF_T_CVT_B(BS);                                                                                             \
        RLHF_T_WAIT(8, 0); RLHF_T_TIE_B(BS);                                                                          \
        RLHF_T_BAR; RLHF_T_MMA(0, BS); RLHF_T_BAR;                                                                    \
        RLHF_T_READ_A(1, BUF);                                                                                        \
        if (more) RLHF_T_ISSUE_B(BS, BUF, kt + 2);                                                                    \
        RLHF_T_WAIT(6, 0); RLHF_T_TIE_A;                                                                              \
        RLHF_T_BAR; RLHF_T_MMA(1, BS); RLHF_T_BAR;                                                                    \
        RLHF_T_READ_B(BS, 1 - BUF);                                                                                   \
        if (more) RLHF_T_ISSUE_A(1, BUF, kt + 2);                                                                     \
        if (CVT && more) wait_part<10>();                                                                             \
        else RLHF_T_WAIT((CVT ? 2 : 4), 0);                                                                           \
        RLHF_T_TIE_B(BS);                                                                                             \
        RLHF_T_BAR; RLHF_T_MMA(1, BF); RLHF_T_BAR;                                                                    \
    } while (0)
    {
        const int t1 = nk > 1 ? 1 : 0;                     // a single tile: requested twice, so that the counts hold
        RLHF_T_ISSUE_B(0, 0, 0); RLHF_T_ISSUE_A(0, 0, 0); RLHF_T_ISSUE_B(1, 0, 0); RLHF_T_ISSUE_A(1, 0, 0);
        RLHF_T_ISSUE_B(1, 1, t1); RLHF_T_ISSUE_A(0, 1, t1); RLHF_T_ISSUE_B(0, 1, t1); RLHF_T_ISSUE_A(1, 1, t1);
    }
    asm volatile("s_waitcnt vmcnt(%0)" : : "n"(CVT ? 10 : 12) : "memory");
    RLHF_T_BAR;
    RLHF_T_READ_B(0, 0);
    asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");
    RLHF_T_TIE_B(0);
    RLHF_T_BAR;                                            // everybody has read W0: the first phase requests it anew
    if (w >= 4) RLHF_T_BAR;                                // the second group runs one part behind
    int kt = 0;
    for (; kt + 4 <= nk; kt += 2) {                        // successors for certain: no branches between the parts
        RLHF_T_TILE(0, true);
        ++kt;
        RLHF_T_TILE(1, true);
        --kt;
    }
    for (;;) {
        RLHF_T_TILE(0, kt + 2 < nk);
        if (++kt >= nk) break;
        RLHF_T_TILE(1, kt + 2 < nk);
        if (++kt >= nk) break;
    }
    if (w < 4) RLHF_T_BAR;
#undef RLHF_T_ISSUE_A
#undef RLHF_T_ISSUE_B
#undef RLHF_T_READ
#undef RLHF_T_READ_A
#undef RLHF_T_READ_B
#undef RLHF_T_TIE_A
#undef RLHF_T_TIE_B
#undef RLHF_T_CVT_B
#undef RLHF_T_MMA
#undef RLHF_T_BAR
#undef RLHF_T_TILE
#undef RLHF_T_WAIT

    // ---- epilogues.  acc[i][j][m][n][e]: row m0 + i*128 + wm*64 + m*16 + fr; column (of W half j)
    // wn*32 + n*16 + fq*4 + e
    typedef typename std::conditional<AF16, f16_t, bf16_t>::type TO;
    const bool odd = fq & 1;
    if constexpr (EPI == kTallPlain) {
        float* Cs = C + (size_t)blockIdx.y * M * N;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const int gm = m0 + i * 128 + wm * 64 + m * 16 + fr;
                if (gm >= M) continue;
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int n = 0; n < 2; ++n) {
                        const int gn = n0 + j * 128 + wn * 32 + n * 16 + fq * 4;
                        const f32x4_t v = acc[i][j][m][n];
                        float* dst = Cs + (size_t)gm * N + gn;
                        if (gn + 3 < N && (N & 3) == 0) {
                            *reinterpret_cast<float4*>(dst) = make_float4(v[0], v[1], v[2], v[3]);
                        } else {
#pragma unroll
                            for (int e = 0; e < 4; ++e)
                                if (gn + e < N) dst[e] = v[e];
                        }
                    }
            }
    }
    if constexpr (EPI == kTallAdd) {                       // N % 4 == 0
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            float4 old[4][2][2];                           // requested together: the stores might alias later loads
#pragma unroll
            for (int m = 0; m < 4; ++m)
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int n = 0; n < 2; ++n) {
                        const int gm = min(m0 + i * 128 + wm * 64 + m * 16 + fr, M - 1);
                        const int gn = min(n0 + j * 128 + wn * 32 + n * 16 + fq * 4, N - 4);
                        old[m][j][n] = *reinterpret_cast<const float4*>(C + (size_t)gm * N + gn);
                    }
#pragma unroll
            for (int m = 0; m < 4; ++m)
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int n = 0; n < 2; ++n) {
                        const int gm = m0 + i * 128 + wm * 64 + m * 16 + fr, gn = n0 + j * 128 + wn * 32 + n * 16 + fq * 4;
                        const f32x4_t v = acc[i][j][m][n];
                        const float4 o = old[m][j][n];
                        if (gm < M && gn < N)
                            *reinterpret_cast<float4*>(C + (size_t)gm * N + gn) = make_float4(o.x + v[0], o.y + v[1], o.z + v[2], o.w + v[3]);
                    }
        }
    }
    if constexpr (EPI == kTallSwiglu) {
        uint16_t* act = reinterpret_cast<uint16_t*>(C);
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const int gm = m0 + i * 128 + wm * 64 + m * 16 + fr;
                uint2 p[2];
#pragma unroll
                for (int n = 0; n < 2; ++n) {
                    float o[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float g = acc[i][0][m][n][e];
                        o[e] = g / (1.f + __expf(-g)) * acc[i][1][m][n][e];
                    }
                    p[n] = pack4<AF16>(o);
                }
                const uint4 pk = swap_quarters(p[0], p[1], odd);
                const int oc = oc0 + wn * 32 + (odd ? 16 : 0) + (fq & 2) * 4;
                if (gm < M && oc < f) *reinterpret_cast<uint4*>(act + (size_t)gm * f + oc) = pk;   // f % 8 == 0
            }
    }
    if constexpr (ROPE) {
        TO* q_out = reinterpret_cast<TO*>(ro.q);
        TO* k_out = reinterpret_cast<TO*>(ro.k);
        TO* v_out = reinterpret_cast<TO*>(ro.v);
        TO* pool = reinterpret_cast<TO*>(ro.pool);
        const int Hq = ro.n_q_heads, Hkv = ro.n_kv_heads;
        const size_t head_stride = (size_t)ro.page_tokens * HD;
        // positions, then the cosines and sines of four rows at a time, requested together: left to the compiler
        // every row's loads wait behind the stores of the row before (the pointers might alias)
        int pos[2][4], slot[2][4];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const int gm = min(m0 + i * 128 + wm * 64 + m * 16 + fr, M - 1);
                pos[i][m] = ro.pos[gm];
                slot[i][m] = pool ? ro.kv_dst[gm] : 0;
            }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            float4 tb[4][2][2];
#pragma unroll
            for (int m = 0; m < 4; ++m)
#pragma unroll
                for (int n = 0; n < 2; ++n) {
                    const int k = (wn * 32 + n * 16 + fq * 4) % HALF;
                    const float* tab = ro.table + (size_t)pos[i][m] * HD + 2 * k;
                    tb[m][n][0] = *reinterpret_cast<const float4*>(tab);
                    tb[m][n][1] = *reinterpret_cast<const float4*>(tab + 4);
                }
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const int gm = m0 + i * 128 + wm * 64 + m * 16 + fr;
                const bool row_ok = gm < M;
                TO* prow = nullptr;                        // this token's K row of head 0 in the pool
                if (pool)
                    prow = pool + ((size_t)(slot[i][m] / ro.page_tokens) * ro.n_layers + ro.layer) * 2 * (size_t)Hkv * ro.page_tokens * HD +
                           (size_t)(slot[i][m] % ro.page_tokens) * HD;
                uint2 p[2][2];                             // [pair half][n]
#pragma unroll
                for (int n = 0; n < 2; ++n) {
                    const int cc = wn * 32 + n * 16 + fq * 4, head = n0 / HD + cc / HALF;
                    float a[4], b[4];
                    const float4 t0 = tb[m][n][0], t1 = tb[m][n][1];
                    const float cs[4] = {t0.x, t0.z, t1.x, t1.z}, sn[4] = {t0.y, t0.w, t1.y, t1.w};
                    const bool rot = head < Hq + Hkv;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float x = acc[i][0][m][n][e], y = acc[i][1][m][n][e];
                        a[e] = rot ? x * cs[e] - y * sn[e] : x;
                        b[e] = rot ? x * sn[e] + y * cs[e] : y;
                    }
                    p[0][n] = pack4<AF16>(a);
                    p[1][n] = pack4<AF16>(b);
                }
                const int cc = wn * 32 + (odd ? 16 : 0) + (fq & 2) * 4, head = n0 / HD + cc / HALF;
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const uint4 pk = swap_quarters(p[j][0], p[j][1], odd);
                    const int c = j * HALF + cc % HALF;
                    if (!row_ok || head >= Hq + 2 * Hkv) continue;
                    if (head < Hq) {
                        *reinterpret_cast<uint4*>(q_out + ((size_t)gm * Hq + head) * HD + c) = pk;
                    } else {
                        const bool is_k = head < Hq + Hkv;
                        const int kh = is_k ? head - Hq : head - Hq - Hkv;
                        TO* dst = is_k ? k_out : v_out;
                        if (dst) *reinterpret_cast<uint4*>(dst + ((size_t)gm * Hkv + kh) * HD + c) = pk;
                        if (prow)
                            *reinterpret_cast<uint4*>(prow + (is_k ? 0 : (size_t)Hkv * head_stride) + kh * head_stride + c) = pk;
                    }
                }
            }
        }
    }
    if constexpr (EPI == kTallLse) {
        float2* red = reinterpret_cast<float2*>(&sA[0][0][0]);       // [4 column groups][256 rows] (max, sum)
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const int lr = i * 128 + wm * 64 + m * 16 + fr, gm = m0 + lr;
                int tgt = -1;
                if (gm < M) tgt = min(max(lo.tokens[lo.target_idx[gm]], 0), N - 1);
                float mx = -INFINITY;
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int n = 0; n < 2; ++n)
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const int gn = n0 + j * 128 + wn * 32 + n * 16 + fq * 4 + e;
                            const float z = acc[i][j][m][n][e];
                            if (gn < N) mx = fmaxf(mx, z);
                            if (gn == tgt) lo.tgt[gm] = z;
                        }
                mx = fmaxf(mx, __shfl_xor(mx, 16, kWave));
                mx = fmaxf(mx, __shfl_xor(mx, 32, kWave));
                float se = 0.f;
                if (mx > -INFINITY) {
#pragma unroll
                    for (int j = 0; j < 2; ++j)
#pragma unroll
                        for (int n = 0; n < 2; ++n)
#pragma unroll
                            for (int e = 0; e < 4; ++e)
                                if (n0 + j * 128 + wn * 32 + n * 16 + fq * 4 + e < N) se += __expf(acc[i][j][m][n][e] - mx);
                }
                se += __shfl_xor(se, 16, kWave);
                se += __shfl_xor(se, 32, kWave);
                if (fq == 0) red[wn * 256 + lr] = make_float2(mx, se);
            }
        __syncthreads();
        const int lr = t & 255, p = t >> 8, gm = m0 + lr;
        if (gm < M) {
            const float2 x = red[(2 * p) * 256 + lr], y = red[(2 * p + 1) * 256 + lr];
            const float mx = fmaxf(x.x, y.x);
            float se = 0.f;
            if (x.x > -INFINITY) se += x.y * __expf(x.x - mx);
            if (y.x > -INFINITY) se += y.y * __expf(y.x - mx);
            lo.part_max[(size_t)gm * lo.n_part + tn * 2 + p] = mx;
            lo.part_sum[(size_t)gm * lo.n_part + tn * 2 + p] = se;
        }
    }
#endif
}

namespace {

template <TallEpi EPI>
hipError_t tall_launch(hipStream_t st, int wdt, int adt, const void* A, const void* W, void* C, int M, int N, int K,
                       int nsplit, const RopeOut& ro, const LseOut& lo) {
    const int tiles_m = (M + 255) / 256, tiles_n = (N + 255) / 256;
    const int kchunk = ((K + nsplit - 1) / nsplit + 63) / 64 * 64;
    if ((long)(nsplit - 1) * kchunk >= K) return hipErrorInvalidValue;        // a split without a K range
    if (256L * K * 2 >= (1L << 32)) return hipErrorInvalidValue;              // offsets inside a tile are 32-bit
    const dim3 grid(xcd_grid(tiles_m, tiles_n), nsplit);
#define RLHF_TALL(AF, CV)                                                                                              \
    k_gemm_tall<AF, CV, EPI><<<grid, 512, 0, st>>>((const bf16_t*)A, (const bf16_t*)W, (float*)C, M, N, K, kchunk, tiles_m, \
                                                   tiles_n, ro, lo)
    if (adt == kBF16) {
        if constexpr (EPI == kTallAdd) return hipErrorInvalidValue;           // the stage's activations are half
        else RLHF_TALL(false, false);
    } else if (wdt == kF16) RLHF_TALL(true, false);
    else RLHF_TALL(true, true);
#undef RLHF_TALL
    return hipGetLastError();
}

}  // namespace

bool gemm_tall_supported(int wdt, int adt, int K) {
    return K > 0 && K % 64 == 0 && ((wdt == kBF16 && (adt == kBF16 || adt == kF16)) || (wdt == kF16 && adt == kF16));
}

hipError_t launch_gemm_tall(hipStream_t st, int wdt, int adt, const void* A, const void* W, float* C, int M, int N, int K,
                            int nsplit) {
    if (M <= 0 || N <= 0) return hipSuccess;
    if (!gemm_tall_supported(wdt, adt, K) || nsplit < 1) return hipErrorInvalidValue;
    return tall_launch<kTallPlain>(st, wdt, adt, A, W, C, M, N, K, nsplit, RopeOut{}, LseOut{});
}

hipError_t launch_gemm_tall_add(hipStream_t st, int wdt, int adt, const void* A, const void* W, float* h, int M, int N, int K) {
    if (M <= 0 || N <= 0) return hipSuccess;
    if (!gemm_tall_supported(wdt, adt, K) || N % 4) return hipErrorInvalidValue;
    return tall_launch<kTallAdd>(st, wdt, adt, A, W, h, M, N, K, 1, RopeOut{}, LseOut{});
}

hipError_t launch_gemm_tall_swiglu(hipStream_t st, int wdt, int adt, const void* A, const void* W, void* act, int M, int ffn,
                                   int K) {
    if (!gemm_tall_supported(wdt, adt, K) || M <= 0 || ffn <= 0 || ffn % 8) return hipErrorInvalidValue;
    return tall_launch<kTallSwiglu>(st, wdt, adt, A, W, act, M, 2 * ffn, K, 1, RopeOut{}, LseOut{});
}

// ---- tall passes with the consumer in the epilogue

static bool rope_shape_ok(int wdt, int adt, int M, int K, int head_dim) {
    return (wdt == kBF16 || wdt == kF16) && half_weights_ok(wdt, adt, K) && (adt == kF16 || adt == kBF16) && M > 256 &&
           K % 64 == 0 && (head_dim == 64 || head_dim == 128);
}

// Below 512 rows the launch cannot split K, and up to 128 tiles (half a round of workgroups) a split launch with the
// rotary kernel behind it is the faster one, us, bf16 weights, 300 rows: N = 2304 19 against 29, 6144 33 against 53, 12288
// 69 against 98, 15360 88 against 117; N = 24576 (192 tiles) 202 against 206, half weights 181 against 167.
bool gemm_rope_supported(int wdt, int adt, int M, int K, const Dims& dm) {
    const long N = ((long)dm.n_q_heads + 2L * dm.n_kv_heads) * dm.head_dim;
    return rope_shape_ok(wdt, adt, M, K, dm.head_dim) && (M >= 512 || ((M + 255) / 256) * ((N + 255) / 256) > 128);
}

hipError_t launch_gemm_rope(hipStream_t st, int wdt, int adt, const void* A, const void* Wqkv, int M, int K,
                            const RopeOut& ro) {
    if (!rope_shape_ok(wdt, adt, M, K, ro.head_dim) || !ro.pos || !ro.table || !ro.q || (ro.pool && !ro.kv_dst))
        return hipErrorInvalidValue;
    const int N = (ro.n_q_heads + 2 * ro.n_kv_heads) * ro.head_dim;
    if (!half_operands_ok(wdt, M, N, K)) return hipErrorInvalidValue;
    return ro.head_dim == 128 ? tall_launch<kTallRope128>(st, wdt, adt, A, Wqkv, nullptr, M, N, K, 1, ro, LseOut{})
                              : tall_launch<kTallRope64>(st, wdt, adt, A, Wqkv, nullptr, M, N, K, 1, ro, LseOut{});
}

bool gemm_lse_supported(int wdt, int adt, int K) {
    return (wdt == kBF16 || wdt == kF16) && half_weights_ok(wdt, adt, K) && (adt == kF16 || adt == kBF16) && K % 64 == 0;
}

int gemm_lse_partials(int N) { return (N + 255) / 256 * 2; }

hipError_t launch_gemm_lse(hipStream_t st, int wdt, int adt, const void* A, const void* W_head, int M, int N, int K,
                           const LseOut& lo) {
    if (M <= 0) return hipSuccess;
    if (!gemm_lse_supported(wdt, adt, K) || N <= 0 || !lo.tokens || !lo.target_idx || !lo.part_max || !lo.part_sum ||
        !lo.tgt || lo.n_part != gemm_lse_partials(N) || !half_operands_ok(wdt, M, N, K))
        return hipErrorInvalidValue;
    return tall_launch<kTallLse>(st, wdt, adt, A, W_head, nullptr, M, N, K, 1, RopeOut{}, lo);
}

// The tile a workgroup of such a launch takes (host copy of the device mapping, for tests).
int gemm_tall_grid(int tiles_m, int tiles_n) { return xcd_grid(tiles_m, tiles_n); }
bool gemm_tall_tile(int bid, int tiles_m, int tiles_n, int* tm, int* tn) { return xcd_tile_of(bid, tiles_m, tiles_n, *tm, *tn); }

}  // namespace rlhf
