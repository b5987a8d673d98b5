// C[m][n] = sum_k A[m][k] * W[n][k]   (activations times a row-major weight matrix, y = W x)
//
// bf16 weights: LDS-tiled MFMA kernel (v_mfma_f32_16x16x32_{bf16,f16}, float accumulate).
// Activations are half (what the stage uses for bf16 models) or bf16; for half the bf16 weight
// chunks are converted to half, exactly, between the global load and the LDS store.  One
// template serves the decode regime (few rows: the weight matrix streams from HBM once, split
// along K so that enough workgroups are in flight to saturate bandwidth) and the prefill /
// scoring regime (thousands of rows: compute-bound 256x256 tiles).  Global loads are 16 bytes per lane,
// consecutive lanes along K; tiles sit in LDS with an XOR swizzle of the 16-byte chunk index
// so that the MFMA-fragment reads (16 rows x one chunk per quarter wave) spread over the banks.
// Split-K partials are written to separate buffers and summed by the consumer kernel, which
// keeps the result deterministic (no float atomics).
//
// fp32 with a K split: a plain LDS-tiled kernel (not tuned; unsplit launches run on gemm_f32.hip).
#include "common.h"
#include "kernels.h"
#include "tile_walk.h"
#include <algorithm>

namespace rlhf {

// 16-byte chunk swizzle inside an LDS tile row: the fragment read of a quarter wave takes one
// chunk column of 16 consecutive rows; XOR-ing the chunk index with row bits spreads those 16
// reads over all banks (rows of 128 bytes: two rows per 256-byte bank sweep; rows of 64 bytes:
// four).
template <int TK> __device__ __forceinline__ int swz(int row, int chunk) {
    return TK == 64 ? (chunk ^ ((row >> 1) & 7)) : (chunk ^ ((row >> 2) & 3));
}

template <bool AF16> struct Mfma;
template <> struct Mfma<false> {
    typedef bf16x8_t frag;
    static __device__ __forceinline__ f32x4_t run(frag a, frag b, f32x4_t c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
    }
};
template <> struct Mfma<true> {
    typedef f16x8_t frag;
    static __device__ __forceinline__ f32x4_t run(frag a, frag b, f32x4_t c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
    }
};

// Tile index of a workgroup.  Few-row launches (XCD == false) walk the N tiles in order, the
// row tiles of a column tile next to each other so that its weights are fetched once; the others as
// tile_walk.h says.
template <bool XCD>
__device__ __forceinline__ bool tile_of(int bid, int tiles_m, int tiles_n, int& tm, int& tn) {
    if (XCD) return xcd_tile_of(bid, tiles_m, tiles_n, tm, tn);
    tn = bid / tiles_m;
    tm = bid - tn * tiles_m;
    return true;
}

// A: 16-bit activations (bf16 if !AF16, half if AF16); W: bf16.
// TM x TN output tile per workgroup of WM x WN waves; each wave owns (TM/WM) x (TN/WN), built
// from 16x16 MFMA fragments; K advances in LDS tiles of TK (32 or 64) elements, double-buffered.
//
// SWIGLU: W is a gate||up matrix [2f, K] (gate rows, then up rows) and N = 2f.  The tile's
// columns alternate, in blocks of 16, between gate rows and the matching up rows, so that a
// lane ends up with gate and up of the same output column in neighbouring fragments; the
// epilogue writes act = silu(gate) * up as 16-bit [M, f] (of the activation type) to C and the
// float [M, 2f] intermediate never exists.
template <int TM, int TN, int TK, int WM, int WN, bool AF16, bool XCD, bool SWIGLU>
__global__ __launch_bounds__(WM * WN * 64) void k_gemm_bf16(const bf16_t* __restrict__ A,
                                                           const bf16_t* __restrict__ W,
                                                           float* __restrict__ C, int M, int N, int K,
                                                           int kchunk, int tiles_m, int tiles_n) {
    constexpr int NT = WM * WN * 64;
    constexpr int FM = TM / WM / 16, FN = TN / WN / 16;
    constexpr int CH = TK / 8;                            // 16-byte chunks per tile row
    constexpr int A_CH = TM * CH, B_CH = TN * CH;
    constexpr int A_IT = (A_CH + NT - 1) / NT, B_IT = (B_CH + NT - 1) / NT;
    __shared__ __attribute__((aligned(16))) bf16_t sA[2][TM * TK];
    __shared__ __attribute__((aligned(16))) bf16_t sB[2][TN * TK];

    int tm, tn;
    if (!tile_of<XCD>(blockIdx.x, tiles_m, tiles_n, tm, tn)) return;
    const int m0 = tm * TM, n0 = tn * TN;
    const int split = blockIdx.y;
    const int kbeg = split * kchunk;
    const int kend = min(K, kbeg + kchunk);
    const int nk = (kend - kbeg + TK - 1) / TK;

    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int wm = w / WN, wn = w - wm * WN;

    uint4 ra[A_IT], rb[B_IT];
    auto gload = [&](int kt) {
        const int k0 = kbeg + kt * TK;
#pragma unroll
        for (int i = 0; i < A_IT; ++i) {
            const int idx = t + i * NT;
            const int row = idx / CH, c = idx % CH;
            const int gm = m0 + row, gk = k0 + c * 8;
            ra[i] = make_uint4(0, 0, 0, 0);
            if (idx < A_CH && gm < M && gk < kend)
                ra[i] = *reinterpret_cast<const uint4*>(A + (size_t)gm * K + gk);
        }
#pragma unroll
        for (int i = 0; i < B_IT; ++i) {
            const int idx = t + i * NT;
            const int row = idx / CH, c = idx % CH;
            int gn = n0 + row;
            bool ok = gn < N;
            if (SWIGLU) {      // tile column -> gate row (even 16-blocks) or up row (odd) of out col
                const int oc = (n0 >> 1) + (row >> 5) * 16 + (row & 15);
                ok = oc < (N >> 1);
                gn = ((row >> 4) & 1) * (N >> 1) + oc;
            }
            const int gk = k0 + c * 8;
            rb[i] = make_uint4(0, 0, 0, 0);
            if (idx < B_CH && ok && gk < kend) {
                if (XCD) {
                    rb[i] = *reinterpret_cast<const uint4*>(W + (size_t)gn * K + gk);
                } else {
                    // few-row launches read every weight once: stream them past the caches (evict first), so
                    // that a tall GEMM on the other stream keeps its tiles in the L2 they share
                    typedef uint32_t u32x4v __attribute__((ext_vector_type(4)));
                    const u32x4v v = __builtin_nontemporal_load(reinterpret_cast<const u32x4v*>(W + (size_t)gn * K + gk));
                    rb[i] = make_uint4(v[0], v[1], v[2], v[3]);
                }
            }
        }
    };
    auto sstore = [&](int buf) {
#pragma unroll
        for (int i = 0; i < A_IT; ++i) {
            const int idx = t + i * NT;
            const int row = idx / CH, c = idx % CH;
            if (idx < A_CH)
                *reinterpret_cast<uint4*>(&sA[buf][row * TK + swz<TK>(row, c) * 8]) = ra[i];
        }
#pragma unroll
        for (int i = 0; i < B_IT; ++i) {
            const int idx = t + i * NT;
            const int row = idx / CH, c = idx % CH;
            if (AF16) {   // bf16 -> half once per element per workgroup (exact in half's normal range)
                rb[i].x = bf16x2_to_f16x2(rb[i].x); rb[i].y = bf16x2_to_f16x2(rb[i].y);
                rb[i].z = bf16x2_to_f16x2(rb[i].z); rb[i].w = bf16x2_to_f16x2(rb[i].w);
            }
            if (idx < B_CH)
                *reinterpret_cast<uint4*>(&sB[buf][row * TK + swz<TK>(row, c) * 8]) = rb[i];
        }
    };

    f32x4_t acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    const int fr = lane & 15, fq = lane >> 4;
    auto compute = [&](int buf) {
#pragma unroll
        for (int s = 0; s < TK / 32; ++s) {
            typename Mfma<AF16>::frag fa[FM], fb[FN];
            const int c = s * 4 + fq;
#pragma unroll
            for (int i = 0; i < FM; ++i) {
                const int row = wm * (TM / WM) + i * 16 + fr;
                fa[i] = *reinterpret_cast<const typename Mfma<AF16>::frag*>(&sA[buf][row * TK + swz<TK>(row, c) * 8]);
            }
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                const int row = wn * (TN / WN) + j * 16 + fr;
                fb[j] = *reinterpret_cast<const typename Mfma<AF16>::frag*>(&sB[buf][row * TK + swz<TK>(row, c) * 8]);
            }
            // weights are the MFMA "A" operand: D[i = n][j = m], so a lane ends up holding four
            // consecutive n of one row m and stores them as one float4.
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j)
                    acc[i][j] = Mfma<AF16>::run(fb[j], fa[i], acc[i][j]);
        }
    };
    if (nk > 0) {
        gload(0);
        sstore(0);
    }
    __syncthreads();
    for (int kt = 0; kt < nk; ++kt) {
        const int buf = kt & 1;
        if (kt + 1 < nk) gload(kt + 1);
        compute(buf);
        if (kt + 1 < nk) sstore(buf ^ 1);
        __syncthreads();
    }

    if (SWIGLU) {
        static_assert(!SWIGLU || (FN % 4 == 0), "gate and up fragments come in pairs, pairs are stored two at a time");
        const int f = N >> 1;
        uint16_t* act = reinterpret_cast<uint16_t*>(C);
        const bool odd = fq & 1;
#pragma unroll
        for (int i = 0; i < FM; ++i) {
            const int m = m0 + wm * (TM / WM) + i * 16 + fr;
            // silu(gate) * up of fragment pair (j, j + 1): four consecutive output columns in 8 bytes
            auto packed = [&](int j) {
                float o[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float g = acc[i][j][e];
                    o[e] = g / (1.f + __expf(-g)) * acc[i][j + 1][e];
                }
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
            };
            // Two fragment pairs cover 32 consecutive output columns; neighbouring quarter waves swap
            // one of them each, so that a lane stores eight consecutive columns (16 bytes).
#pragma unroll
            for (int j = 0; j < FN; j += 4) {
                const uint2 p0 = packed(j), p1 = packed(j + 2);
                const uint2 give = odd ? p0 : p1;
                uint2 got;
                got.x = (uint32_t)__shfl_xor((int)give.x, 16, kWave);
                got.y = (uint32_t)__shfl_xor((int)give.y, 16, kWave);
                const uint4 pk = odd ? make_uint4(got.x, got.y, p1.x, p1.y) : make_uint4(p0.x, p0.y, got.x, got.y);
                const int oc = (n0 >> 1) + ((wn * (TN / WN) + (odd ? j + 2 : j) * 16) >> 1) + (fq & 2) * 4;
                if (m >= M || oc >= f) continue;       // f is a multiple of 8: a group of 8 is in or out
                *reinterpret_cast<uint4*>(act + (size_t)m * f + oc) = pk;
            }
        }
        return;
    }
    float* Cs = C + (size_t)split * M * N;
#pragma unroll
    for (int i = 0; i < FM; ++i) {
        const int m = m0 + wm * (TM / WM) + i * 16 + fr;
        if (m >= M) continue;
#pragma unroll
        for (int j = 0; j < FN; ++j) {
            const int n = n0 + wn * (TN / WN) + j * 16 + fq * 4;
            float* dst = Cs + (size_t)m * N + n;
            if (n + 3 < N && (N & 3) == 0) {
                *reinterpret_cast<float4*>(dst) =
                    make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (n + e < N) dst[e] = acc[i][j][e];
            }
        }
    }
}

// ------------------------------------------------------------------------------ fp32 path
// 64x64 tile, K step 16, 256 threads each computing a 4x4 block.
__global__ __launch_bounds__(256) void k_gemm_f32(const float* __restrict__ A,
                                                  const float* __restrict__ W,
                                                  float* __restrict__ C, int M, int N, int K,
                                                  int kchunk, int tiles_n) {
    __shared__ float sA[16][64 + 4];
    __shared__ float sB[16][64 + 4];
    const int tile = blockIdx.x;
    const int tm = tile / tiles_n, tn = tile - tm * tiles_n;
    const int m0 = tm * 64, n0 = tn * 64;
    const int split = blockIdx.y;
    const int kbeg = split * kchunk, kend = min(K, kbeg + kchunk);
    const int t = threadIdx.x;
    const int ty = t >> 4, tx = t & 15;        // 16 x 16 threads, 4 x 4 outputs each
    const int lr = t >> 2, lc = (t & 3) * 4;   // loader: row 0..63, k offset 0,4,8,12
    float acc[4][4] = {};
    for (int k0 = kbeg; k0 < kend; k0 += 16) {
        float4 va = make_float4(0, 0, 0, 0), vb = make_float4(0, 0, 0, 0);
        if (m0 + lr < M && k0 + lc < kend)
            va = *reinterpret_cast<const float4*>(A + (size_t)(m0 + lr) * K + k0 + lc);
        if (n0 + lr < N && k0 + lc < kend)
            vb = *reinterpret_cast<const float4*>(W + (size_t)(n0 + lr) * K + k0 + lc);
        __syncthreads();
        sA[lc + 0][lr] = va.x; sA[lc + 1][lr] = va.y; sA[lc + 2][lr] = va.z; sA[lc + 3][lr] = va.w;
        sB[lc + 0][lr] = vb.x; sB[lc + 1][lr] = vb.y; sB[lc + 2][lr] = vb.z; sB[lc + 3][lr] = vb.w;
        __syncthreads();
#pragma unroll
        for (int kk = 0; kk < 16; ++kk) {
            float a[4], b[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) { a[i] = sA[kk][ty * 4 + i]; b[i] = sB[kk][tx * 4 + i]; }
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[i][j] += a[i] * b[j];
        }
    }
    float* Cs = C + (size_t)split * M * N;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int m = m0 + ty * 4 + i;
        if (m >= M) continue;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int n = n0 + tx * 4 + j;
            if (n < N) Cs[(size_t)m * N + n] = acc[i][j];
        }
    }
}

// ----------------------------------------------------------------------------- dispatch
namespace {
// Tilings.  Variants 1-4 stream the weights for few rows (split along K); 5-7 are the
// compute-bound tilings of prefill / scoring passes.  Measured at M = 8192 on the 7B layer
// shapes (half activations): 5: 650-820, 6: 800-900, 7: 950-1050 TFLOP/s (7 is gemm_tall.hip since, wherever K is a
// multiple of 64: 1320-1470 with half weights, 1080-1200 with bf16).  Tried and dropped:
// 256x256 with four 128x128 wave tiles (750-830), global loads two tiles ahead (no change: L2
// latency is already hidden), fragment loads software-pipelined against the MFMAs (-5 %),
// 256x256 with 32-wide K tiles (half the LDS and fewer registers, so that a decode workgroup fits
// beside it on a compute unit: 740-890 alone, no net gain for the fused stage).  For up to 64
// rows, 64-column tiles (20-32 KB of LDS, 52-72 registers) stream as fast as or slightly faster
// than 128-column ones (36-48 KB, 68-108) and fit beside a 256x256 workgroup on a compute unit;
// 32-wide K tiles (64-byte row pieces) are slower.
struct TileCfg { int variant, tm, tn, tk; bool xcd; };
constexpr TileCfg kCfgs[] = {
    {0, 0, 0, 0, false},
    {1, 16, 64, 64, false}, {2, 32, 64, 64, false}, {3, 64, 64, 64, false}, {4, 128, 128, 64, false},
    {5, 128, 128, 64, true}, {6, 256, 128, 32, true}, {7, 256, 256, 64, true},
    {8, 64, 16, 64, false},      // k_gemm_stream (gemm_stream.hip): few rows, whole K range per workgroup (no split)
};
constexpr int kNumCfgs = sizeof(kCfgs) / sizeof(kCfgs[0]);

// K split of the 128 x 128 tiles.  Every split writes a float plane of M x N that the consumer reads back, which at
// these M is no longer small beside the weights: the split that minimises (weight bytes + plane bytes) / (share of
// the chip in use), 384 workgroups filling it.
int split_128(int M, int N, int K, int max_split) {
    const long tiles = (long)((M + 127) / 128) * ((N + 127) / 128);
    const int kmax = K / 256 > 0 ? K / 256 : 1;                   // keep >= 4 K tiles per split
    const double wbytes = 2.0 * N * K, plane = 8.0 * M * N;
    double best = 0;
    int ns = 1;
    for (int c = 1; c <= kmax && c <= max_split; c *= 2) {
        const double fill = (double)(tiles * c) / 384.0;
        const double cost = (wbytes + plane * c) / (fill < 1.0 ? fill : 1.0);
        if (c == 1 || cost < best) { best = cost; ns = c; }
    }
    return ns;
}

// Few rows: the smallest row tile that holds them, weights streamed once, K split.  Many rows: the tall
// kernel.  In between, and for narrow matrices, 128 x 128 tiles with K split.
// K split of the tall kernel (gemm_tall.hip), 0 where another tiling is the better one.
// 129..256 rows of a large matrix: one row of tiles, K split so that the tiles times the splits come
// close to, and never exceed, one workgroup per compute unit (a second round costs more than it adds:
// 7B QKV at 256 rows 36 us with 4 splits, 62 with 6), eight at most (down 41 us with 8, 37 with 12 and
// 47 with 16, but every plane costs its reader 1 us).
// More rows: the kernel and split with the least cost.  Up to 511 rows, or N below 4096:
//   tall        rounds * (1.1 us a K tile + 11) and 8 bytes of plane at 6.5 TB/s an output; unsplit it finishes the
//               residual stream: 16 instead of 11, 4 bytes.  A round is 32 workgroups on the XCD that has most: tile
//               columns are dealt to the XCDs (tile_walk.h), so that N = 1280 has 160 compute units, N = 1024 128.
//   128 x 128   512 workgroups a round, two a compute unit: 1.3 us a K tile and 5.5, 1.15 in a last round of at
//               most 256; planes as above.  Taken where it is 5 % cheaper (it reads bf16 weights only).
// (Fitted to 257..16384 rows of N = 512..2048, O and down with the RMSNorm behind them, to 6 %; over those and
// 257..511 rows of QKV and gate||up at N = 1536..57344 the choice is 2 % above the best measured on average and at
// most 1 % above 128 x 128 with its split.  300 rows of N = K = 1536: 20.7 us with 128 x 128 and 4 splits, 26.5
// tall; 8192 rows of N = 1280, K = 3456: 170 against 120 tall, 109 with half weights.)  Up to N = 1024 the tall
// kernel, with half the compute units or fewer, never wins (16384 rows of N = 1024: 117 against 103).
// From 512 rows and N = 4096 on: a workgroup takes about 1.15 us per K tile and 4 us besides, one per compute
// unit at a time, and a plane is written and read once at about 5 TB/s; the split with the least sum, if that is
// a tenth below the unsplit launch (which finishes the residual stream itself and leaves no planes).
// N = 4096: 1024 rows 47 us with 2 splits (128 x 128 tiles: 65), 2048 rows 58 with 2 (77 unsplit), 4160 rows 156
// unsplit, though its second round is nearly empty (128 x 128 tiles: 270).
int tall_nsplit(int M, int N, int K, int max_split) {
    if (K % 64 || M <= 128) return 0;
    const long tiles = (long)((M + 255) / 256) * ((N + 255) / 256);
    const int steps = K / 64;
    int ns = 1;
    if (M <= 256) {
        if ((long)N * K < 40L * 1000 * 1000) return 0;
        ns = (int)(256 / tiles);
        if (ns > steps / 4) ns = steps / 4;      // at least four K tiles per split
        if (ns > 8) ns = 8;
        if (ns > max_split) ns = max_split;
        if (ns < 1 || tiles * ns < 120) return 0;
    } else if (N < 4096 || M < 512) {
        if (N <= 1024) return 0;
        const double plane = 8.0 * M * N / 6.5e6;
        const long per_xcd = (long)((M + 255) / 256) * xcd_cols((N + 255) / 256);
        double best = 0;
        for (int c : {1, 2, 3, 4, 6, 8}) {
            if (c > max_split || c > (steps + 3) / 4 || (c - 1) * ((steps + c - 1) / c) >= steps) continue;
            const double rounds = (double)((per_xcd * c + 31) / 32);
            const double us = c == 1 ? rounds * (steps * 1.1 + 16.0) + plane / 2
                                     : rounds * (((steps + c - 1) / c) * 1.1 + 11.0) + plane * c;
            if (c == 1 || us < best) { best = us; ns = c; }
        }
        const int n4 = split_128(M, N, K, max_split), s4 = (steps + n4 - 1) / n4;
        const long wgs = (long)((M + 127) / 128) * ((N + 127) / 128) * n4, full = wgs / 512, rest = wgs % 512;
        const double us4 = full * (s4 * 1.3 + 5.5) + (rest ? s4 * (rest <= 256 ? 1.15 : 1.3) + 5.5 : 0.0) + plane * n4;
        if (us4 * 1.05 < best) return 0;
    } else {
        double best = 0;
        for (int c = 1; c <= 8 && c <= max_split && c <= (steps + 3) / 4; ++c) {
            const double rounds = (double)((tiles * c + 255) / 256);
            const double us = rounds * (((steps + c - 1) / c) * 1.15 + 4.0) + (c == 1 ? 0.0 : 8.0 * M * N * c / 5e6);
            if (c == 1 || us < best) { best = c == 1 ? 0.9 * us : us; ns = c; }
        }
    }
    while (ns > 1) {                             // every split gets a K range
        const int kchunk = ((K + ns - 1) / ns + 63) / 64 * 64;
        if ((long)(ns - 1) * kchunk < K) break;
        --ns;
    }
    return ns;
}

int pick_variant(int M, int N, int K, int nsplit = 0) {
    if (M <= 16) return 1;
    if (M <= 32) return 2;
    if (M <= 64) return 3;
    if (K % 64 == 0 && M >= 512 && N >= 4096) return 7;
    if (K % 64 == 0 || M <= 256) return nsplit > 0 && tall_nsplit(M, N, K, nsplit) == nsplit ? 7 : 4;
    const long tiles = (long)((M + 255) / 256) * ((N + 255) / 256);
    const long rounds = (tiles + 255) / 256;            // one 256 x 256 tile per compute unit at a time
    return tiles * 10 >= rounds * 256 * 6 ? 7 : 4;      // at least 60 % of the tile slots filled
}
constexpr int kTargetBlocks = 1024;      // about four workgroups per compute unit (tiles of up to 64 rows)
}  // namespace

// True when launch_gemm would run the 256 x 256 tiling for this shape and split (the shapes for
// which a half copy of the weights, if there is one, is the better operand).
bool gemm_is_tall(int M, int N, int K, int nsplit) { return K % 64 == 0 && kCfgs[pick_variant(M, N, K, nsplit)].xcd; }

// bf16 -> IEEE half, element by element (round toward zero; exact in half's normal range, values
// below 2^-14 land on half's subnormal grid): the same conversion the kernels apply on the fly.
// Bound by memory: 16 bytes a lane, four loads in flight (N = 22016, K = 4096, read and written: 78 us with 4 bytes a lane,
// 73.5 this way; a device copy of as much takes 68).
__global__ __launch_bounds__(256) void k_bf16_to_half(const uint32_t* __restrict__ src, uint32_t* __restrict__ dst, size_t n_pairs) {
    const size_t n4 = n_pairs >> 2, stride = (size_t)gridDim.x * 256, t = (size_t)blockIdx.x * 256 + threadIdx.x;
    constexpr int U = 4;
    for (size_t i = t; i < n4; i += U * stride) {
        uint4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (i + u * stride < n4) v[u] = reinterpret_cast<const uint4*>(src)[i + u * stride];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (i + u * stride < n4)
                reinterpret_cast<uint4*>(dst)[i + u * stride] = make_uint4(bf16x2_to_f16x2(v[u].x), bf16x2_to_f16x2(v[u].y),
                                                                           bf16x2_to_f16x2(v[u].z), bf16x2_to_f16x2(v[u].w));
    }
    if (t < (n_pairs & 3)) dst[n4 * 4 + t] = bf16x2_to_f16x2(src[n4 * 4 + t]);
}
__global__ __launch_bounds__(256) void k_bf16_to_half_unaligned(const uint16_t* __restrict__ src, uint16_t* __restrict__ dst, size_t n) {
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256)
        dst[i] = (uint16_t)bf16x2_to_f16x2(src[i]);
}
hipError_t launch_bf16_to_half(hipStream_t st, const void* src, void* dst, size_t n) {
    if (n == 0) return hipSuccess;
    if (n % 2) return hipErrorInvalidValue;
    if (((uintptr_t)src | (uintptr_t)dst) & 15)            // a caller's tensor may start anywhere
        k_bf16_to_half_unaligned<<<4096, 256, 0, st>>>((const uint16_t*)src, (uint16_t*)dst, n);
    else
        k_bf16_to_half<<<(unsigned)std::min<size_t>(4096, (n / 8 + 1023) / 1024 + 1), 256, 0, st>>>((const uint32_t*)src, (uint32_t*)dst, n / 2);
    return hipGetLastError();
}

// Float planes against the unsplit kernel of gemm_f32.hip, which also finishes rotary, SwiGLU or the residual stream.  Planes:
// 0.065 us a k of a split, more from about 512 workgroups on, and a plane is written and read.  us, unsplit / planes with
// their reading: N = K = 1024 64 rows 31 / 7, 512 rows 37 / 22; N = 11008, K = 2048 256 rows 122 / 176, 64 rows 62 / 54;
// N = K = 4096 512 rows 174 / 238, 256 rows 142 / 133; N = 4096, K = 256 448 rows 15 / 24.
static double f32_planes_us(int M, int N, int K, int ns) {
    const double wgs = (double)((M + 63) / 64) * ((N + 63) / 64) * ns;
    return 3. + (double)((K + ns - 1) / ns) * std::max(0.065, 0.01 + 1.02e-4 * wgs) + 8. * M * N * ns / 5e6;
}

int gemm_choose_nsplit(int wdt, int M, int N, int K, int max_split) {
    int tm, tn, kgran;
    if (wdt == kBF16) {
        const int tall = tall_nsplit(M, N, K, max_split);
        if (tall > 0) return tall;
        const TileCfg& c = kCfgs[pick_variant(M, N, K)];
        if (c.xcd) return 1;
        tm = c.tm; tn = c.tn; kgran = c.tk;
    } else { tm = 64; tn = 64; kgran = 16; }
    const long tiles = (long)((M + tm - 1) / tm) * ((N + tn - 1) / tn);
    const int kmax = K / (4 * kgran) > 0 ? K / (4 * kgran) : 1;   // keep >= 4 K tiles per split
    int ns;
    if (tm >= 128) {
        ns = split_128(M, N, K, max_split);
    } else {
        ns = (int)((kTargetBlocks + tiles - 1) / tiles);
    }
    if (ns > kmax) ns = kmax;
    if (ns > max_split) ns = max_split;
    if (ns < 1) ns = 1;
    // a split that would get no K range is pointless: shrink until every split is non-empty
    while (ns > 1) {
        int kchunk = ((K + ns - 1) / ns + kgran - 1) / kgran * kgran;
        if ((long)(ns - 1) * kchunk < K) break;
        --ns;
    }
    if (wdt == kF32 && ns > 1 && gemm_f32_tall_us(M, N, K) < f32_planes_us(M, N, K, ns)) ns = 1;
    return ns;
}

double gemm_f32_us(int M, int N, int K) {
    const int ns = gemm_choose_nsplit(kF32, M, N, K, 16);
    return ns > 1 ? f32_planes_us(M, N, K, ns) : gemm_f32_tall_us(M, N, K);
}

template <bool AF16>
static hipError_t launch_bf16(hipStream_t st, int variant, const bf16_t* a, const bf16_t* w, float* C, int M,
                              int N, int K, int nsplit) {
    const TileCfg& c = kCfgs[variant];
    const int tiles_m = (M + c.tm - 1) / c.tm, tiles_n = (N + c.tn - 1) / c.tn;
    const int kchunk = ((K + nsplit - 1) / nsplit + c.tk - 1) / c.tk * c.tk;
    int blocks = tiles_m * tiles_n;
    if (c.xcd) blocks = xcd_grid(tiles_m, tiles_n);
    dim3 grid(blocks, nsplit);
#define RLHF_GEMM(TM, TN, TK, WM, WN, XCD)                                                            \
    k_gemm_bf16<TM, TN, TK, WM, WN, AF16, XCD, false><<<grid, WM * WN * 64, 0, st>>>(a, w, C, M, N, K, kchunk, \
                                                                                     tiles_m, tiles_n)
    switch (variant) {
        case 1: RLHF_GEMM(16, 64, 64, 1, 4, false); break;
        case 2: RLHF_GEMM(32, 64, 64, 1, 4, false); break;
        case 3: RLHF_GEMM(64, 64, 64, 2, 2, false); break;
        case 4: RLHF_GEMM(128, 128, 64, 2, 2, false); break;
        case 8: {
            if (M > 16 || K % 256 || (K / 64) % (4 * nsplit)) return hipErrorInvalidValue;
            return launch_gemm_stream(st, kBF16, AF16 ? kF16 : kBF16, 0, a, w, C, M, N, K, RowsEpi{}, nsplit);
        }
        case 5: RLHF_GEMM(128, 128, 64, 2, 2, true); break;
        case 6: RLHF_GEMM(256, 128, 32, 2, 2, true); break;
        case 7:                                                  // gemm_tall.hip, unless K leaves a remainder or a split without a range
            if (K % 64 == 0 && (long)(nsplit - 1) * kchunk < K) return launch_gemm_tall(st, kBF16, AF16 ? kF16 : kBF16, a, w, C, M, N, K, nsplit);
            RLHF_GEMM(256, 256, 64, 4, 2, true);
            break;
        default: return hipErrorInvalidValue;
    }
#undef RLHF_GEMM
    return hipGetLastError();
}

static bool swiglu_shape_ok(int wdt, int adt, int M, int ffn, int K) {
    return (wdt == kBF16 || wdt == kF16) && half_weights_ok(wdt, adt, K) && (adt == kF16 || adt == kBF16) && M > 256 &&
           ffn % 8 == 0 && K % 8 == 0;
}

// Below 448 rows the fused launch has to have more than half a round of tiles, as in gemm_rope_supported; its epilogue is
// the lighter one, so that from 448 on it is level with the others at few tiles too.  us, bf16 weights, 300 / 511 rows,
// fused and best other: N = 4096 24 and 20 / 24 and 25, 8192 39 and 31 / 39 and 35, 16384 69 and 59 / 71 and 65;
// N = 22016 (172 tiles) 95 and 104 / 94 and 109.
bool gemm_swiglu_supported(int wdt, int adt, int M, int ffn, int K) {
    return swiglu_shape_ok(wdt, adt, M, ffn, K) &&
           (M >= 512 || (K % 64 == 0 && (M >= 448 || (M + 255) / 256 * ((2L * ffn + 255) / 256) > 128)));
}

hipError_t launch_gemm_swiglu(hipStream_t st, int wdt, int adt, const void* A, const void* W_gate_up,
                              void* act, int M, int ffn, int K) {
    if (!swiglu_shape_ok(wdt, adt, M, ffn, K) || !half_operands_ok(wdt, M, 2L * ffn, K)) return hipErrorInvalidValue;
    if (K % 64 == 0) return launch_gemm_tall_swiglu(st, wdt, adt, A, W_gate_up, act, M, ffn, K);
    constexpr int TM = 256, TN = 256;
    const int N = 2 * ffn;
    const int tiles_m = (M + TM - 1) / TM, tiles_n = (N + TN - 1) / TN;
    dim3 grid(xcd_grid(tiles_m, tiles_n), 1);
    const int kchunk = (K + 63) / 64 * 64;
#define RLHF_SWIGLU(AF)                                               \
    k_gemm_bf16<TM, TN, 64, 4, 2, AF, true, true><<<grid, 512, 0, st>>>( \
        (const bf16_t*)A, (const bf16_t*)W_gate_up, (float*)act, M, N, K, kchunk, tiles_m, tiles_n)
    if (adt == kF16) RLHF_SWIGLU(true); else RLHF_SWIGLU(false);
#undef RLHF_SWIGLU
    return hipGetLastError();
}

hipError_t launch_gemm(hipStream_t st, int wdt, int adt, const void* A, const void* W, float* C,
                       int M, int N, int K, int nsplit, int variant) {
    if (M <= 0 || N <= 0) return hipSuccess;
    if (nsplit < 1 || K <= 0) return hipErrorInvalidValue;
    if (wdt == kF16) {
        // half copy of a bf16 matrix: the tall tiling with both operands global -> LDS directly
        if (adt != kF16 || K % 64 || (variant != 0 && variant != 7) || !half_operands_ok(wdt, M, N, K))
            return hipErrorInvalidValue;
        return launch_gemm_tall(st, wdt, adt, A, W, C, M, N, K, nsplit);
    }
    if (wdt == kBF16) {
        if (adt != kBF16 && adt != kF16) return hipErrorInvalidValue;
        if (K % 8 || variant < 0 || variant >= kNumCfgs) return hipErrorInvalidValue;
        if (variant == 0) {
            variant = pick_variant(M, N, K, nsplit);
            if (kCfgs[variant].xcd && nsplit != 1 && K % 64) variant = 4;   // only the kernel for whole K tiles splits
        }
        const bf16_t* a = (const bf16_t*)A;
        const bf16_t* w = (const bf16_t*)W;
        return adt == kF16 ? launch_bf16<true>(st, variant, a, w, C, M, N, K, nsplit)
                           : launch_bf16<false>(st, variant, a, w, C, M, N, K, nsplit);
    }
    if (K % 4 || adt != kF32) return hipErrorInvalidValue;
    // unsplit: gemm_f32.hip, which stores 16 bytes at a time and has 16 bits of row tiles
    if (nsplit == 1 && ((uintptr_t)C & 15) == 0 && M <= 65535L * 64)
        return launch_gemm_f32_tall(st, 0, (const float*)A, (const float*)W, C, M, N, K, RowsEpi{});
    const int tiles_m = (M + 63) / 64, tiles_n = (N + 63) / 64;
    const int kchunk = ((K + nsplit - 1) / nsplit + 15) / 16 * 16;
    dim3 grid(tiles_m * tiles_n, nsplit);
    k_gemm_f32<<<grid, 256, 0, st>>>((const float*)A, (const float*)W, C, M, N, K, kchunk, tiles_n);
    return hipGetLastError();
}

}  // namespace rlhf
