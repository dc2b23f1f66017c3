// Coefficients of many tokens at once, for the threshold calibration (Sec. 4).
// Part of cd_kernels.hip (its only includer).
//
// Calibration needs the dense coefficient vector of every calibration token.
// That is a matrix product C[T][d_ff] = X[T][d_model] . W[d_ff][d_model]^T, so
// the weights are read once for all tokens instead of once per decode-sized
// batch: 256 tokens of a 4096 x 11008 layer through a one-token plan took 256
// streams of W_up (14.3 us each) and 256 one-workgroup selects (6.6 us each),
// 5.6 ms a call.
//
// k_calib_gemm: a workgroup owns BM tokens x BN neurons. Both operands are
// K-contiguous, so tiles of 64 columns (128 B of a row: one cache line) go to
// LDS as they lie in memory, their 16-byte chunks swizzled by the row so that
// the 16 rows an MFMA operand read touches lie on different banks. Two LDS
// buffers, one barrier per tile, and DEPTH tiles in flight in registers. What
// bounds it is LDS traffic and the vector instructions of the sums: a single
// MFMA chain over 4096 columns rounds more often than the decode kernels' sums
// (relative error of the quantiles against fp64 7.5e-8; theirs 4.7e-8), so every
// 128 columns, 64 up to kFineCols, the accumulators go into a compensated fp32 sum
// (fold(): 3.8e-8 at 4096 columns, 3.1e-8 at 2048 and 3.5e-8 at 256, the decode
// kernels 4.7e-8, 5.1e-8 and 3.7e-8; means over 8 layers of 256 tokens). At 256
// tokens of 4096 x 11008 the whole call takes 78 us.
#pragma once

#include "cd_device.hpp"
#include "cd_internal.hpp"

namespace cdk {

namespace {

constexpr int kFineCols = 2048;  // up to so many columns, chains of 64 columns (else 128)

enum GemmKind { kGemmPlain, kGemmSilu, kGemmPair, kGemmTern };

struct GemmArgs {
    const uint16_t *X;    // [T][K] bf16
    const uint16_t *W0;   // [N][K] bf16 (Pair: W_gate)
    const uint16_t *W1;   // Pair: W_up
    const uint32_t *Tp;   // Tern: the packed ternary weights, twords words a row
    int T, N, K, twords;
    int nt;               // neuron tiles of the grid
    int mt;               // token tiles
    int ktiles;           // column tiles per split of K (gridDim.y splits)
    float *C;             // [splits][T][N]
};

// tot += acc, the rounding error of the addition added up in err; acc = 0
__device__ __forceinline__ void fold(f32x4_t &acc, f32x4_t &tot, f32x4_t &err)
{
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const float t = tot[r] + acc[r];
        err[r] += acc[r] - (t - tot[r]);
        tot[r] = t;
        acc[r] = 0.0f;
    }
}

// the folded sum (an infinite or NaN sum has no error term)
__device__ __forceinline__ float folded(float tot, float err)
{
    return fabsf(tot) < INFINITY ? tot + err : tot;
}

// KC columns per tile, DEPTH tiles in flight
template <int BM, int BN, int KC, int DEPTH, int KIND>
__global__ __launch_bounds__(kBlock) void k_calib_gemm(const GemmArgs a)
{
    constexpr int kGemmCols = KC, kGemmChunks = KC / 8, kDepth = DEPTH;
    // 16-byte chunk c of tile row r in LDS
    const auto swz = [](int r, int c) { return r * kGemmChunks + (c ^ (r & 7)); };
    constexpr bool kPair = KIND == kGemmPair;
    constexpr int kWM = BM >= 2 * kTile ? 2 : 1, kWN = kWavesPerBlock / kWM;  // waves of a tile
    constexpr int FM = BM / kWM / kTile, FN = BN / kWN / kTile;  // 16 x 16 tiles per wave
    static_assert(FM >= 1 && FN >= 1, "tile");
    constexpr int kRows = BM + BN * (kPair ? 2 : 1);
    constexpr int kChunks = kRows * kGemmChunks;
    constexpr int kLoads = kChunks / kBlock;
    static_assert(kChunks % kBlock == 0, "whole loads");
    __shared__ __align__(16) u32x4 lds[2][kChunks];
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    const int wm = wave / kWN, wn = wave % kWN;
    // token tiles of one neuron tile sit 8 workgroups apart, on the same XCD, so
    // the second reads the weights from its L2
    const int per = 8 * a.mt;
    const int nq = (int)blockIdx.x / per * 8 + (int)blockIdx.x % 8;
    const int mq = (int)blockIdx.x % per / 8;
    if (nq >= a.nt)  // the grid is a multiple of 8 neuron tiles
        return;
    const int m0 = mq * BM, n0 = nq * BN;
    const int kt0 = blockIdx.y * a.ktiles;
    const int kall = (a.K + kGemmCols - 1) / kGemmCols;
    const int nk = max(0, min(a.ktiles, kall - kt0));
    const int kend = min(a.K, (kt0 + nk) * kGemmCols);  // columns of this split end here

    // This thread's chunks: byte offsets from the tile's first row, one buffer
    // resource per operand; the column offset is scalar. Chunks of rows past the
    // operand, and of columns past kend, take an offset past the resource and read
    // zeros (one select per load; no branches and no 64-bit addresses).
    const auto resource = [](const void *p, size_t bytes) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)bytes, 0x00027000);
    };
    const size_t rb = (size_t)a.K * 2, tb = (size_t)a.twords * 4;  // bytes of a row
    const int rm = min(BM, a.T - m0), rn = min(BN, a.N - n0);
    const auto rx = resource(a.X + (size_t)m0 * a.K, rm * rb);
    const auto rw0 = KIND == kGemmTern ? resource(a.Tp + (size_t)n0 * a.twords, rn * tb)
                                       : resource(a.W0 + (size_t)n0 * a.K, rn * rb);
    const auto rw1 = kPair ? resource(a.W1 + (size_t)n0 * a.K, rn * rb) : rw0;
    static_assert(BM * kGemmChunks % kBlock == 0 && BN * kGemmChunks % kBlock == 0,
                  "a load is of one operand");
    constexpr int kOutside = 0x40000000;  // past every resource (at most 128 rows)
    constexpr int kLx = BM * kGemmChunks / kBlock, kLw = BN * kGemmChunks / kBlock;
    int off[kLoads];
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
        const int f = threadIdx.x + i * kBlock;
        const int r = f / kGemmChunks - (i < kLx ? 0 : i < kLx + kLw ? BM : BM + BN);
        const int c = f % kGemmChunks;
        if (KIND == kGemmTern && i >= kLx)
            off[i] = r < rn ? r * (int)tb + c * (a.twords / kWave) * 4 : kOutside;
        else
            off[i] = r < (i < kLx ? rm : rn) ? r * (int)rb + c * 16 : kOutside;
    }
    u32x4 reg[kDepth][kLoads];
    const auto load_tile = [&](u32x4 (&g)[kLoads], int kt) {
        const int k0 = min((kt0 + kt) * kGemmCols, kend);  // uniform; within a row of the resource
        // the packed word of columns k0 .. k0 + 7 (a tile lies within one unit of 512)
        const int tw = (k0 % kColsPerLoad / 8 * (a.twords / kWave) + (k0 / kColsPerLoad >> 1)) * 4;
        const bool in = (int)(threadIdx.x % kGemmChunks) * 8 < kend - k0;  // every load's columns
#pragma unroll
        for (int i = 0; i < kLoads; ++i) {
            const auto &rs = i < kLx ? rx : i < kLx + kLw ? rw0 : rw1;
            const int vo = in ? off[i] : kOutside;
            if (KIND == kGemmTern && i >= kLx)
                g[i].x = __builtin_amdgcn_raw_buffer_load_b32(rs, vo, tw, 0);
            else
                g[i] = __builtin_bit_cast(u32x4,
                                          __builtin_amdgcn_raw_buffer_load_b128(rs, vo, k0 * 2, 0));
        }
        __builtin_amdgcn_sched_barrier(0);  // tiles load in the order they are waited for
    };

    f32x4_t acc[kPair ? 2 : 1][FM][FN], tot[kPair ? 2 : 1][FM][FN], err[kPair ? 2 : 1][FM][FN];
#pragma unroll
    for (int p = 0; p < (kPair ? 2 : 1); ++p)
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j)
                acc[p][i][j] = tot[p][i][j] = err[p][i][j] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};

#pragma unroll
    for (int d = 0; d < kDepth; ++d)
        load_tile(reg[d], d);
    // (tiles past nk are zeros: whole groups of kDepth)
    static_assert(kDepth % 2 == 0, "the buffer of a tile is a constant");
    for (int kb = 0; kb < nk; kb += kDepth) {
#pragma unroll
        for (int d = 0; d < kDepth; ++d) {
            const int kt = kb + d;
            u32x4 *buf = lds[d & 1];
#pragma unroll
            for (int i = 0; i < kLoads; ++i) {
                const int f = threadIdx.x + i * kBlock;
                u32x4 v = reg[d][i];
                if (KIND == kGemmTern && i >= kLx) {
                    const uint32_t W = v.x;
                    const int j = (kt0 + kt) * kGemmCols / kColsPerLoad;  // unit (uniform)
                    v = u32x4{tern_pair(W, j, 0), tern_pair(W, j, 1), tern_pair(W, j, 2),
                              tern_pair(W, j, 3)};
                }
                buf[swz(f / kGemmChunks, f % kGemmChunks)] = v;
            }
            load_tile(reg[d], kt + kDepth);
            __syncthreads();  // (the buffer of tile kt - 1 is free: its readers passed this barrier)
#pragma unroll
            for (int h = 0; h < kGemmCols / 32; ++h) {
                const int i16 = lane % kTile, g = lane / kTile;
                u32x4 xa[FM];
#pragma unroll
                for (int i = 0; i < FM; ++i)
                    xa[i] = buf[swz((wm * FM + i) * kTile + i16, h * 4 + g)];
#pragma unroll
                for (int p = 0; p < (kPair ? 2 : 1); ++p)
#pragma unroll
                    for (int j = 0; j < FN; ++j) {
                        const u32x4 wb =
                            buf[swz(BM + p * BN + (wn * FN + j) * kTile + i16, h * 4 + g)];
#pragma unroll
                        for (int i = 0; i < FM; ++i)
                            acc[p][i][j] = mfma16(xa[i], wb, acc[p][i][j]);
                    }
                const int cols = (d * KC) + (h + 1) * 32;  // since the last whole group of tiles
                if (cols % 128 == 0 || (cols % 64 == 0 && a.K <= kFineCols)) {  // uniform
#pragma unroll
                    for (int p = 0; p < (kPair ? 2 : 1); ++p)
#pragma unroll
                        for (int i = 0; i < FM; ++i)
#pragma unroll
                            for (int j = 0; j < FN; ++j)
                                fold(acc[p][i][j], tot[p][i][j], err[p][i][j]);
                }
            }
        }
    }
    static_assert(kDepth * KC % 128 == 0, "the last fold ends the loop");
    // lane l holds D[4 (l / 16) + r][l % 16] of each 16 x 16 tile
    float *C = a.C + (size_t)blockIdx.y * a.T * a.N;
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) {
            const int n = n0 + (wn * FN + j) * kTile + lane % kTile;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int t = m0 + (wm * FM + i) * kTile + 4 * (lane / kTile) + r;
                float c = folded(tot[0][i][j][r], err[0][i][j][r]);
                if (KIND == kGemmSilu)
                    c = silu(c);
                else if (KIND == kGemmPair)
                    c = folded(tot[kPair][i][j][r], err[kPair][i][j][r]) * silu(c);  // u * SiLU(g)
                else if (KIND == kGemmTern)
                    c = 2.0f * c;  // the decoded weights are halves
                if (t < a.T && n < a.N)
                    C[(size_t)t * a.N + n] = c;
            }
        }
}

// lat[i] = sum of the splits' partial latents, in split order, compensated
__global__ __launch_bounds__(kBlock) void k_calib_latent_sum(const float *__restrict__ part,
                                                             int splits, int n,
                                                             float *__restrict__ lat)
{
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= n)
        return;
    float v = 0.0f, err = 0.0f;
    for (int s = 0; s < splits; ++s) {
        const float p = part[(size_t)s * n + i];
        const float t = v + p;
        err += p - (t - v);
        v = t;
    }
    lat[i] = folded(v, err);
}

// Predictor scores of many tokens: C[T][N] = lat[T][R] (fp32) . B_t[N][R]^T on
// the fp32 matrix instruction v_mfma_f32_16x16x4_f32 (the latent stays fp32,
// as in the decode kernels; B_t widens exactly). A workgroup owns 64 tokens x
// 64 neurons, a wave 32 x 32; 32 columns of the rank per LDS tile. LDS words of
// a row are padded by 4: the 16 rows of an operand read lie on different banks.
constexpr int kScoreTile = 64, kScoreCols = 32, kScoreStride = kScoreCols + 4;

__global__ __launch_bounds__(kBlock) void k_calib_score(const float *__restrict__ lat,
                                                        const uint16_t *__restrict__ Bt, int T,
                                                        int N, int R, float *__restrict__ C)
{
    __shared__ __align__(16) float la[kScoreTile * kScoreStride], lb[kScoreTile * kScoreStride];
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    const int n0 = blockIdx.x * kScoreTile, m0 = blockIdx.y * kScoreTile;
    const int wm = wave / 2, wn = wave % 2;
    f32x4_t acc[2][2], tot[2][2], err[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
            acc[i][j] = tot[i][j] = err[i][j] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
    // per tile and thread: two 16-byte chunks of the latent, one of B_t
    const int ra = threadIdx.x / 8, ca = threadIdx.x % 8 * 4;   // rows ra and ra + 32
    const int rb = threadIdx.x / 4, cb = threadIdx.x % 4 * 8;
    u32x4 va[2], vb;
    const auto load = [&](int k0) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
            va[h] = *or_zero(m0 + ra + 32 * h < T && k0 + ca < R,
                             reinterpret_cast<const u32x4 *>(lat + (size_t)(m0 + ra + 32 * h) * R + k0 + ca));
        vb = load16(or_zero(n0 + rb < N && k0 + cb < R, Bt + (size_t)(n0 + rb) * R + k0 + cb));
        __builtin_amdgcn_sched_barrier(0);
    };
    load(0);
    for (int k0 = 0; k0 < R; k0 += kScoreCols) {
        __syncthreads();
#pragma unroll
        for (int h = 0; h < 2; ++h)
            *reinterpret_cast<u32x4 *>(la + (ra + 32 * h) * kScoreStride + ca) = va[h];
        float *db = lb + rb * kScoreStride + cb;
        *reinterpret_cast<float4 *>(db) = make_float4(bf16_lo(vb.x), bf16_hi(vb.x), bf16_lo(vb.y), bf16_hi(vb.y));
        *reinterpret_cast<float4 *>(db + 4) = make_float4(bf16_lo(vb.z), bf16_hi(vb.z), bf16_lo(vb.w), bf16_hi(vb.w));
        __syncthreads();
        load(k0 + kScoreCols);  // under this tile's products (past R: zeros)
#pragma unroll
        for (int kk = 0; kk < kScoreCols; kk += 4) {
            const int r16 = lane % kTile, k = kk + lane / kTile;
            float fa[2], fb[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                fa[i] = la[((wm * 2 + i) * kTile + r16) * kScoreStride + k];
                fb[i] = lb[((wn * 2 + i) * kTile + r16) * kScoreStride + k];
            }
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[i], fb[j], acc[i][j], 0, 0, 0);
            if ((kk + 4) % 16 == 0)
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j)
                        fold(acc[i][j], tot[i][j], err[i][j]);
        }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int n = n0 + (wn * 2 + j) * kTile + lane % kTile;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int t = m0 + (wm * 2 + i) * kTile + 4 * (lane / kTile) + r;
                if (t < T && n < N)
                    C[(size_t)t * N + n] = folded(tot[i][j][r], err[i][j][r]);
            }
        }
}

template <int BM, int BN, int KC, int DEPTH, int KIND>
hipError_t gemm_launch(GemmArgs a, int splits, hipStream_t s)
{
    a.mt = (a.T + BM - 1) / BM;
    a.nt = (a.N + BN - 1) / BN;
    const int ktiles = (a.K + KC - 1) / KC;
    a.ktiles = (ktiles + splits - 1) / splits;
    const int grid = (a.nt + 7) / 8 * 8 * a.mt;
    k_calib_gemm<BM, BN, KC, DEPTH, KIND><<<dim3(grid, splits), kBlock, 0, s>>>(a);
    return hipGetLastError();
}

template <int KIND>
hipError_t gemm(const GemmArgs &a, int splits, hipStream_t s)
{
    // Up to 32 tokens the product is a stream of W: small tiles, 256 bytes of a row
    // at a time (8192 x 28672 at 32 tokens: 149 us a call, 789 as 8 decode batches).
    // Past that 64 x 64, three workgroups to a CU: a call of 256 tokens of 4096 x 11008
    // takes 78 us, with 128 x 64 tiles, whose 344 workgroups leave two thirds of the CUs
    // half loaded, 91; 64 tokens there 54 against 72. With many more workgroups 64 x 64
    // stays ahead too (256 tokens of 8192 x 28672: 272 against 291 us), but for 128 tokens
    // of 14336 neurons and more at 4096 columns and up (98 against 96; 8192 x 28672: 193
    // against 172).
    if (a.T <= 32)
        return gemm_launch<32, 32, 128, 2, KIND>(a, splits, s);
    return gemm_launch<64, KIND == kGemmPair ? 32 : 64, 64, 2, KIND>(a, splits, s);
}

// splits of the latent product: its few neuron tiles (the rank) leave the chip
// idle otherwise; at least 256 columns each
int latent_splits(int d_model)
{
    const int s = (d_model + 255) / 256;
    return s < 16 ? s : 16;
}

}  // namespace

size_t calib_scratch_floats(int variant, int T, int d_model, int d_rank)
{
    return variant == kDualPred ? (size_t)T * d_rank * (1 + latent_splits(d_model)) : 0;
}

hipError_t launch_calib_coef(int variant, const CalibArgs &c, hipStream_t s)
{
    GemmArgs a = {};
    a.X = c.X;
    a.T = c.T;
    a.N = c.d_ff;
    a.K = c.d_model;
    a.C = c.coef;
    switch (variant) {
    case kMono:
        a.W0 = c.Wu;
        return gemm<kGemmPlain>(a, 1, s);
    case kCats:
        a.W0 = c.Wg;
        return gemm<kGemmSilu>(a, 1, s);
    case kDualIdeal:
        a.W0 = c.Wg;
        a.W1 = c.Wu;
        return gemm<kGemmPair>(a, 1, s);
    case kDualTern:
        a.Tp = c.Tp;
        a.twords = tern_row_words(c.d_model);
        return gemm<kGemmTern>(a, 1, s);
    case kDualPred: {
        float *lat = c.scratch, *part = c.scratch + (size_t)c.T * c.d_rank;
        const int splits = latent_splits(c.d_model);
        a.W0 = c.At;
        a.N = c.d_rank;
        a.C = part;
        hipError_t e = gemm<kGemmPlain>(a, splits, s);
        if (e != hipSuccess)
            return e;
        const int n = c.T * c.d_rank;
        k_calib_latent_sum<<<(n + kBlock - 1) / kBlock, kBlock, 0, s>>>(part, splits, n, lat);
        if ((e = hipGetLastError()) != hipSuccess)
            return e;
        const dim3 grid((c.d_ff + kScoreTile - 1) / kScoreTile, (c.T + kScoreTile - 1) / kScoreTile);
        k_calib_score<<<grid, kBlock, 0, s>>>(lat, c.Bt, c.T, c.d_ff, c.d_rank, c.coef);
        return hipGetLastError();
    }
    default:
        return hipErrorInvalidValue;
    }
}

}  // namespace cdk
