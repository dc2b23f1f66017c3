// Coefficient and gather kernels for batches of 3-8 tokens (where: batch_coef). Part of
// cd_kernels.hip (its only includer).
//
// At 3-8 tokens a row's products with the batch are a thin matrix product. These
// kernels run it on v_mfma_f32_4x4x4_16b_bf16: sixteen independent 4 x 4 x 4
// blocks, lane l = 4 block + i holding 4 columns of row i (A operand) and of token
// i (B operand). The blocks take different columns of the same four neurons and
// tokens and are added across the lanes at the end, so
//   - a pair of load instructions covers 4 rows x 512 contiguous bytes and goes to
//     the matrix core after one exchange between neighbouring lanes, with no staging
//     of weights through LDS;
//   - the eight waves of a workgroup take an eighth of the columns each, and keep
//     their slice of the tokens in registers (4 to 32 of them): there is no token
//     copy in LDS (32-64 KB, reloaded by every four or 32 neurons before, and read
//     once per token and weight chunk), and a weight chunk costs 2 MFMA
//     instructions per four tokens instead of 4 v_dot2 per token.
// A workgroup owns up to kPredRows = 32 neurons, eight row quads; a wave keeps up to
// eight loads (8 KB) in flight over the next quads. The waves' sums of a quad meet in
// LDS, and from there one thread per (token, neuron) goes on: threshold, union,
// compaction of the active neurons to dense quads for the gather of the second
// projection(s), s.
#pragma once

namespace cdk {

constexpr int kBatWaves = 8;
constexpr int kBatThreads = kBatWaves * kWave;
constexpr int kQuads = kPredRows / 4;  // row quads of a workgroup
constexpr int kOutside = 0x40000000;   // byte offset past every buffer resource here

typedef short i16x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// 8 columns of a quad's rows times 8 columns of a quad of tokens
__device__ __forceinline__ f32x4_t mfma4(const u32x4 &w, const u32x4 &x, f32x4_t c)
{
    const u32x2 w0 = {w.x, w.y}, w1 = {w.z, w.w}, x0 = {x.x, x.y}, x1 = {x.z, x.w};
    c = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(__builtin_bit_cast(i16x4_t, w0),
                                               __builtin_bit_cast(i16x4_t, x0), c, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(__builtin_bit_cast(i16x4_t, w1),
                                                  __builtin_bit_cast(i16x4_t, x1), c, 0, 0, 0);
}

// Sum of d over the 16 blocks. Lane l returns row l / 16, token l % 4 of the quads.
__device__ __forceinline__ float quad_sum(const f32x4_t &d)
{
    const auto add32 = [](float a, float b) {  // a's sum in lanes 0-31, b's in 32-63
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
        return __uint_as_float(r[0]) + __uint_as_float(r[1]);
    };
    const float p = add32(d[0], d[2]), q = add32(d[1], d[3]);
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(p), __float_as_uint(q), false, false);
    float v = __uint_as_float(r[0]) + __uint_as_float(r[1]);  // 16-lane row r: matrix row r
    v += dpp0<0x124>(v);  // row_ror:4
    v += dpp0<0x128>(v);  // row_ror:8
    return v;
}

using BufRsrc = decltype(__builtin_amdgcn_make_buffer_rsrc(nullptr, 0, 0, 0));

__device__ __forceinline__ BufRsrc buffer(const void *p, int bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, bytes, 0x00027000);
}

// A wave's columns of a row are S steps of 16 chunks of 8 columns, one chunk per
// block. A load in operand layout, row l % 4 on lane l, takes the vector memory unit
// one cycle per lane: it merges the accesses of four neighbouring lanes only, so it
// delivers 16 B/clk, 38 GB/s per CU, little above a CU's share of HBM (27 GB/s) and
// below it with the token loads. So steps are loaded in pairs, neighbouring lanes on
// neighbouring chunks of one row (32 B/clk, measured 76 GB/s per CU; 151 for 64
// bytes, which would need a second exchange): load A holds rows 0 and 2 and load B
// rows 1 and 3 at both steps, lane l row (l & 2) and step l & 1, and one exchange
// between neighbouring lanes (swap_pair) sorts them. An odd last step is loaded as it
// is used.
//
// Plain slices: the wave's steps are one run of 128 S columns. Ternary slices: the
// columns whose packed weights lie together (TernQuad).
template <int S, bool TERN>
struct Columns {
    static_assert(!TERN || S == 1 || S % 2 == 0, "whole units");
    static constexpr int kPairs = S / 2, kStride = TERN ? kColsPerLoad : 256;
    int pair0, single, d_model;  // this lane's column in pair 0 and in the odd last step

    __device__ __forceinline__ void init(int wave, int lane, int dm)
    {
        d_model = dm;
        const int b = lane / 4;
        if constexpr (!TERN) {
            pair0 = wave * S * 128 + (2 * b + (lane & 1)) * 8;
            single = wave * S * 128 + (S - 1) * 128 + b * 8;
        } else {  // S >= 2: packed lanes 8 wave + 2 (b % 4) + step, units (b / 4) S / 2 + pair
            pair0 = b / 4 * (S / 2) * kColsPerLoad + (wave * 8 + 2 * (b % 4) + (lane & 1)) * 8;
            // S = 1: one unit, packed lane 16 wave + b (waves 4-7: past the row); or two,
            // packed lane 8 wave + b % 8 of unit b / 8
            single = dm <= kColsPerLoad ? (wave * 16 + b) * 8
                                        : b / 8 * kColsPerLoad + (wave * 8 + b % 8) * 8;
        }
    }
};

// a, b: loads A and B of a pair of steps; afterwards row l % 4 at its first and second
__device__ __forceinline__ void swap_pair(u32x4 &a, u32x4 &b, bool odd)
{
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint32_t x = a[k], y = b[k];
        const uint32_t xs = __builtin_amdgcn_update_dpp(x, x, kDppQuadSwap1, 0xF, 0xF, true);
        const uint32_t ys = __builtin_amdgcn_update_dpp(y, y, kDppQuadSwap1, 0xF, 0xF, true);
        a[k] = odd ? ys : x;
        b[k] = odd ? y : xs;
    }
}

// The loads of four rows of one matrix (or of four tokens) at the wave's steps.
// row(i): this lane's row at position i of the quad, < 0 for none.
template <int S, bool TERN, int AUX, class RowF>
__device__ __forceinline__ void issue_rows(u32x4 (&w)[S], const BufRsrc &m, RowF row,
                                           const Columns<S, TERN> &cols, int lane)
{
    using C = Columns<S, TERN>;
    if constexpr (C::kPairs > 0) {
        const int ra = row(lane & 2), rb = row((lane & 2) | 1);
        const int oa = (ra * cols.d_model + cols.pair0) * 2, ob = (rb * cols.d_model + cols.pair0) * 2;
#pragma unroll
        for (int h = 0; h < C::kPairs; ++h) {
            const bool in = cols.pair0 + h * C::kStride < cols.d_model;
            w[2 * h] = __builtin_bit_cast(
                u32x4, __builtin_amdgcn_raw_buffer_load_b128(
                           m, (in && ra >= 0 ? oa : kOutside) + h * C::kStride * 2, 0, AUX));
            w[2 * h + 1] = __builtin_bit_cast(
                u32x4, __builtin_amdgcn_raw_buffer_load_b128(
                           m, (in && rb >= 0 ? ob : kOutside) + h * C::kStride * 2, 0, AUX));
        }
    }
    if constexpr (S % 2 == 1) {
        const int r = row(lane & 3);
        const bool in = cols.single < cols.d_model;
        w[S - 1] = __builtin_bit_cast(
            u32x4, __builtin_amdgcn_raw_buffer_load_b128(
                       m, in && r >= 0 ? (r * cols.d_model + cols.single) * 2 : kOutside, 0, AUX));
    }
}

template <int S>
__device__ __forceinline__ void sort_rows(u32x4 (&w)[S], int lane)
{
#pragma unroll
    for (int h = 0; h < S / 2; ++h)
        swap_pair(w[2 * h], w[2 * h + 1], lane & 1);
}

// The wave's slice of the tokens as MFMA operands, in registers for the whole kernel
template <int TQ, int S, bool TERN>
struct TokenSlice {
    u32x4 x[TQ][S];

    __device__ __forceinline__ void issue(const CoefArgs &a, const Columns<S, TERN> &cols, int lane)
    {
        const BufRsrc r = buffer(a.x, a.nb * a.d_model * 2);
#pragma unroll
        for (int t = 0; t < TQ; ++t)
            issue_rows<S, TERN, 0>(
                x[t], r, [&](int i) { return t * 4 + i < a.nb ? t * 4 + i : -1; }, cols, lane);
    }
    __device__ __forceinline__ void sort(int lane)
    {
#pragma unroll
        for (int t = 0; t < TQ; ++t)
            sort_rows<S>(x[t], lane);
    }
};

// LDS [matrix][wave][token][row position]: the waves' sums, rows padded by one word
template <int TQ>
struct PartSums {
    static constexpr int kTok = TQ * 4, kRow = kPredRows + 1;
    static constexpr int kWaveWords = kTok * kRow;
    float *p;

    // the wave's sums of quad q of matrix m
    __device__ __forceinline__ void put(int m, int wave, int q, int lane, const f32x4_t (&d)[TQ])
    {
#pragma unroll
        for (int t = 0; t < TQ; ++t) {
            const float v = quad_sum(d[t]);
            if ((lane & 12) == 0)
                p[(m * kBatWaves + wave) * kWaveWords + (t * 4 + lane % 4) * kRow + q * 4 +
                  lane / 16] = v;
        }
    }
    __device__ __forceinline__ float get(int m, int tok, int pos) const
    {
        float v[kBatWaves];
#pragma unroll
        for (int w = 0; w < kBatWaves; ++w)
            v[w] = p[(m * kBatWaves + w) * kWaveWords + tok * kRow + pos];
        return ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
    }
};

// Products of the block's quads of rows with the token slice, into sums. With two
// matrices a quad is two items, one per matrix, in turn. Up to 8 loads (8 KB) are in
// flight per wave: with 16 the two workgroups of a CU hold 256 KB in flight, and every
// case measured the same or slower (dense 4096 x 14336 at 8 tokens 72.8 against 65.1 us,
// where 128 registers spilled; M at 4 tokens 40.7 against 39.7). row(q, i): the row
// within the block at position i of quad q, < 0 for none.
// Loads past the last quad read nothing (an outside offset), so the loop has no
// branches around loads. SORT: the tokens are still as loaded; they are sorted behind
// the first weight loads.
template <int NM, int TQ, int S, bool TERN, bool SORT, class RowF>
__device__ __forceinline__ void run_quads(const BufRsrc (&m)[NM], int nq, RowF row,
                                          const Columns<S, TERN> &cols,
                                          TokenSlice<TQ, S, TERN> &tok, PartSums<TQ> sums,
                                          int wave, int lane)
{
    constexpr int D = S >= 6 ? 1 : 2;  // items in flight
    u32x4 buf[D][S];
    const int n = nq * NM;
    const auto issue = [&](u32x4 (&w)[S], int it) {
        const int q = it / NM;
        issue_rows<S, TERN, 2 /* non-temporal */>(
            w, m[it % NM], [&](int i) { return it < n ? row(q, i) : -1; }, cols, lane);
    };
#pragma unroll
    for (int d = 0; d < D; ++d)
        issue(buf[d], d);
    if constexpr (SORT) {
        __builtin_amdgcn_sched_barrier(0);
        tok.sort(lane);
    }
    for (int it0 = 0; it0 < n; it0 += D) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const int it = it0 + d;
            f32x4_t acc[TQ];
            sort_rows<S>(buf[d], lane);
#pragma unroll
            for (int t = 0; t < TQ; ++t)
                acc[t] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int i = 0; i < S; ++i)
#pragma unroll
                for (int t = 0; t < TQ; ++t)
                    acc[t] = mfma4(buf[d][i], tok.x[t][i], acc[t]);
            __builtin_amdgcn_sched_barrier(0);
            issue(buf[d], it + D);
            if (it < n)  // uniform
                sums.put(it % NM, wave, it / NM, lane, acc);
        }
    }
}

// The neurons of a workgroup: quads [first, first + nq), at most kQuads. The layer's
// quads are spread evenly over kCus shares and a share over the gridDim.x / kCus
// workgroups that the dispatch deals to one CU (workgroups i, i + kCus, ...), so that
// the CUs' shares differ by at most one quad (see batch_grid).
constexpr int kCus = 256;

struct Block {
    int r0, nq, rows;

    __device__ __forceinline__ Block(const CoefArgs &a)
    {
        const int64_t quads = a.d_ff / 4;  // d_ff is a multiple of 8
        const int shares = min(kCus, (int)gridDim.x), parts = (int)gridDim.x / shares;
        const int share = blockIdx.x % shares, part = blockIdx.x / shares;
        const int q0 = (int)(quads * share / shares), q1 = (int)(quads * (share + 1) / shares);
        const int first = q0 + (q1 - q0) * part / parts;
        nq = q0 + (q1 - q0) * (part + 1) / parts - first;
        r0 = first * 4;
        rows = nq * 4;
    }
    // the block's rows of a matrix
    __device__ __forceinline__ BufRsrc rows_of(const uint16_t *W, int d_model) const
    {
        return buffer(W + (size_t)r0 * d_model, rows * d_model * 2);
    }
};

// Row within the block at position pos of the active neurons M (< 0 past the last):
// lane i pushes its row to the lane of its rank, readers pull from there.
struct ActiveRows {
    int list, n;

    __device__ __forceinline__ void init(uint32_t M, int lane)
    {
        n = __builtin_popcount(M);
        const bool on = lane < kPredRows && ((M >> lane) & 1u);
        const int rank = __builtin_popcount(M & ((1u << (lane & 31)) - 1u));
        // inactive lanes push to lane 63, past every rank
        list = __builtin_amdgcn_ds_permute((on ? rank : kWave - 1) * 4, lane);
    }
    __device__ __forceinline__ int row(int q, int i) const
    {
        const int pos = q * 4 + i;
        const int r = __builtin_amdgcn_ds_bpermute(pos * 4, list);
        return pos < n ? r : -1;
    }
};

// This thread's neuron and token after the products: threads [0, 32 x tokens)
template <int TQ>
struct Cell {
    int row, tok;
    bool live;  // a token of the batch and a neuron of the block

    __device__ __forceinline__ Cell(const CoefArgs &a, const Block &b)
    {
        row = threadIdx.x % kPredRows;
        tok = threadIdx.x / kPredRows;
        live = tok < a.nb && row < b.rows;
    }
    __device__ __forceinline__ size_t at(const CoefArgs &a, const Block &b) const
    {
        return (size_t)tok * a.d_ff + b.r0 + row;
    }
};

// Union over the tokens of the cells' votes: every wave's ballot covers the 32
// neurons for two tokens. wflag: LDS [kBatWaves]. One barrier.
__device__ __forceinline__ uint32_t block_union(bool vote, uint32_t *wflag, int wave, int lane)
{
    const uint64_t b = ballot(vote);
    if (lane == 0)
        wflag[wave] = (uint32_t)b | (uint32_t)(b >> 32);
    __syncthreads();
    uint32_t M = 0;
#pragma unroll
    for (int v = 0; v < kBatWaves; ++v)
        M |= wflag[v];
    return M;
}

__device__ __forceinline__ void store_flags(const CoefArgs &a, const Block &b, uint32_t M)
{
    if ((int)threadIdx.x < b.rows)
        a.act[b.r0 + threadIdx.x] = (M >> threadIdx.x) & 1u;
}

__device__ __forceinline__ void zero_y_batch(const CoefArgs &a)
{
    const int n = a.nb * a.d_model;
    for (int i = blockIdx.x * kBatThreads + threadIdx.x; i < n; i += gridDim.x * kBatThreads)
        a.y[i] = 0.0f;
}

// Gather of the block's active neurons M: W_gate and W_up (NM 2) or the one second
// projection (NM 1, w2), s from the sums. first: the cell's coefficient (NM 1: s =
// first * SiLU(p), or p * first for CATS).
template <int NM, int TQ, int S, bool TERN>
__device__ __forceinline__ void gather_block(const CoefArgs &a, const uint16_t *w2, bool cats,
                                             float first, uint32_t M, const Block &b,
                                             const Columns<S, TERN> &cols,
                                             TokenSlice<TQ, S, TERN> &tok,
                                             PartSums<TQ> sums, int wave, int lane)
{
    if (M == 0)  // uniform
        return;
    ActiveRows act;
    act.init(M, lane);
    BufRsrc m[NM];
    m[0] = b.rows_of(NM == 2 ? a.Wg : w2, a.d_model);
    if constexpr (NM == 2)
        m[1] = b.rows_of(a.Wu, a.d_model);
    run_quads<NM, TQ, S, TERN, false>(m, (act.n + 3) / 4, [&](int q, int i) { return act.row(q, i); }, cols,
                               tok, sums, wave, lane);
    __syncthreads();
    const Cell<TQ> c(a, b);
    if (c.live && ((M >> c.row) & 1u)) {
        const int pos = __builtin_popcount(M & ((1u << c.row) - 1u));
        const float p = sums.get(0, c.tok, pos);
        float s;
        if constexpr (NM == 2)
            s = sums.get(1, c.tok, pos) * silu(p);
        else
            s = cats ? p * first : first * silu(p);
        a.s[c.at(a, b)] = s;
    }
}

// M-CountDown and CATS: the dense projection of the block, threshold, gather of the
// other projection. The waves stream quads in ascending order.
template <int TQ, int S>
__global__ __launch_bounds__(kBatThreads, 4) void k_batch_mono(const CoefArgs a, bool cats)
{
    __shared__ float psum[kBatWaves * PartSums<TQ>::kWaveWords];
    __shared__ uint32_t wflag[kBatWaves];
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    const Block b(a);
    Columns<S, false> cols;
    cols.init(wave, lane, a.d_model);
    TokenSlice<TQ, S, false> tok;
    tok.issue(a, cols, lane);
    PartSums<TQ> sums{psum};
    const BufRsrc m[1] = {b.rows_of(cats ? a.Wg : a.Wu, a.d_model)};
    run_quads<1, TQ, S, false, true>(
        m, b.nq, [](int q, int i) { return q * 4 + i; }, cols, tok, sums, wave, lane);
    zero_y_batch(a);
    __syncthreads();
    const Cell<TQ> c(a, b);
    float v = 0.0f;
    if (c.live) {
        v = sums.get(0, c.tok, c.row);
        v = cats ? silu(v) : v;
        if (a.coef)
            a.coef[c.at(a, b)] = v;
    }
    // (its barrier also ends the reads of the sums, which the gather reuses)
    const uint32_t M = block_union(c.live && fabsf(v) > a.thld, wflag, wave, lane);
    store_flags(a, b, M);
    gather_block<1, TQ, S, false>(a, cats ? a.Wu : a.Wg, cats, v, M, b, cols, tok, sums, wave,
                                  lane);
}

// Ideal D-CountDown and the dense layer: both projections of the block
template <int TQ, int S>
__global__ __launch_bounds__(kBatThreads, 4) void k_batch_dual(const CoefArgs a, bool dense)
{
    __shared__ float psum[2 * kBatWaves * PartSums<TQ>::kWaveWords];
    __shared__ uint32_t wflag[kBatWaves];
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    const Block b(a);
    Columns<S, false> cols;
    cols.init(wave, lane, a.d_model);
    TokenSlice<TQ, S, false> tok;
    tok.issue(a, cols, lane);
    PartSums<TQ> sums{psum};
    const BufRsrc m[2] = {b.rows_of(a.Wg, a.d_model), b.rows_of(a.Wu, a.d_model)};
    run_quads<2, TQ, S, false, true>(
        m, b.nq, [](int q, int i) { return q * 4 + i; }, cols, tok, sums, wave, lane);
    zero_y_batch(a);
    __syncthreads();
    const Cell<TQ> c(a, b);
    float s = 0.0f;
    if (c.live) {
        s = sums.get(1, c.tok, c.row) * silu(sums.get(0, c.tok, c.row));
        if (a.coef)
            a.coef[c.at(a, b)] = s;
    }
    const uint32_t M = block_union(c.live && (dense || fabsf(s) > a.thld), wflag, wave, lane);
    store_flags(a, b, M);
    if (c.live && ((M >> c.row) & 1u))
        a.s[c.at(a, b)] = s;
}

// Practical D-CountDown: every wave scores four of the block's neurons from their
// B_t rows, then the gather. The tokens' loads are issued before the scores.
template <int TQ, int S, int LCPR>
__global__ __launch_bounds__(kBatThreads, 4) void k_batch_pred(const CoefArgs a)
{
    constexpr int B = TQ * 4, R = kPredRows / kBatWaves;
    __shared__ float psum[2 * kBatWaves * PartSums<TQ>::kWaveWords];
    __shared__ uint32_t wflag[kBatWaves];
    extern __shared__ __align__(16) uint32_t xs[];  // latent [B][d_rank] (rank 1024 only)
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    const Block b(a);
    const int wr0 = wave < b.nq ? b.r0 + wave * R : a.d_ff;  // (past the block: nothing to score)
    using LR = LatentRegs<B, LCPR>;
    u32x4 wb[PredShape<LCPR, R>::kLoads];
    pred_issue_bt<LCPR, R>(wb, a, wr0, lane);
    LR lr;
    lr.issue(a.lat, a.nb, a.d_rank, lane);
    Columns<S, false> cols;
    cols.init(wave, lane, a.d_model);
    TokenSlice<TQ, S, false> tok;
    tok.issue(a, cols, lane);
    __builtin_amdgcn_sched_barrier(0);
    zero_y_batch(a);
    if constexpr (!LR::kRegs) {
        if (threadIdx.x < kBlock) {
            LatentStage<B> ls;
            ls.issue(a.lat, a.nb, a.d_rank);
            ls.write(reinterpret_cast<u32x4 *>(xs), a.lat, a.nb, a.d_rank);
        }
        __syncthreads();
    }
    const uint32_t wmask =
        pred_score<B, LCPR, R>(wb, lr, reinterpret_cast<const float *>(xs), a, wr0, lane);
    if (lane == 0)
        wflag[wave] = wmask << (wave * R);
    __syncthreads();
    uint32_t M = 0;
#pragma unroll
    for (int v = 0; v < kBatWaves; ++v)
        M |= wflag[v];
    tok.sort(lane);
    gather_block<2, TQ, S, false>(a, nullptr, false, 0.0f, M, b, cols, tok, PartSums<TQ>{psum},
                                  wave, lane);
}

// Packed ternary weights of a wave's slice of a quad of rows, for the columns of
// Columns<S, true>. Block c of lane l = 4 c + i needs, of row i and both steps s of a
// pair, the words of packed lane 8 wave + 2 (c % 4) + s that hold units (c / 4) S / 2
// and up (S / 4 words; a half of one for S = 2). They are loaded with neighbouring
// lanes on neighbouring words (lane 16 i + 4 (c % 4) + c / 4) and pulled across.
// S = 1 (d_model <= 1024) loads its one word as it is used.
template <int S>
struct TernQuad {
    static constexpr int kW = S >= 8 ? S / 4 : 1, kLoads = S >= 2 ? 2 : 1;
    uint32_t w[kLoads][kW];

    __device__ __forceinline__ void issue(const BufRsrc &r, bool ok, int q, int words, int wave,
                                          int lane, int dm)
    {
        const int lw = words / kWave;  // words per packed lane
        if constexpr (S == 1) {
            const int c = lane / 4;
            const int pl = dm <= kColsPerLoad ? wave * 16 + c : wave * 8 + c % 8;
            const int off = ok && pl < kWave ? ((q * 4 + lane % 4) * words + pl * lw) * 4 : kOutside;
            w[0][0] = __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 2);
        } else {
            const int row = q * 4 + lane / 16, p = lane % 16 / 4, g = lane % 4;
            const int at = (row * words + (wave * 8 + 2 * p) * lw + g * S / 4) * 4;
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const int off = ok ? at + s * lw * 4 : kOutside;
                if constexpr (kW == 2) {
                    const u32x2 v =
                        __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 2));
                    w[s][0] = v.x, w[s][1] = v.y;
                } else {
                    w[s][0] = __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 2);
                }
            }
        }
    }
    // to the lanes that use the words
    __device__ __forceinline__ void sort(int lane, int dm)
    {
        const int c = lane / 4;
        if constexpr (S >= 2) {
            const int from = 16 * (lane % 4) + 4 * (c % 4) + c / 4;
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int k = 0; k < kW; ++k)
                    w[s][k] = (uint32_t)__builtin_amdgcn_ds_bpermute(from * 4, (int)w[s][k]);
        }
        // S <= 2: a block's unit may be the odd one of its word; move it to where the even
        // one is decoded
        const int unit = S == 2 ? c / 4 : dm <= kColsPerLoad ? 0 : c / 8;
        if (S <= 2 && (unit & 1))
#pragma unroll
            for (int s = 0; s < kLoads; ++s)
                w[s][0] <<= 8;
    }
    // the 8 weights (+-0.5 or 0) of step i = 2 pair + s
    __device__ __forceinline__ u32x4 step(int i) const
    {
        const int h = i / 2;  // unit within the lane's
        const uint32_t W = w[S == 1 ? 0 : i % 2][S >= 4 ? h / 2 : 0];
        return u32x4{tern_pair(W, h, 0), tern_pair(W, h, 1), tern_pair(W, h, 2), tern_pair(W, h, 3)};
    }
};

// The ternary predictor: scores of the block's quads from the packed theta on the
// same MFMA blocks (every quad's words are loaded at once: 8 to 32 registers),
// then the gather.
template <int TQ, int S>
__global__ __launch_bounds__(kBatThreads, 4) void k_batch_tern(const CoefArgs a, int words)
{
    __shared__ float psum[2 * kBatWaves * PartSums<TQ>::kWaveWords];
    __shared__ uint32_t wflag[kBatWaves];
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    const Block b(a);
    const BufRsrc tp = buffer(a.Tp + (size_t)b.r0 * words, b.rows * words * 4);
    TernQuad<S> tq[kQuads];
#pragma unroll
    for (int q = 0; q < kQuads; ++q)
        tq[q].issue(tp, q < b.nq, q, words, wave, lane, a.d_model);
    Columns<S, true> cols;
    cols.init(wave, lane, a.d_model);
    TokenSlice<TQ, S, true> tok;
    tok.issue(a, cols, lane);
    __builtin_amdgcn_sched_barrier(0);
    zero_y_batch(a);
    tok.sort(lane);
    PartSums<TQ> sums{psum};
#pragma unroll
    for (int q = 0; q < kQuads; ++q) {
        if (q >= b.nq)  // uniform
            break;
        tq[q].sort(lane, a.d_model);
        f32x4_t acc[TQ];
#pragma unroll
        for (int t = 0; t < TQ; ++t)
            acc[t] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int i = 0; i < S; ++i) {
            const u32x4 w = tq[q].step(i);
#pragma unroll
            for (int t = 0; t < TQ; ++t)
                acc[t] = mfma4(w, tok.x[t][i], acc[t]);
        }
        sums.put(0, wave, q, lane, acc);
    }
    __syncthreads();
    const Cell<TQ> c(a, b);
    float v = 0.0f;
    if (c.live) {
        v = 2.0f * sums.get(0, c.tok, c.row);  // the decoded weights are halves
        if (a.coef)
            a.coef[c.at(a, b)] = v;
    }
    const uint32_t M = block_union(c.live && v > a.thld, wflag, wave, lane);
    store_flags(a, b, M);
    gather_block<2, TQ, S, true>(a, nullptr, false, 0.0f, M, b, cols, tok, sums, wave, lane);
}

// Per-token thresholds: flags of the block against every token's own quantile, then
// the gather (NM 1: M-CountDown and CATS; NM 2: the predictors, signed scores)
template <int NM, int TQ, int S>
__global__ __launch_bounds__(kBatThreads, 4) void k_batch_topk(const CoefArgs a,
                                                            const double *__restrict__ q, bool cats)
{
    __shared__ float psum[NM * kBatWaves * PartSums<TQ>::kWaveWords];
    __shared__ uint32_t wflag[kBatWaves];
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    const Block b(a);
    const Cell<TQ> c(a, b);
    float v = 0.0f;
    double qv = 0.0;
    if (c.live) {
        v = a.coef[c.at(a, b)];
        qv = q[c.tok];
    }
    Columns<S, false> cols;
    cols.init(wave, lane, a.d_model);
    TokenSlice<TQ, S, false> tok;
    tok.issue(a, cols, lane);
    zero_y_batch(a);
    const uint32_t M =
        block_union(c.live && (double)(NM == 2 ? v : fabsf(v)) > qv, wflag, wave, lane);
    store_flags(a, b, M);
    tok.sort(lane);
    gather_block<NM, TQ, S, false>(a, cats ? a.Wu : a.Wg, cats, v, M, b, cols, tok,
                                   PartSums<TQ>{psum}, wave, lane);
}

// Workgroups: two per CU (all resident at up to 128 registers), or a multiple, so that
// every CU gets the same share: a CU reads about 27 GB/s here, its share of the chip's
// rate and not much more, so what one has too much is not made up elsewhere. (Blocks of
// 32 neurons, 344 workgroups, left two thirds of the CUs idle for half of the dense 4096 x
// 11008 layer: 62 us against 52 at 4 tokens; three workgroups per CU reload the tokens
// and measured 2-5 us slower.)
// One per CU up to three quads per CU, where a workgroup's barriers and token loads weigh
// more than its rows: 4096 x 2048, M at 8 tokens 18.1 us with two, 16.2 with one, low-rank
// (rank 128) 22.7 against 20.8; from 4096 neurons on two are even or faster (1024 x 8192
// ternary at 8 tokens 9% faster). And one per CU up to eight quads, a workgroup's most,
// where each workgroup keeps the latents in LDS (rank 1024): 1024 x 4096 at 8 tokens 57.3 us
// with two, 39.7 with one; 4096 x 8192 69.8 against 56.8.
inline int batch_grid(int d_ff, bool lds_latent)
{
    const int quads = d_ff / 4, per = 2 * kCus * kQuads;
    if (quads <= (lds_latent ? kQuads : 3) * kCus)
        return quads < kCus ? quads : kCus;
    return (quads + per - 1) / per * 2 * kCus;
}

// steps of 128 columns per wave
inline int batch_steps(int d_model) { return (d_model + 128 * kBatWaves - 1) / (128 * kBatWaves); }

template <int TQ, int S>
static hipError_t batch_pred(const CoefArgs &a, int grid, hipStream_t s)
{
    const size_t lat = a.d_rank == 1024 ? (size_t)TQ * 4 * 1024 * 4 : 0;
    switch (a.d_rank) {
    case 8: k_batch_pred<TQ, S, 0><<<grid, kBatThreads, 0, s>>>(a); break;
    case 16: k_batch_pred<TQ, S, 1><<<grid, kBatThreads, 0, s>>>(a); break;
    case 32: k_batch_pred<TQ, S, 2><<<grid, kBatThreads, 0, s>>>(a); break;
    case 64: k_batch_pred<TQ, S, 3><<<grid, kBatThreads, 0, s>>>(a); break;
    case 128: k_batch_pred<TQ, S, 4><<<grid, kBatThreads, 0, s>>>(a); break;
    case 256: k_batch_pred<TQ, S, 5><<<grid, kBatThreads, 0, s>>>(a); break;
    case 512: k_batch_pred<TQ, S, 6><<<grid, kBatThreads, 0, s>>>(a); break;
    case 1024: k_batch_pred<TQ, S, 7><<<grid, kBatThreads, lat, s>>>(a); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// the kernel of a variant; q (per-token thresholds) selects the gather after a select
template <int TQ, int S>
static hipError_t batch_ts(int variant, const CoefArgs &a, const double *q, hipStream_t s)
{
    const int grid = batch_grid(a.d_ff, variant == kDualPred && !q && a.d_rank == 1024);
    if (q) {
        if (variant == kDualPred)
            k_batch_topk<2, TQ, S><<<grid, kBatThreads, 0, s>>>(a, q, false);
        else
            k_batch_topk<1, TQ, S><<<grid, kBatThreads, 0, s>>>(a, q, variant == kCats);
        return hipGetLastError();
    }
    switch (variant) {
    case kMono:
    case kCats: k_batch_mono<TQ, S><<<grid, kBatThreads, 0, s>>>(a, variant == kCats); break;
    case kDualIdeal:
    case kDense: k_batch_dual<TQ, S><<<grid, kBatThreads, 0, s>>>(a, variant == kDense); break;
    case kDualPred: return batch_pred<TQ, S>(a, grid, s);
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <int TQ>
static hipError_t batch_tern(const CoefArgs &a, hipStream_t s)
{
    const int grid = batch_grid(a.d_ff, false);
    const int words = tern_row_words(a.d_model);
    switch (col_tile(a.d_model)) {  // units of 512 columns: two per wave step
    case 1:
    case 2: k_batch_tern<TQ, 1><<<grid, kBatThreads, 0, s>>>(a, words); break;
    case 4: k_batch_tern<TQ, 2><<<grid, kBatThreads, 0, s>>>(a, words); break;
    case 8: k_batch_tern<TQ, 4><<<grid, kBatThreads, 0, s>>>(a, words); break;
    default:
        if constexpr (TQ == 1) {
            k_batch_tern<TQ, 8><<<grid, kBatThreads, 0, s>>>(a, words);
            break;
        }
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <int TQ>
static hipError_t batch_t(int variant, const CoefArgs &a, const double *q, hipStream_t s)
{
    if (variant == kDualTern && !q)
        return batch_tern<TQ>(a, s);
    switch (batch_steps(a.d_model)) {
    case 1: return batch_ts<TQ, 1>(variant, a, q, s);
    case 2: return batch_ts<TQ, 2>(variant, a, q, s);
    case 3: return batch_ts<TQ, 3>(variant, a, q, s);
    case 4: return batch_ts<TQ, 4>(variant, a, q, s);
    default:
        if constexpr (TQ == 1)  // batch x d_model <= 32768: up to 4 tokens past 4096 columns
            return batch_steps(a.d_model) <= 6 ? batch_ts<TQ, 6>(variant, a, q, s)
                                               : batch_ts<TQ, 8>(variant, a, q, s);
        return hipErrorInvalidValue;
    }
}

// batches of kBatchMin tokens and more
static hipError_t launch_batch(int variant, const CoefArgs &a, const double *q, hipStream_t s)
{
    return a.nb <= 4 ? batch_t<1>(variant, a, q, s) : batch_t<2>(variant, a, q, s);
}

}  // namespace cdk
