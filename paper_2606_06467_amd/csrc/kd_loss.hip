// The distillation loss of Eq. 6 and its gradient (Section 2.2).  P = abar (a
// constant), Q = softmax(I_t) over the valid keys, I the unscaled index scores
// of Eq. 3; the loss is the mean over rows with at least one key of KL(P || Q),
// dL/dI = (Q - P) / n_rows, dq = dL/dI K_idx and dk = dL/dI^T Q_idx.
//
// The scores are never stored: they cost 512 operations per (row, key) on the
// bf16 matrix cores, less than writing and reading them back, so each pass
// recomputes its tiles.
//   * kd_limits_kernel, kd_count_kernel: the most keys of any row of each 64-row
//     block, and the number of rows with keys;
//   * kd_stats_kernel: the log-sum-exp of every row (online, log2 units);
//   * kd_grad_kernel: one workgroup holds 128 rows (dq, with the row terms) or
//     128 keys (dk) in registers, 32 per wave, and streams the other side
//     through LDS 64 vectors at a time, double-buffered.  Per tile a wave makes
//     32 x 64 scores (v_mfma_f32_32x32x16_bf16; lane l supplies A row / B column
//     (l & 31) for contraction indices 8 * (l >> 5) .. + 8 and receives C rows
//     8 * (r >> 2) + 4 * (l >> 5) + (r & 3) of column (l & 31)), turns them into
//     Q - P in its registers, and multiplies them with the same staged vectors,
//     read transposed (ds_read_b64_tr_b16).
//     Q - P keeps all of its 24 bits: it is cut into three bf16 pieces of 8
//     bits each (exact), and each piece has a matrix product of its own
//     accumulated in fp32; the bf16 vectors enter exactly;
//     What bounds it: the register file.  128 accumulators, 64 registers of own
//     vectors and the pipeline's scores, targets and pieces leave one wave per
//     SIMD, so the matrix products (64 per 32 x 32 pairs, 2048 cycles) have only
//     their own wave's vector work to overlap with; they are busy a third of the
//     time.  Without the loads of abar the pass takes 1.2 instead of 1.5 ms.
//   Measured, 32768 causal rows (5.4e8 pairs): scores stored and read back, row
//   terms, and both gradients in fp32 matrix instructions 14.6 ms (dq 3.35, dk
//   7.1, scores 2.07, rows 1.77); this file with the steps of a tile one after
//   another 4.5; pipelined with the compiler's order 4.1, in a pinned order 3.35,
//   with operand rings of four instead of eight 3.15 ms (statistics 0.36, dq and dk
//   1.3-1.4 each; the accumulators in AGPRs: kept in VGPRs it takes 4.3).
//   * kd_finish_rows_kernel, kd_finish_keys_kernel: the sums over the ranges of
//     the streamed side, where it is split to fill and balance the chip (a
//     fixed order: the result does not depend on timing);
//   * kd_loss_kernel: the mean row term, summed in double in a fixed order.
#include "clsa_internal.h"
#include "device_common.h"

namespace clsa {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));

constexpr float kLossLog2e = 1.4426950408889634f;
constexpr float kLossLn2 = 0.6931471805599453f;
constexpr int kIdxDim = 256;               // index vector width
constexpr int kGrTile = 64;                // streamed vectors per tile
constexpr int kGrBlock = 128;              // rows (keys) held by a workgroup
constexpr int kGrPitch = kIdxDim + 16;     // bf16 per staged vector (544 bytes): the 16-byte
                                           // reads of 8 vectors and the transposing reads of
                                           // 4 both fall on distinct banks
constexpr int kGrMaxList = 256;            // tiles of one range of rows (dk)
constexpr int kStWaves = 8;                // waves (of 32 rows) of the statistics pass

struct KdLossArgs {
    const float *abar;         // [rows, max_len]
    const uint16_t *q_idx;     // [rows, 256]
    const uint16_t *k_idx;     // index-key cache
    const int32_t *page_table, *seq_lens, *q_pos;
    float *lse2;               // [rows] log-sum-exp, log2 units
    float *row_kl;             // [splits_q, rows]
    float *stats;              // [0] = 1 / n_rows (0 when none), [1] = n_rows
    uint32_t *tile_info;       // [batch, row_tiles]: see kd_limits_kernel
    int32_t *flags;            // [splits, batch, blocks]: dk partial written
    float *part;               // partials of the statistics, dq or dk
    float *loss, *dq, *dk;
    int batch, n_q, rows, max_len, page_shift, max_pages, causal;
    int row_tiles;                        // 64-row blocks per sequence
    int blocks, splits, span;             // of the current launch: see the kernels
};

__device__ __forceinline__ int row_limit(const KdLossArgs &a, int b, int t) {
    return t < a.n_q ? valid_keys(a.seq_lens, a.q_pos, a.causal, b, b * a.n_q + t, a.max_len) : 0;
}

__device__ __forceinline__ int lanes_max(int x) {
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) x = max(x, __shfl_xor(x, d));
    return __builtin_amdgcn_readfirstlane(x);
}
__device__ __forceinline__ int lanes_min(int x) {
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) x = min(x, __shfl_xor(x, d));
    return __builtin_amdgcn_readfirstlane(x);
}
// Maximum / sum over lanes l and l ^ 32 (the two lanes of a column).
__device__ __forceinline__ float both_max(float x) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float both_sum(float x) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

__device__ __forceinline__ void write_row_count(const KdLossArgs &a, int n) {
    a.stats[0] = n > 0 ? 1.0f / (float)n : 0.0f;
    a.stats[1] = (float)n;
}

// One wave per 64-row block: the most keys of any row (bits 8 up) and the number
// of rows with keys (bits 0 .. 7).  A grid of one workgroup walks every block and
// counts the rows itself.
constexpr int kLimitThreads = 1024;
constexpr int kLimitOneGroup = 64;  // row blocks up to which one workgroup does both
__global__ __launch_bounds__(kLimitThreads) void kd_limits_kernel(KdLossArgs a) {
    __shared__ int s_cnt[kLimitThreads / 64];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, total = a.batch * a.row_tiles;
    int cnt = 0;
    for (int tile = blockIdx.x * (kLimitThreads / 64) + wave; tile < total;
         tile += gridDim.x * (kLimitThreads / 64)) {
        const int b = tile / a.row_tiles, t = (tile % a.row_tiles) * kGrTile + lane;
        const int n = row_limit(a, b, t);
        const uint32_t most = lanes_max(n);
        const uint32_t some = __builtin_popcountll(__builtin_amdgcn_ballot_w64(n > 0));
        if (lane == 0) a.tile_info[tile] = (most << 8) | some;
        cnt += (int)some;
    }
    if (gridDim.x > 1) return;
    if (lane == 0) s_cnt[wave] = cnt;
    __syncthreads();
    if (threadIdx.x == 0) {
        int n = 0;
        for (int w = 0; w < kLimitThreads / 64; ++w) n += s_cnt[w];
        write_row_count(a, n);
    }
}

// One workgroup: the rows with keys, from the blocks' counts.
__global__ __launch_bounds__(1024) void kd_count_kernel(KdLossArgs a) {
    __shared__ int s_cnt[16];
    int cnt = 0;
    for (int i = threadIdx.x; i < a.batch * a.row_tiles; i += 1024) cnt += (int)(a.tile_info[i] & 255u);
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) cnt += __shfl_xor(cnt, d);
    if ((threadIdx.x & 63) == 0) s_cnt[threadIdx.x >> 6] = cnt;
    __syncthreads();
    if (threadIdx.x == 0) {
        int n = 0;
        for (int w = 0; w < 16; ++w) n += s_cnt[w];
        write_row_count(a, n);
    }
}

// 64 streamed index vectors into registers (PER 16-byte pieces per thread) and
// from there into an LDS tile.  Query rows past the last and keys past `last`
// are clamped (and masked by the caller).
template <bool KEYS, bool PAGED, int NT>
struct VectorTile {
    static constexpr int PER = kGrTile * kIdxDim / 8 / NT;
    u32x4 v[PER];
    __device__ __forceinline__ void fetch(const KdLossArgs &a, int b, int y0, int last) {
        const int tid = threadIdx.x;
        if (!PAGED && y0 + kGrTile - 1 <= last) {  // uniform: one lane offset, uniform bases
            const uint16_t *base = (KEYS ? a.k_idx + (size_t)b * a.max_len * kIdxDim
                                         : a.q_idx + (size_t)b * a.n_q * kIdxDim) + (size_t)y0 * kIdxDim;
#pragma unroll
            for (int i = 0; i < PER; ++i)
                v[i] = *reinterpret_cast<const u32x4 *>(base + i * (NT / 32) * kIdxDim + tid * 8);
            return;
        }
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int y = min(y0 + (tid >> 5) + i * (NT / 32), last);
            size_t off;
            if (!KEYS) off = (size_t)b * a.n_q + y;
            else if (!PAGED) off = (size_t)b * a.max_len + y;
            else
                off = ((size_t)a.page_table[(size_t)b * a.max_pages + (y >> a.page_shift)] << a.page_shift) +
                      (y & ((1 << a.page_shift) - 1));
            v[i] = *reinterpret_cast<const u32x4 *>((KEYS ? a.k_idx : a.q_idx) + off * kIdxDim +
                                                    (tid & 31) * 8);
        }
    }
    __device__ __forceinline__ void stage(uint16_t (*s)[kGrPitch]) const {
#pragma unroll
        for (int i = 0; i < PER; ++i)
            *reinterpret_cast<u32x4 *>(&s[(threadIdx.x >> 5) + i * (NT / 32)][(threadIdx.x & 31) * 8]) = v[i];
    }
};

// The wave's own 32 vectors as B operands (column l & 31).
__device__ __forceinline__ void load_own(const uint16_t *p, int hi, bf16x8 (&x)[16]) {
#pragma unroll
    for (int s = 0; s < 16; ++s)
        x[s] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(p + 16 * s + 8 * hi));
}

// Scores of 32 staged vectors (from row 32 kt of the tile) with the wave's own 32.
__device__ __forceinline__ void tile_scores(const uint16_t (*s)[kGrPitch], int kt, int col, int hi,
                                            const bf16x8 (&x)[16], f32x16 &c) {
#pragma unroll
    for (int r = 0; r < 16; ++r) c[r] = 0.0f;
#pragma unroll
    for (int ks = 0; ks < 16; ++ks) {
        const bf16x8 y = __builtin_bit_cast(
            bf16x8, *reinterpret_cast<const u32x4 *>(&s[32 * kt + col][16 * ks + 8 * hi]));
        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(y, x[ks], c, 0, 0, 0);
    }
}

// Row statistics: 8 waves x 32 rows and one range of keys per workgroup.  grid:
// (split * batch + b) * blocks + block, the last (causal: longest) rows first.
template <bool PAGED>
__global__ __launch_bounds__(64 * kStWaves, 2) void kd_stats_kernel(KdLossArgs a) {
    __shared__ __align__(16) uint16_t s_y[2][kGrTile][kGrPitch];
    __shared__ int s_lim[kStWaves];
    const int blk = a.blocks - 1 - (int)(blockIdx.x % a.blocks);
    const int b = (blockIdx.x / a.blocks) % a.batch, split = blockIdx.x / a.blocks / a.batch;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int col = lane & 31, hi = lane >> 5;
    const int t = (blk * kStWaves + wave) * 32 + col;
    const int n = row_limit(a, b, t);
    const int nmax = lanes_max(n), nmin = lanes_min(n);
    if (lane == 0) s_lim[wave] = nmax;
    bf16x8 x[16];
    load_own(a.q_idx + ((size_t)b * a.n_q + min(t, a.n_q - 1)) * kIdxDim, hi, x);
    __syncthreads();
    int wg_max = s_lim[0];
#pragma unroll
    for (int w = 1; w < kStWaves; ++w) wg_max = max(wg_max, s_lim[w]);
    const int j_begin = split * a.span, j_end = min(wg_max, j_begin + a.span);
    const int tiles = j_end > j_begin ? div_up(j_end - j_begin, kGrTile) : 0;
    float m = -INFINITY, l = 0.0f;
    VectorTile<true, PAGED, 64 * kStWaves> y;
    if (tiles > 0) {
        y.fetch(a, b, j_begin, wg_max - 1);
        y.stage(s_y[0]);
        __syncthreads();
    }
    for (int u = 0; u < tiles; ++u) {
        const int j0 = j_begin + u * kGrTile;
        y.fetch(a, b, j0 + kGrTile, wg_max - 1);  // past the range: never used
        if (j0 < nmax) {  // uniform per wave
            f32x16 c[2];
#pragma unroll
            for (int kt = 0; kt < 2; ++kt) tile_scores(s_y[u & 1], kt, col, hi, x, c[kt]);
            if (j0 + kGrTile > nmin) {
#pragma unroll
                for (int kt = 0; kt < 2; ++kt)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        c[kt][r] = j0 + 32 * kt + 8 * (r >> 2) + 4 * hi + (r & 3) < n ? c[kt][r] : -INFINITY;
            }
            float mx = fmaxf(c[0][0], c[1][0]);
#pragma unroll
            for (int r = 1; r < 16; ++r) mx = fmaxf(mx, fmaxf(c[0][r], c[1][r]));
            mx *= kLossLog2e;
            if (__builtin_amdgcn_ballot_w64(mx > m + 8.0f)) {  // the base lags by up to 2^8
                const float nm = fmaxf(m, mx);
                if (nm != -INFINITY) l *= __builtin_amdgcn_exp2f(m - nm);
                m = nm;
            }
            const float base = m == -INFINITY ? 0.0f : m;
            float sum[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int kt = 0; kt < 2; ++kt)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    sum[r & 3] += __builtin_amdgcn_exp2f(fmaf(c[kt][r], kLossLog2e, -base));
            l += (sum[0] + sum[1]) + (sum[2] + sum[3]);
        }
        y.stage(s_y[(u + 1) & 1]);
        __syncthreads();
    }
    if (t >= a.n_q) return;
    const float M = both_max(m);
    const float L = both_sum(m == -INFINITY ? 0.0f : l * __builtin_amdgcn_exp2f(m - M));
    if (hi) return;
    const size_t row = (size_t)b * a.n_q + t;
    if (a.splits == 1) a.lse2[row] = n > 0 ? M + log2f(L) : 0.0f;
    else if (n > j_begin) *reinterpret_cast<float2 *>(a.part + ((size_t)split * a.rows + row) * 2) = make_float2(M, L);
}

// The ranges' statistics combined, one thread per row.
__global__ __launch_bounds__(256) void kd_stats_merge_kernel(KdLossArgs a) {
    const int row = blockIdx.x * 256 + threadIdx.x;
    if (row >= a.rows) return;
    const int n = valid_keys(a.seq_lens, a.q_pos, a.causal, row / a.n_q, row, a.max_len);
    float M = -INFINITY, L = 0.0f;
    const int used = div_up(n, a.span);
    for (int s = 0; s < used; ++s) {
        const float2 p = *reinterpret_cast<const float2 *>(a.part + ((size_t)s * a.rows + row) * 2);
        const float nm = fmaxf(M, p.x);
        const float base = nm == -INFINITY ? 0.0f : nm;
        L = L * exp2f(M - base) + p.y * exp2f(p.x - base);
        M = nm;
    }
    a.lse2[row] = n > 0 ? M + log2f(L) : 0.0f;
}

// Where the 256 values of row / key x go: the output, or the range's partial.
template <bool DK>
__device__ __forceinline__ float *grad_dst(const KdLossArgs &a, int b, int x, int split) {
    if (a.splits > 1) {
        const size_t own = DK ? (size_t)a.batch * a.max_len : (size_t)a.rows;
        const size_t at = DK ? (size_t)b * a.max_len + x : (size_t)b * a.n_q + x;
        return a.part + ((size_t)split * own + at) * kIdxDim;
    }
    return DK ? a.dk + token_offset(a.page_table, a.page_shift, a.max_pages, a.max_len, b, x, kIdxDim)
              : a.dq + ((size_t)b * a.n_q + x) * kIdxDim;
}

// Not an infinity and not a NaN.
__device__ __forceinline__ bool finite(float x) { return x - x == 0.0f; }

// Gradient of one side.  DK false: own = rows, streamed = keys, out = dq, and
// the rows' KL terms; true: own = keys, streamed = rows, out = dk.
// grid: (split * batch + b) * blocks + block.
// One wave per SIMD (128 accumulators, 64 registers of own vectors), so the loop
// overlaps its parts itself: per 32 streamed vectors it issues the products of
// step i, the scores of step i + 2 and, beside them on the vector unit, turns the
// scores of step i + 1 into Q - P and its three pieces.  Three LDS tiles (the
// scores run a tile ahead of the products), one barrier per tile.
template <bool DK, bool PAGED>
__global__ __launch_bounds__(256, 1) void kd_grad_kernel(KdLossArgs a) {
    __shared__ __align__(16) uint16_t s_y[3][kGrTile][kGrPitch];
    __shared__ int s_lim[4];
    __shared__ int s_list[DK ? kGrMaxList : 1];
    __shared__ __align__(16) float s_lse[DK ? 3 : 1][kGrTile];
    __shared__ __align__(16) int s_n[DK ? 3 : 1][kGrTile];
    const int b = (blockIdx.x / a.blocks) % a.batch, split = blockIdx.x / a.blocks / a.batch;
    // causal: the last rows see the most keys, the first keys are seen by the most rows
    const int blk = DK ? (int)(blockIdx.x % a.blocks) : a.blocks - 1 - (int)(blockIdx.x % a.blocks);
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int col = lane & 31, hi = lane >> 5;
    const int x0 = blk * kGrBlock + wave * 32, xi = x0 + col;  // this lane's row / key
    const int len = clamp_len(a.seq_lens[b], a.max_len);
    const int y_begin = split * a.span;
    int n = 0, tiles = 0, wg_max = 0;
    float lse = 0.0f;
    if (DK) {
        // the useful 64-row tiles of the range (a row that sees the block's
        // first key), in order
        const int tl = y_begin / kGrTile + tid;
        const uint32_t info =
            tid < a.span / kGrTile && tl < a.row_tiles ? a.tile_info[b * a.row_tiles + tl] : 0u;
        const bool useful = blk * kGrBlock < len && (int)(info >> 8) > blk * kGrBlock;
        const uint64_t mk = __builtin_amdgcn_ballot_w64(useful);
        if (lane == 0) s_lim[wave] = __builtin_popcountll(mk);
        __syncthreads();
        int off = 0;
        for (int w = 0; w < wave; ++w) off += s_lim[w];
        tiles = s_lim[0] + s_lim[1] + s_lim[2] + s_lim[3];
        if (useful) s_list[off + __builtin_popcountll(mk & ((1ull << lane) - 1ull))] = tl * kGrTile;
        if (tid == 0 && a.splits > 1)
            a.flags[((size_t)split * a.batch + b) * a.blocks + blk] = tiles > 0;
        if (tiles == 0 && (a.splits > 1 || blk * kGrBlock >= len)) return;  // uniform
        __syncthreads();
    } else {
        n = row_limit(a, b, xi);
        const int nmax = lanes_max(n);
        if (lane == 0) s_lim[wave] = nmax;
        __syncthreads();
        wg_max = max(max(s_lim[0], s_lim[1]), max(s_lim[2], s_lim[3]));
        const int j_end = min(wg_max, y_begin + a.span);
        tiles = j_end > y_begin ? div_up(j_end - y_begin, kGrTile) : 0;
        if (tiles == 0 && a.splits > 1) return;  // uniform
        if (n > 0) lse = a.lse2[(size_t)b * a.n_q + xi];
    }
    bf16x8 x[16];
    auto own_vectors = [&](int xi, int hi) {
        if (DK)
            load_own(a.k_idx + token_offset(a.page_table, a.page_shift, a.max_pages, a.max_len, b,
                                            min(xi, len - 1), kIdxDim), hi, x);
        else
            load_own(a.q_idx + ((size_t)b * a.n_q + min(xi, a.n_q - 1)) * kIdxDim, hi, x);
    };
    own_vectors(xi, hi);
    f32x16 acc[8];
#pragma unroll
    for (int d = 0; d < 8; ++d)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[d][r] = 0.0f;
    // the row term by tiles, so that a long range is no chain of its length
    float kl = 0.0f, total = 0.0f;

    // first vector of tile u (past the last: the last one again, nothing valid)
    auto start = [&](int u) {
        const int v = min(u, tiles - 1);
        return DK ? s_list[v] : y_begin + v * kGrTile;
    };
    VectorTile<!DK, PAGED, 256> y;
    float ylse = 0.0f;
    int yn = 0;
    auto fetch = [&](int y0) {
        y.fetch(a, b, y0, DK ? a.n_q - 1 : wg_max - 1);
        if (DK && tid < kGrTile) {
            const int t = y0 + tid;
            yn = row_limit(a, b, t);
            ylse = a.lse2[(size_t)b * a.n_q + min(t, a.n_q - 1)];
        }
    };
    auto stage = [&](int buf) {
        y.stage(s_y[buf]);
        if (DK && tid < kGrTile) {
            s_lse[buf][tid] = ylse;
            s_n[buf][tid] = yn;
        }
    };
    // abar of the lane's 16 (row, key) pairs of half a tile; what is not valid is
    // read from inside the buffer and not used
    const float *arow = a.abar + ((size_t)b * a.n_q + (DK ? 0 : min(xi, a.n_q - 1))) * a.max_len;
    const int jx = DK ? min(xi, len - 1) : 0;
    const uint32_t xoff = DK ? (uint32_t)(4 * hi) * (uint32_t)a.max_len + (uint32_t)jx : 0u;
    auto target = [&](int y0, float (&p)[16], float (&pn)[16]) {
        const bool inside = y0 + kGrTile <= (DK ? a.n_q : a.max_len);  // uniform
        if (inside) {
            const float *base = DK ? arow + (size_t)y0 * a.max_len : arow + y0 + 4 * hi;
#pragma unroll
            for (int e = 0; e < 32; ++e) {
                const int at = 8 * (e >> 2) + (e & 3);
                float &dst = e < 16 ? p[e] : pn[e - 16];
                if (DK) {
                    dst = (base + (size_t)at * a.max_len)[xoff];
                } else if ((e & 3) == 0) {
                    const f32x4u v = *reinterpret_cast<const f32x4u *>(base + at);
                    float *d4 = &dst;
                    d4[0] = v[0], d4[1] = v[1], d4[2] = v[2], d4[3] = v[3];
                }
            }
        } else {
#pragma unroll
            for (int e = 0; e < 32; ++e) {
                const int yy = y0 + 8 * (e >> 2) + 4 * hi + (e & 3);
                float &dst = e < 16 ? p[e] : pn[e - 16];
                dst = DK ? arow[(size_t)min(yy, a.n_q - 1) * a.max_len + jx] : arow[min(yy, a.max_len - 1)];
            }
        }
    };
    // Q - P of pairs e and e + 1 (e even) of half a tile, cut into three bf16
    // pieces, two pairs to a word
    auto pieces2 = [&](int e, int hi, float lse, const f32x16 &c, const float (&p)[16], int lim, int kt, int buf,
                       uint32_t (&pl)[3][8]) {
        uint32_t h[2], md[2], lo[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int yl = 32 * kt + 8 * (e >> 2) + 4 * hi + (e & 3) + k;
            const float z = fmaf(c[e + k], kLossLog2e, DK ? -s_lse[buf][yl] : -lse);
            const bool valid = DK ? lim < s_n[buf][yl] : yl < lim;
            const float pv = valid ? p[e + k] : 0.0f;
            const float q = valid ? __builtin_amdgcn_exp2f(z) : 0.0f;
            if constexpr (!DK) {
                // 0 log 0 = 0; the logarithm is clamped below 2^-126
                const float t = __builtin_amdgcn_logf(fmaxf(pv, 0x1p-126f)) - z;
                kl = pv > 0.0f ? fmaf(pv, t, kl) : kl;
            }
            const float d = q - pv;
            h[k] = __float_as_uint(d) & 0xffff0000u;
            const float d1 = d - __uint_as_float(h[k]);
            md[k] = __float_as_uint(d1) & 0xffff0000u;
            lo[k] = __float_as_uint(d1 - __uint_as_float(md[k]));
        }
        pl[0][e >> 1] = __builtin_amdgcn_perm(h[1], h[0], 0x07060302u);
        pl[1][e >> 1] = __builtin_amdgcn_perm(md[1], md[0], 0x07060302u);
        pl[2][e >> 1] = __builtin_amdgcn_perm(lo[1], lo[0], 0x07060302u);
    };
    // The limit that pieces2 compares with (nothing valid in a tile past the last).
    auto limit = [&](int y0, bool exists) {
        return exists ? (DK ? xi : n - y0) : (DK ? 0x7fffffff : 0);
    };
    const int yrow = 4 * hi + ((lane & 15) >> 2);                    // transposing reads
    const int ycol = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
    typedef __attribute__((address_space(3))) s16x4 lds4;
    bf16x8 v[4], w[4];  // operands read ahead
    auto read_at = [&](bf16x8 &v, int buf, int kt, int kb, int d, int yrow, int ycol) {
        const int yr = 32 * kt + 16 * kb + yrow;
        const s16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4 *)&s_y[buf][yr][32 * d + ycol]);
        const s16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4 *)&s_y[buf][yr + 8][32 * d + ycol]);
        v = __builtin_bit_cast(bf16x8, __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    auto read_v = [&](bf16x8 &v, int buf, int kt, int kb, int d) { read_at(v, buf, kt, kb, d, yrow, ycol); };
    auto read_w = [&](int buf, int kt, int ks) {
        w[ks & 3] = __builtin_bit_cast(
            bf16x8, *reinterpret_cast<const u32x4 *>(&s_y[buf][32 * kt + col][16 * ks + 8 * hi]));
    };
    // One step: the products of the pieces pl with half a tile (kt of tile buf),
    // the scores of half a tile of the next (kt of tile nbuf), and the pieces po
    // of the half tile between them (scores co), in 16 parts of four matrix
    // products that keep their order.  Operands are read from LDS two or three
    // parts before they are used; v holds the first two on entry, and the next
    // step's (half nkt of tile vbuf) on return.
    auto step = [&](const uint32_t (&pl)[3][8], int kt, int buf, int nbuf, f32x16 &c, const f32x16 &co,
                    const float (&po)[16], int lim, int obuf, uint32_t (&out)[3][8], int vbuf, int nkt) {
#pragma unroll
        for (int ks = 0; ks < 3; ++ks) read_w(nbuf, kt, ks);
#pragma unroll
        for (int r = 0; r < 16; ++r) c[r] = 0.0f;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int kb = e >> 3, d = e & 7;
            if (e < 14) read_v(v[(e + 2) & 3], buf, kt, (e + 2) >> 3, (e + 2) & 7);
            else read_v(v[(e + 2) & 3], vbuf, nkt, 0, e - 14);
            if (e + 3 < 16) read_w(nbuf, kt, e + 3);
#pragma unroll
            for (int i = 2; i >= 0; --i) {
                const bf16x8 pb = __builtin_bit_cast(bf16x8, u32x4{pl[i][4 * kb], pl[i][4 * kb + 1],
                                                                   pl[i][4 * kb + 2], pl[i][4 * kb + 3]});
                acc[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v[e & 3], pb, acc[d], 0, 0, 0);
            }
            if ((e & 1) == 0) pieces2(e, hi, lse, co, po, lim, kt ^ 1, obuf, out);
            c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[e & 3], x[e], c, 0, 0, 0);
            if (e & 1) __builtin_amdgcn_sched_barrier(0);
        }
    };
    if (tiles > 0) {  // uniform
        fetch(start(0));
        stage(0);
        fetch(start(1));
        stage(1);
        __syncthreads();
        f32x16 c0, c1;
        float p0[16], p1[16];  // abar of the next tile's first half, this tile's second
        uint32_t pl0[3][8], pl1[3][8];
        target(start(0), p0, p1);
        tile_scores(s_y[0], 0, col, hi, x, c0);
        tile_scores(s_y[0], 1, col, hi, x, c1);
#pragma unroll
        for (int e = 0; e < 16; e += 2) pieces2(e, hi, lse, c0, p0, limit(start(0), true), 0, 0, pl0);
#pragma unroll
        for (int d = 0; d < 2; ++d) read_v(v[d], 0, 0, 0, d);
        int buf = 0;
        for (int u = 0; u < tiles; ++u) {
            const int y0 = start(u), y1 = start(u + 1);
            const int nbuf = buf == 2 ? 0 : buf + 1, sbuf = nbuf == 2 ? 0 : nbuf + 1;
            float pn[16];
            target(y1, p0, pn);
            fetch(start(u + 2));
            __builtin_amdgcn_sched_barrier(0);
            step(pl0, 0, buf, nbuf, c0, c1, p1, limit(y0, true), buf, pl1, buf, 1);
            step(pl1, 1, buf, nbuf, c1, c0, p0, limit(y1, u + 1 < tiles), nbuf, pl0, nbuf, 0);
            stage(sbuf);
            if (!DK) {
                total += kl;
                kl = 0.0f;
            }
            __syncthreads();
            buf = nbuf;
#pragma unroll
            for (int r = 0; r < 16; ++r) p1[r] = pn[r];
        }
    }
    if (!DK) {
        kl = both_sum(total + kl);
        if (hi == 0 && xi < a.n_q) a.row_kl[(size_t)split * a.rows + (size_t)b * a.n_q + xi] = kl * kLossLn2;
    }
    const int own = DK ? len : a.n_q;
    if (x0 >= own) return;
    const float f = a.splits > 1 ? 1.0f : a.stats[0];
    // A streamed value that is not finite reaches the products of own vectors that do
    // not meet it (Q - P of zero does not remove it).  A wave with such a result makes
    // it again, 32 streamed vectors at a time in its own sixth of the tiles (the loop's
    // last barrier is behind every wave's last read): once the scores are made, values
    // that are not finite become zeros there and are added by hand for the pairs that
    // count.  8192 causal rows with one infinity 0.6 (a query) and 1.5 ms (a key), 0.4
    // without; one pair at a time it was hundreds of times the usual.
    float odd = 0.0f;
#pragma unroll
    for (int d = 0; d < 8; ++d)
#pragma unroll
        for (int r = 0; r < 16; ++r) odd = fmaf(acc[d][r], 0.0f, odd);
    if (__builtin_amdgcn_ballot_w64(odd != 0.0f && xi < own)) {
        // the lane's place and its own vectors are made again: held over the loop for
        // this they would spill
        const int lane = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
        const int col = lane & 31, hi = lane >> 5, xi = x0 + col;
        const int n = DK ? 0 : row_limit(a, b, xi);
        const float lse = n > 0 ? a.lse2[(size_t)b * a.n_q + xi] : 0.0f;
        const int sb = wave >> 1, sk = wave & 1, last = DK ? a.n_q - 1 : wg_max - 1;
        uint16_t(*slot)[kGrPitch] = &s_y[sb][32 * sk];
        auto vector_at = [&](int yy) {
            yy = min(yy, last);
            return DK ? a.q_idx + ((size_t)b * a.n_q + yy) * kIdxDim
                      : a.k_idx + token_offset(a.page_table, a.page_shift, a.max_pages, a.max_len, b, yy, kIdxDim);
        };
#pragma unroll
        for (int d = 0; d < 8; ++d)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[d][r] = 0.0f;
        own_vectors(xi, hi);
        for (int h = 0; h < 2 * tiles; ++h) {
            const int y0 = start(h >> 1) + 32 * (h & 1);
            const int lim = DK ? xi : n - y0 + 32 * sk;
#pragma unroll 4
            for (int i = 0; i < 16; ++i)
                *reinterpret_cast<u32x4 *>(&slot[2 * i + hi][col * 8]) =
                    *reinterpret_cast<const u32x4 *>(vector_at(y0 + 2 * i + hi) + col * 8);
            if (DK && lane < 32) {
                s_lse[sb][32 * sk + lane] = a.lse2[(size_t)b * a.n_q + min(y0 + lane, last)];
                s_n[sb][32 * sk + lane] = row_limit(a, b, y0 + lane);
            }
            __builtin_amdgcn_wave_barrier();
            f32x16 c;
            tile_scores(s_y[sb], sk, col, hi, x, c);
            __builtin_amdgcn_wave_barrier();
            uint32_t bad = 0u;  // streamed vectors with a value that is not finite
#pragma unroll 1
            for (int i = 0; i < 16; ++i) {
                u32x4 v = *reinterpret_cast<const u32x4 *>(&slot[2 * i + hi][col * 8]);
                bool some = false;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const bool lo = finite(bf16_lo(v[e])), up = finite(bf16_hi(v[e]));
                    some |= !lo || !up;
                    v[e] &= (lo ? 0x0000ffffu : 0u) | (up ? 0xffff0000u : 0u);
                }
                *reinterpret_cast<u32x4 *>(&slot[2 * i + hi][col * 8]) = v;
                const uint64_t rows = __builtin_amdgcn_ballot_w64(some);
                bad |= (((uint32_t)rows ? 1u : 0u) | ((uint32_t)(rows >> 32) ? 2u : 0u)) << (2 * i);
            }
            __builtin_amdgcn_wave_barrier();
            float p[16];
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int i = 8 * (e >> 2) + 4 * hi + (e & 3), yy = y0 + i;
                const bool valid = DK ? xi < s_n[sb][32 * sk + i] : yy < n;
                p[e] = valid ? a.abar[((size_t)b * a.n_q + (DK ? yy : xi)) * a.max_len + (DK ? xi : yy)] : 0.0f;
            }
            uint32_t pl[3][8];
#pragma unroll
            for (int e = 0; e < 16; e += 2) pieces2(e, hi, lse, c, p, lim, sk, sb, pl);
#pragma unroll
            for (int i = 0; i < 8; ++i) {  // an infinite Q - P (of an infinite target) is its first piece alone
                const uint32_t f = pl[0][i];
                const uint32_t keep = ((f & 0x7fffu) == 0x7f80u ? 0u : 0x0000ffffu) |
                                      ((f & 0x7fff0000u) == 0x7f800000u ? 0u : 0xffff0000u);
                pl[1][i] &= keep;
                pl[2][i] &= keep;
            }
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int d = 0; d < 8; ++d) {
                    bf16x8 v;
                    read_at(v, sb, sk, kb, d, 4 * hi + ((lane & 15) >> 2), 16 * ((lane >> 4) & 1) + 4 * (lane & 3));
#pragma unroll
                    for (int i = 2; i >= 0; --i)
                        acc[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                            v, __builtin_bit_cast(bf16x8, u32x4{pl[i][4 * kb], pl[i][4 * kb + 1],
                                                                pl[i][4 * kb + 2], pl[i][4 * kb + 3]}),
                            acc[d], 0, 0, 0);
                }
            __builtin_amdgcn_wave_barrier();
            for (; bad; bad &= bad - 1u) {  // uniform
                const int i = __builtin_ctz(bad);
                const bool valid = DK ? xi < s_n[sb][32 * sk + i] : y0 + i < n;
                // Q - P of vector i: pair 4 (i >> 3) + (i & 3) of lanes hi = (i >> 2) & 1
                float q = 0.0f;
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    float g = 0.0f;
#pragma unroll
                    for (int k = 0; k < 3; ++k) g += e & 1 ? bf16_hi(pl[k][e >> 1]) : bf16_lo(pl[k][e >> 1]);
                    q = e == 4 * (i >> 3) + (i & 3) ? g : q;
                }
                const auto both = __builtin_amdgcn_permlane32_swap(__float_as_uint(q), __float_as_uint(q), false, false);
                const float qt = __uint_as_float(both[0]), qu = __uint_as_float(both[1]);
                const uint16_t *yp = vector_at(y0 + i) + 4 * hi;
#pragma unroll
                for (int d = 0; d < 8; ++d)
#pragma unroll
                    for (int r = 0; r < 16; r += 4) {
                        const uint2 w = *reinterpret_cast<const uint2 *>(yp + 32 * d + 2 * r);
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            const uint32_t word = k < 2 ? w.x : w.y;
                            const float v = k & 1 ? bf16_hi(word) : bf16_lo(word);
                            if (valid && !finite(v)) acc[d][r + k] = fmaf((i >> 2) & 1 ? qu : qt, v, acc[d][r + k]);
                        }
                    }
            }
        }
    }
    if (xi >= own) return;
    float *dst = grad_dst<DK>(a, b, xi, split);
#pragma unroll
    for (int d = 0; d < 8; ++d)
#pragma unroll
        for (int r = 0; r < 16; r += 4)
            *reinterpret_cast<float4 *>(dst + 32 * d + 2 * r + 4 * hi) =
                make_float4(acc[d][r] * f, acc[d][r + 1] * f, acc[d][r + 2] * f, acc[d][r + 3] * f);
}

// Sums over the ranges: one thread per four columns of a row (dq, and its KL
// term) or of a key (dk).
__global__ __launch_bounds__(256) void kd_finish_rows_kernel(KdLossArgs a) {
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    const int row = (int)(i >> 6), c = (int)(i & 63) * 4;
    if (row >= a.rows) return;
    const int n = valid_keys(a.seq_lens, a.q_pos, a.causal, row / a.n_q, row, a.max_len);
    const int used = div_up(n, a.span);
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    float kl = 0.0f;
    for (int k = 0; k < used; ++k) {
        const float4 v = *reinterpret_cast<const float4 *>(a.part + ((size_t)k * a.rows + row) * kIdxDim + c);
        s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
        if (c == 0) kl += a.row_kl[(size_t)k * a.rows + row];
    }
    const float f = a.stats[0];
    *reinterpret_cast<float4 *>(a.dq + (size_t)row * kIdxDim + c) = make_float4(s.x * f, s.y * f, s.z * f, s.w * f);
    if (c == 0) a.row_kl[row] = kl;
}
__global__ __launch_bounds__(256) void kd_finish_keys_kernel(KdLossArgs a) {
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    const size_t at = i >> 6;  // b * max_len + j
    const int c = (int)(i & 63) * 4, b = (int)(at / a.max_len), j = (int)(at % a.max_len);
    if (b >= a.batch || j >= clamp_len(a.seq_lens[b], a.max_len)) return;
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int k = 0; k < a.splits; ++k) {
        if (!a.flags[((size_t)k * a.batch + b) * a.blocks + j / kGrBlock]) continue;
        const float4 v = *reinterpret_cast<const float4 *>(
            a.part + ((size_t)k * a.batch * a.max_len + at) * kIdxDim + c);
        s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
    }
    const float f = a.stats[0];
    *reinterpret_cast<float4 *>(a.dk + token_offset(a.page_table, a.page_shift, a.max_pages, a.max_len, b, j,
                                                    kIdxDim) + c) =
        make_float4(s.x * f, s.y * f, s.z * f, s.w * f);
}

// One workgroup: the mean row term.
__global__ __launch_bounds__(1024) void kd_loss_kernel(KdLossArgs a) {
    __shared__ double red[1024];
    const int tid = threadIdx.x;
    double tot = 0.0;
#pragma unroll 8
    for (int r = tid; r < a.rows; r += 1024) tot += (double)a.row_kl[r];
    red[tid] = tot;
    __syncthreads();
    for (int w = 512; w > 0; w >>= 1) {
        if (tid < w) red[tid] += red[tid + w];
        __syncthreads();
    }
    if (tid == 0) a.loss[0] = a.stats[1] > 0.0f ? (float)(red[0] / (double)a.stats[1]) : 0.0f;
}

static bool grid_fits(long long n) { return n >= 1 && n <= 0x7fffffffLL; }

bool kd_loss_supported(const Geometry &g) {
    return grid_fits((long long)g.batch * div_up(g.n_q, 64) * 4) &&
           grid_fits((long long)g.batch * div_up(g.max_len, 64) * 4);
}

// Ranges of the streamed side for `blocks` workgroups of a pass: about
// kGrWorkgroups in all (causal rows make unequal ranges: 32768 rows 3.8 ms with
// 2048 workgroups against 4.1 with 1024), each range a multiple of 64 and at least
// kGrMinSpan long.
constexpr int kGrWorkgroups = 2048, kGrMinSpan = 512;
static void plan_ranges(long blocks, int length, long most, int &splits, int &span) {
    const int tiles = div_up(length, kGrTile);
    long want = (kGrWorkgroups + blocks - 1) / blocks;
    const long cap = div_up(length, kGrMinSpan);
    if (want > cap) want = cap;
    if (want > most) want = most;
    if (want < 1) want = 1;
    span = div_up(tiles, (int)want) * kGrTile;
    splits = div_up(length, span);
}

size_t kd_loss_ws_floats(const Geometry &g) {
    return (size_t)g.rows * g.max_len + g.rows + 2 + (size_t)g.batch * div_up(g.n_q, 32);
}

// Ranges of the passes and the workspace (floats):
//   [partials of the statistics, then of dq][row terms: splits_q * rows]
//   [lse2: rows][stats: 2][tile_info][flags].
// The partials of dk come when the row terms are summed up, and take their place
// too.  With one range everywhere there are no partials and no flags, which the
// smallest workspace holds; each further range costs 256 floats and a row term per
// row (dq) or 256 floats and its flags per token (dk), taken from half of the rest
// each.  More than kGrMaxList row tiles need several ranges whatever is left: at
// 16384 rows a range their partials, 256 floats per token, are less than the row
// terms (16384 per token) even at one key per row, and their flags less than the
// half of kd_loss_ws_floats' last term that tile_info does not use.
KdLossPlan kd_loss_plan(const Geometry &g) {
    KdLossPlan p;
    const int q_blocks = div_up(g.n_q, kGrBlock), k_blocks = div_up(g.max_len, kGrBlock);
    const size_t rows = g.rows, tokens = (size_t)g.batch * g.max_len;
    const size_t room = rows * g.max_len;  // beside one row term per row, stats and tile_info
    const size_t left = room > rows ? room - rows : 0;
    const long most_q = (long)(left / (2 * rows * (kIdxDim + 1)));
    const long most_k = (long)(left / (2 * tokens * (kIdxDim + 1)));
    plan_ranges((long)g.batch * q_blocks, g.max_len, most_q, p.splits_q, p.span_q);
    plan_ranges((long)g.batch * k_blocks, g.n_q, most_k, p.splits_k, p.span_k);
    const int row_list = kGrMaxList * kGrTile;  // rows of one range: the kernel's tile list
    if (p.span_k > row_list) {
        p.span_k = row_list;
        p.splits_k = div_up(g.n_q, row_list);
    }
    const int s_blocks = div_up(g.n_q, 32 * kStWaves);
    plan_ranges((long)g.batch * s_blocks, g.max_len, most_q, p.splits_s, p.span_s);
    size_t part = 0;
    if (p.splits_q > 1) part = p.splits_q * rows * kIdxDim;
    if (p.splits_s > 1 && p.splits_s * rows * 2 > part) part = p.splits_s * rows * 2;
    p.row_kl = part;
    p.lse2 = part + p.splits_q * rows;
    if (p.splits_k > 1 && p.splits_k * tokens * kIdxDim > p.lse2) p.lse2 = p.splits_k * tokens * kIdxDim;
    p.stats = p.lse2 + rows;
    p.tile_info = p.stats + 2;
    p.flags = p.tile_info + (size_t)g.batch * div_up(g.n_q, kGrTile);
    p.floats = p.flags + (p.splits_k > 1 ? (size_t)p.splits_k * g.batch * k_blocks : 0);
    return p;
}

hipError_t launch_kd_loss(const Geometry &g, const float *abar, const void *q_idx,
                          const void *k_idx, const int32_t *page_table, const int32_t *seq_lens,
                          const int32_t *q_pos, float *loss, float *dq, float *dk, float *ws,
                          hipStream_t stream, hipEvent_t after_scores, hipEvent_t after_loss) {
    if (!kd_loss_supported(g)) return hipErrorInvalidValue;
    KdLossArgs a{};
    a.abar = abar;
    a.q_idx = static_cast<const uint16_t *>(q_idx);
    a.k_idx = static_cast<const uint16_t *>(k_idx);
    a.page_table = page_table;
    a.seq_lens = seq_lens;
    a.q_pos = q_pos;
    a.loss = loss;
    a.dq = dq;
    a.dk = dk;
    a.batch = g.batch;
    a.n_q = g.n_q;
    a.rows = g.rows;
    a.max_len = g.max_len;
    a.page_shift = g.page_shift;
    a.max_pages = g.max_pages;
    a.causal = g.causal;
    a.row_tiles = div_up(g.n_q, kGrTile);
    const KdLossPlan p = kd_loss_plan(g);
    if (p.floats > kd_loss_ws_floats(g)) return hipErrorInvalidValue;
    const int q_blocks = div_up(g.n_q, kGrBlock), k_blocks = div_up(g.max_len, kGrBlock);
    const int s_blocks = div_up(g.n_q, 32 * kStWaves);
    const size_t rows = g.rows, tokens = (size_t)g.batch * g.max_len;
    a.part = ws;
    a.row_kl = ws + p.row_kl;
    a.lse2 = ws + p.lse2;
    a.stats = ws + p.stats;
    a.tile_info = reinterpret_cast<uint32_t *>(ws + p.tile_info);
    a.flags = reinterpret_cast<int32_t *>(ws + p.flags);
    const bool paged = g.page_shift >= 0;
#define KD_LAUNCH(KERNEL, GRID, THREADS) \
    KERNEL<<<dim3((unsigned)(GRID)), dim3(THREADS), 0, stream>>>(a)

    const int row_blocks = g.batch * a.row_tiles;
    if (row_blocks <= kLimitOneGroup) {
        KD_LAUNCH(kd_limits_kernel, 1, kLimitThreads);
    } else {
        KD_LAUNCH(kd_limits_kernel, div_up(row_blocks, kLimitThreads / 64), kLimitThreads);
        KD_LAUNCH(kd_count_kernel, 1, 1024);
    }
    a.blocks = s_blocks;
    a.splits = p.splits_s;
    a.span = p.span_s;
    const long s_grid = (long)g.batch * s_blocks * p.splits_s;
    if (paged) KD_LAUNCH(kd_stats_kernel<true>, s_grid, 64 * kStWaves);
    else KD_LAUNCH(kd_stats_kernel<false>, s_grid, 64 * kStWaves);
    if (a.splits > 1) KD_LAUNCH(kd_stats_merge_kernel, div_up(g.rows, 256), 256);
    if (after_scores && hipEventRecord(after_scores, stream) != hipSuccess) return hipErrorUnknown;

    a.blocks = q_blocks;
    a.splits = p.splits_q;
    a.span = p.span_q;
    const long q_grid = (long)g.batch * q_blocks * a.splits;
    if (paged) KD_LAUNCH((kd_grad_kernel<false, true>), q_grid, 256);
    else KD_LAUNCH((kd_grad_kernel<false, false>), q_grid, 256);
    if (a.splits > 1) KD_LAUNCH(kd_finish_rows_kernel, (rows * 64 + 255) / 256, 256);
    KD_LAUNCH(kd_loss_kernel, 1, 1024);
    if (after_loss && hipEventRecord(after_loss, stream) != hipSuccess) return hipErrorUnknown;

    a.blocks = k_blocks;
    a.splits = p.splits_k;
    a.span = p.span_k;
    const long k_grid = (long)g.batch * k_blocks * a.splits;
    if (paged) KD_LAUNCH((kd_grad_kernel<true, true>), k_grid, 256);
    else KD_LAUNCH((kd_grad_kernel<true, false>), k_grid, 256);
    if (a.splits > 1) KD_LAUNCH(kd_finish_keys_kernel, (tokens * 64 + 255) / 256, 256);
#undef KD_LAUNCH
    return hipGetLastError();
}

hipError_t take_device_error_kd_loss(uint32_t *bits) { return take_source_device_error(bits); }

}  // namespace clsa
