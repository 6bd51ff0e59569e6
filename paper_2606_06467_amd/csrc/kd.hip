// Training side of the shared indexer (Section 2.2): the distillation target
// of Eq. 5 (its loss, Eq. 6, is in kd_loss.hip).
//
// Eq. 5: abar[b,t,j] = (1 / (L * Hq)) * sum over layers l and query heads h of
// softmax_j(scale * q_l[b,t,h] . K[b,j,g(h)]) over the valid keys of row (b,t),
// one shared key cache for every layer.  Logits on the bf16 matrix cores:
//   * kd_lse_kernel: an online softmax over the row's keys gives each row's
//     log-sum-exp (log2 units, in the workspace).  When the caller already has
//     these log-sum-exps (the dense forward pass of every layer makes them),
//     kd_lse_import_kernel copies them in instead;
//   * kd_target_kernel: per (16-row, 64-key) tile, every (layer, head) adds
//     exp(logit - lse) into the tile held in registers; the key operands of a
//     KV head are loaded once for all layers and heads of its group, the four
//     waves of a workgroup share their rows' query operands, and abar is
//     written once, with no atomics (v_mfma_f32_16x16x32_bf16: A = 16 query rows
//     x 32 dims, B = 32 dims x 16 keys; lane l supplies row / key (l & 15) for
//     dims (l >> 4) * 8 .. +8 and receives rows 4 * (l >> 4) + r of key (l & 15)).
#include "clsa_internal.h"
#include "device_common.h"

namespace clsa {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr float kKdLog2e = 1.4426950408889634f;
constexpr int kKdDim = 128;  // attention head dimension
constexpr int kKdTile = 64;  // rows and keys per target tile

struct KdArgs {
    const uint16_t *q_layers;  // [L, rows, Hq, 128]
    const uint16_t *k_cache;   // [B, max_len, Hkv, 128] | paged
    const int32_t *page_table, *seq_lens, *q_pos;
    float *lse2;               // [L, Hq, rows_pad], log2 units (rows_pad = rows + 16)
    float *abar;               // [rows, max_len]
    int n_layers, batch, n_q, rows, max_len, page_shift, max_pages, causal;
    int q_heads, kv_heads, group, row_tiles, key_tiles, rows_pad;
    float scale_log2, inv_lh;  // softmax_scale * log2(e), 1 / (L * Hq)
};

// 2^x by the hardware instruction alone: results below 2^-126 may flush to
// zero, which is far below every tolerance here (exp2f adds a rescaling for
// such results, five more VALU operations per call).
__device__ __forceinline__ float kd_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

__device__ __forceinline__ bf16x8 kd_ld8(const uint16_t *p) {
    return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(p));
}

// Key limits of the lane's four rows t0 + 4 * grp + r (0 for rows past n_q).
__device__ __forceinline__ void kd_row_limits(const KdArgs &a, int b, int t0, int grp,
                                              int (&n)[4]) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int t = t0 + 4 * grp + r;
        n[r] = t < a.n_q ? valid_keys(a.seq_lens, a.q_pos, a.causal, b, b * a.n_q + t, a.max_len)
                         : 0;
    }
}

// B operands of keys j0 + 16 * ct + col of KV head g (keys past len clamped to
// the last one; their logits are masked by the caller).  Paged caches: the four
// page-table reads are issued together, before the key reads.
template <bool PAGED>
__device__ __forceinline__ void kd_load_keys(const KdArgs &a, int b, int j0, int len, int g,
                                             int col, int grp, bf16x8 (&kv)[4][4]) {
    size_t tok[4];
#pragma unroll
    for (int ct = 0; ct < 4; ++ct) {
        const int j = min(j0 + 16 * ct + col, len - 1);
        if (PAGED) {
            const int page = a.page_table[(size_t)b * a.max_pages + (j >> a.page_shift)];
            tok[ct] = ((size_t)page << a.page_shift) + (j & ((1 << a.page_shift) - 1));
        } else {
            tok[ct] = (size_t)b * a.max_len + j;
        }
    }
#pragma unroll
    for (int ct = 0; ct < 4; ++ct) {
        const uint16_t *p = a.k_cache + (tok[ct] * a.kv_heads + g) * kKdDim + grp * 8;
#pragma unroll
        for (int kb = 0; kb < 4; ++kb) kv[ct][kb] = kd_ld8(p + kb * 32);
    }
}

// Unscaled logits of the lane's 4 rows x 4 keys: c[ct][r] = row 4 * grp + r,
// key 16 * ct + col.
__device__ __forceinline__ void kd_logits(const bf16x8 (&qa)[4], const bf16x8 (&kv)[4][4],
                                          f32x4 (&c)[4]) {
#pragma unroll
    for (int ct = 0; ct < 4; ++ct) {
        c[ct] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kb = 0; kb < 4; ++kb)
            c[ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qa[kb], kv[ct][kb], c[ct], 0, 0, 0);
    }
}

// Largest / smallest of a per-lane-group value over the four groups of a wave.
__device__ __forceinline__ int kd_groups_max(int v) {
    v = max(v, __shfl_xor(v, 16));
    return max(v, __shfl_xor(v, 32));
}
__device__ __forceinline__ int kd_groups_min(int v) {
    v = min(v, __shfl_xor(v, 16));
    return min(v, __shfl_xor(v, 32));
}

// The log-sum-exps of every (layer, row, query head) supplied by the caller
// (natural log, [L, rows, Hq], as the dense attention returns them) into the
// statistics layout [L, Hq, rows_pad] in log2 units.  grid-stride over L*rows*Hq.
__global__ __launch_bounds__(256) void kd_lse_import_kernel(KdArgs a, const float *lse_in) {
    const size_t total = (size_t)a.n_layers * a.rows * a.q_heads;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (size_t)gridDim.x * 256) {
        const int h = (int)(i % a.q_heads);
        const size_t lr = i / a.q_heads;
        const int r = (int)(lr % a.rows), l = (int)(lr / a.rows);
        a.lse2[((size_t)l * a.q_heads + h) * a.rows_pad + r] = lse_in[i] * kKdLog2e;
    }
}

// IEEE maximum (gfx950 v_maximum3_f32; no operand canonicalisation).
__device__ __forceinline__ float kd_max(float x, float y) {
    return __builtin_elementwise_maximum(x, y);
}

constexpr int kStagePitch = kKdDim + 8;  // bf16 per staged row (272 bytes): the 16 rows read
                                         // by one 16-lane group fall on distinct banks

constexpr int kLseWaves = 4;
// Workgroups of the statistics pass from which a wave takes two items: two rounds
// of the 512 such workgroups the chip holds.  Below, one item per wave fills it
// better (32 / 8 heads, 1000 rows, 4 layers, 512 workgroups: 96 us with one, 103
// with two; 8 / 8, 500 rows, 2 layers: 36 and 42); above, two share every key read
// (16384 rows, 16 layers: 37.8 ms with one, 36.0 with two; about 1000 and 1500
// workgroups measured the same either way).
constexpr int kLseWide = 1024;

// Log-sum-exp (log2 units) of every (layer, query head, row): a wave holds the
// queries of IT (32-row block, query head) items of one KV head and layer in
// registers (B of v_mfma_f32_32x32x16_bf16: lane l supplies column (l & 31) for
// dims 8 * (l >> 5) .. + 8 and receives rows 8 * (r >> 2) + 4 * (l >> 5) + (r & 3)
// of that column), and the KV head's keys stream through LDS 64 at a time,
// double-buffered and shared by the four waves (one barrier per tile); each key
// operand serves every item.  The logits come transposed, 32 keys of one row per
// lane, so a row's base and sum are one value per lane, the lanes' statistics are
// combined once at the end, and the maximum of a tile is 16 three-operand maxima.
// What bounds the pass is the vector work on the logits (it and the matrix
// products hardly overlap on this chip): an fma, an exp2, an add and half a
// maximum each.  The base follows the running maximum lazily: it moves only when a
// logit exceeds it by more than 2^kLazyMargin (a branch the whole wave takes).
// Measured, both passes of the target, against 16 rows x 16 keys per product with
// four rows per lane (5.75 vector operations per logit): 16384 rows, 16 layers, 32
// / 8 heads 35.2 ms against 37.4; 3000 rows, 8 layers, 20 / 4 heads 459 us against
// 623; 500 rows, 2 layers, 32 / 8 heads 54 against 62.
// grid: ((b * blocks + block of 4 * IT items) * L + l) * kv_heads + g, the last
// rows first; the workgroups of one KV head land on the same XCD when kv_heads
// divides 8.
constexpr float kLazyMargin = 16.0f;
template <int G, int IT, bool PAGED>  // G: query heads per KV head, IT: items per wave
__global__ __launch_bounds__(64 * kLseWaves, 2) void kd_lse_kernel(KdArgs a) {
    __shared__ __align__(16) uint16_t s_k[2][kKdTile][kStagePitch];
    __shared__ int s_nmax[kLseWaves];
    int x = blockIdx.x;
    const int g = x % a.kv_heads;
    x /= a.kv_heads;
    const int l = x % a.n_layers;
    x /= a.n_layers;
    const int blk = a.row_tiles - 1 - x % a.row_tiles, b = x / a.row_tiles;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, hi = lane >> 5;
    const int len = clamp_len(a.seq_lens[b], a.max_len);
    int t[IT], h[IT], n[IT], nmax = 0, nmin = a.max_len;
    bf16x8 q[IT][8];
#pragma unroll
    for (int i = 0; i < IT; ++i) {
        const int item = (blk * kLseWaves + wave) * IT + i;
        h[i] = g * G + item % G;
        t[i] = item / G * 32 + col;
        n[i] = t[i] < a.n_q
                   ? valid_keys(a.seq_lens, a.q_pos, a.causal, b, b * a.n_q + t[i], a.max_len) : 0;
        nmax = max(nmax, n[i]);
        nmin = min(nmin, n[i]);
        const uint16_t *p = a.q_layers +
                            (((size_t)l * a.rows + (size_t)b * a.n_q + min(t[i], a.n_q - 1)) * a.q_heads +
                             h[i]) * kKdDim + hi * 8;
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) q[i][ks] = kd_ld8(p + 16 * ks);
    }
#pragma unroll
    for (int d = 1; d < 32; d <<= 1) {
        nmax = max(nmax, __shfl_xor(nmax, d));
        nmin = min(nmin, __shfl_xor(nmin, d));
    }
    nmax = __builtin_amdgcn_readfirstlane(nmax);
    nmin = __builtin_amdgcn_readfirstlane(nmin);
    if (lane == 0) s_nmax[wave] = nmax;
    float m[IT], s[IT];  // base (log2 units) and sum
#pragma unroll
    for (int i = 0; i < IT; ++i) {
        m[i] = -INFINITY;
        s[i] = 0.0f;
    }
    __syncthreads();
    const int wg_max = max(max(s_nmax[0], s_nmax[1]), max(s_nmax[2], s_nmax[3]));
    const int tiles = div_up(wg_max, kKdTile);

    // staging: thread -> key row kr of the tile, 16-byte pieces 4 * kq .. 4 * kq + 3
    const int kr = tid >> 2, kq = tid & 3;
    auto fetch = [&](int u, u32x4 (&v)[4]) {
        const int j = min(u * kKdTile + kr, len - 1);
        size_t tok;
        if (PAGED) {
            const int page = a.page_table[(size_t)b * a.max_pages + (j >> a.page_shift)];
            tok = ((size_t)page << a.page_shift) + (j & ((1 << a.page_shift) - 1));
        } else {
            tok = (size_t)b * a.max_len + j;
        }
        const uint16_t *p = a.k_cache + (tok * a.kv_heads + g) * kKdDim + kq * 32;
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = *reinterpret_cast<const u32x4 *>(p + i * 8);
    };
    auto stage = [&](int buf, const u32x4 (&v)[4]) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            *reinterpret_cast<u32x4 *>(&s_k[buf][kr][kq * 32 + i * 8]) = v[i];
    };
    u32x4 v[4];
    if (tiles > 0) {
        fetch(0, v);
        stage(0, v);
    }
    __syncthreads();
    for (int u = 0; u < tiles; ++u) {
        if (u + 1 < tiles) fetch(u + 1, v);
        const int j0 = u * kKdTile;
        if (j0 < nmax) {  // uniform per wave
            f32x16 c[IT][2];  // [item][half of the tile]
#pragma unroll
            for (int kt = 0; kt < 2; ++kt) {
#pragma unroll
                for (int i = 0; i < IT; ++i)
#pragma unroll
                    for (int r = 0; r < 16; ++r) c[i][kt][r] = 0.0f;
#pragma unroll
                for (int ks = 0; ks < 8; ++ks) {
                    const bf16x8 k = *reinterpret_cast<const bf16x8 *>(
                        &s_k[u & 1][32 * kt + col][16 * ks + 8 * hi]);
#pragma unroll
                    for (int i = 0; i < IT; ++i)
                        c[i][kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k, q[i][ks], c[i][kt], 0, 0, 0);
                }
            }
            if (j0 + kKdTile > nmin) {  // uniform per wave
#pragma unroll
                for (int i = 0; i < IT; ++i)
#pragma unroll
                    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
                        for (int r = 0; r < 16; ++r)
                            c[i][kt][r] = j0 + 32 * kt + 8 * (r >> 2) + 4 * hi + (r & 3) < n[i] ? c[i][kt][r]
                                                                                               : -INFINITY;
            }
            float mx[IT];
            bool over = false;
#pragma unroll
            for (int i = 0; i < IT; ++i) {
                float w = kd_max(c[i][0][0], c[i][1][0]);
#pragma unroll
                for (int r = 1; r < 16; ++r) w = kd_max(kd_max(w, c[i][0][r]), c[i][1][r]);
                mx[i] = w * a.scale_log2;
                over |= mx[i] > m[i] + kLazyMargin;
            }
            if (__builtin_amdgcn_ballot_w64(over)) {
#pragma unroll
                for (int i = 0; i < IT; ++i) {
                    const float nb = kd_max(m[i], mx[i]);
                    if (nb != -INFINITY) {
                        s[i] *= kd_exp2(m[i] - nb);  // base = -inf: s is 0 anyway
                        m[i] = nb;
                    }
                }
            }
#pragma unroll
            for (int i = 0; i < IT; ++i) {
                const float base = m[i] == -INFINITY ? 0.0f : m[i];  // no key of the lane yet
                float sum[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int kt = 0; kt < 2; ++kt)
#pragma unroll
                    for (int r = 0; r < 16; ++r) sum[r & 3] += kd_exp2(fmaf(c[i][kt][r], a.scale_log2, -base));
                s[i] += (sum[0] + sum[1]) + (sum[2] + sum[3]);
            }
        }
        if (u + 1 < tiles) stage((u + 1) & 1, v);
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < IT; ++i) {
        auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(m[i]), __float_as_uint(m[i]), false, false);
        const float mr = kd_max(__uint_as_float(r[0]), __uint_as_float(r[1]));
        const float part = m[i] == -INFINITY ? s[i] : s[i] * exp2f(m[i] - mr);
        r = __builtin_amdgcn_permlane32_swap(__float_as_uint(part), __float_as_uint(part), false, false);
        const float sr = __uint_as_float(r[0]) + __uint_as_float(r[1]);
        if (hi == 0 && t[i] < a.n_q)
            a.lse2[((size_t)l * a.q_heads + h[i]) * a.rows_pad + (size_t)b * a.n_q + t[i]] =
                n[i] > 0 ? mr + log2f(sr) : -INFINITY;
    }
}

constexpr int kTgtChunk = 4;              // (layer, head) combinations per LDS stage
constexpr int kTgtWaveTiles = 1;          // 64-key tiles per wave in the target pass

template <bool FULL>
__device__ __forceinline__ void kd_accumulate(float sl, const bf16x8 (&qa)[4],
                                              const float4 &lse, const bf16x8 (&kv)[4][4],
                                              int j0, int col, const int (&n)[4],
                                              f32x4 (&acc)[4]) {
    f32x4 c[4];
    kd_logits(qa, kv, c);
    const float lr[4] = {lse.x, lse.y, lse.z, lse.w};
#pragma unroll
    for (int ct = 0; ct < 4; ++ct)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float e = kd_exp2(fmaf(c[ct][r], sl, -lr[r]));
            if (FULL) acc[ct][r] += e;
            else acc[ct][r] += j0 + 16 * ct + col < n[r] ? e : 0.0f;
        }
}

// A workgroup covers 16 rows x (4 * kTgtWaveTiles * 64) keys: each of its four
// waves holds the key operands of kTgtWaveTiles 64-key tiles of the current KV
// head in registers, and the query operands and log-sum-exps of the 16 rows
// are staged through LDS, kTgtChunk (layer, head) combinations at a time,
// double-buffered: the next stage's global reads are in flight while the
// current one is on the matrix cores, one barrier per stage.  Each staged query
// tile serves every key tile of the workgroup, so the query traffic per output
// falls with the keys a workgroup covers.  Workgroups are dealt to the 8 XCDs
// in turn; the mapping gives every key block of a row block to the same XCD,
// one after another, so the 2 MB of query operands of a row block (16 rows x
// every layer and head) are read from that XCD's L2 as far as it holds them.
// grid: ((row block group * key_blocks + key block) * 8 + xcd); row block
// index over all sequences = row block group * 8 + xcd.
template <int G, bool PAGED>  // G: query heads per KV head
__global__ __launch_bounds__(256) void kd_target_kernel(KdArgs a) {
    constexpr int KT = kTgtWaveTiles;
    __shared__ __align__(16) uint16_t s_q[2][kTgtChunk][16][kStagePitch];
    __shared__ __align__(16) float s_l[2][kTgtChunk][16];
    const int xcd = blockIdx.x & 7, local = blockIdx.x >> 3;
    const int kblk = local % a.key_tiles;
    const int rb_all = (local / a.key_tiles) * 8 + xcd;
    if (rb_all >= a.batch * a.row_tiles) return;  // padding of the last group (uniform)
    const int rblk = rb_all % a.row_tiles, b = rb_all / a.row_tiles;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int col = lane & 15, grp = lane >> 4;
    const int t0 = rblk * 16;
    const int jw = (kblk * 4 + wave) * KT * kKdTile;  // this wave's first key
    int n[4];
    kd_row_limits(a, b, t0, grp, n);
    const int nmax = kd_groups_max(max(max(n[0], n[1]), max(n[2], n[3])));
    const int nmin = kd_groups_min(min(min(n[0], n[1]), min(n[2], n[3])));
    if (kblk * 4 * KT * kKdTile >= nmax) return;  // no valid key in the block (uniform)
    const bool active = jw < nmax;                 // this wave's tiles hold valid keys
    const bool full = jw + KT * kKdTile <= nmin;
    const int len = clamp_len(a.seq_lens[b], a.max_len);

    // staging: thread -> (row sr, 16-byte piece sd) of every combination of a stage
    const int sr = tid >> 4, sd = tid & 15;
    const size_t layer_q = (size_t)a.rows * a.q_heads * kKdDim;
    const uint16_t *qsrc = a.q_layers +
                           ((size_t)b * a.n_q + min(t0 + sr, a.n_q - 1)) * a.q_heads * kKdDim +
                           sd * 8;
    // Combination ci = l * G + hh of KV head g is (layer l, query head g * G + hh);
    // a stage holds kTgtChunk consecutive combinations of one KV head.  G is a
    // compile-time constant, so the index arithmetic has no division.
    const int combos = a.n_layers * G;
    const int nchunk = div_up(combos, kTgtChunk);
    auto fetch = [&](int g, int c0, u32x4 (&v)[kTgtChunk], float &lv) {
#pragma unroll
        for (int c = 0; c < kTgtChunk; ++c) {
            const int ci = min(c0 + c, combos - 1);
            const int l = ci / G, h = g * G + ci % G;
            v[c] = *reinterpret_cast<const u32x4 *>(qsrc + l * layer_q + (size_t)h * kKdDim);
        }
        if (tid < kTgtChunk * 16) {
            const int ci = min(c0 + (tid >> 4), combos - 1);
            const int l = ci / G, h = g * G + ci % G;
            lv = a.lse2[((size_t)l * a.q_heads + h) * a.rows_pad + (size_t)b * a.n_q + t0 +
                        (tid & 15)];
        }
    };
    auto stage = [&](int buf, const u32x4 (&v)[kTgtChunk], float lv) {
#pragma unroll
        for (int c = 0; c < kTgtChunk; ++c)
            *reinterpret_cast<u32x4 *>(&s_q[buf][c][sr][sd * 8]) = v[c];
        if (tid < kTgtChunk * 16) s_l[buf][tid >> 4][tid & 15] = lv;
    };

    f32x4 acc[KT][4];
#pragma unroll
    for (int kt = 0; kt < KT; ++kt)
#pragma unroll
        for (int ct = 0; ct < 4; ++ct) acc[kt][ct] = f32x4{0.f, 0.f, 0.f, 0.f};
    u32x4 v[kTgtChunk];
    float lv = 0.0f;
    fetch(0, 0, v, lv);
    stage(0, v, lv);
    __syncthreads();
    bf16x8 kv[KT][4][4];
    // stage u = (KV head g, block k of kTgtChunk combinations), walked in order
    int g = 0, k = 0, buf = 0;
    for (;;) {
        if (k == 0 && active) {
#pragma unroll
            for (int kt = 0; kt < KT; ++kt)
                kd_load_keys<PAGED>(a, b, jw + kt * kKdTile, len, g, col, grp, kv[kt]);
        }
        const int k1 = k + 1 == nchunk ? 0 : k + 1, g1 = k + 1 == nchunk ? g + 1 : g;
        const bool more = g1 < a.kv_heads;
        if (more) fetch(g1, k1 * kTgtChunk, v, lv);
        if (active) {
#pragma unroll
            for (int c = 0; c < kTgtChunk; ++c) {
                if (k * kTgtChunk + c >= combos) break;  // uniform: short last stage
                bf16x8 qa[4];
#pragma unroll
                for (int kb = 0; kb < 4; ++kb)
                    qa[kb] = *reinterpret_cast<const bf16x8 *>(&s_q[buf][c][col][kb * 32 + grp * 8]);
                const float4 lse = *reinterpret_cast<const float4 *>(&s_l[buf][c][4 * grp]);
#pragma unroll
                for (int kt = 0; kt < KT; ++kt) {
                    if (full)
                        kd_accumulate<true>(a.scale_log2, qa, lse, kv[kt], jw + kt * kKdTile, col,
                                            n, acc[kt]);
                    else
                        kd_accumulate<false>(a.scale_log2, qa, lse, kv[kt], jw + kt * kKdTile,
                                             col, n, acc[kt]);
                }
            }
        }
        if (more) stage(buf ^ 1, v, lv);
        __syncthreads();
        if (!more) break;
        g = g1;
        k = k1;
        buf ^= 1;
    }
    if (!active) return;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int t = t0 + 4 * grp + r;
        float *row = a.abar + ((size_t)b * a.n_q + t) * a.max_len;
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
#pragma unroll
            for (int ct = 0; ct < 4; ++ct) {
                const int j = jw + kt * kKdTile + 16 * ct + col;
                if (j < n[r]) row[j] = acc[kt][ct][r] * a.inv_lh;
            }
    }
}

static bool grid_fits(long long n) { return n >= 1 && n <= 0x7fffffffLL; }

// Row blocks of 16 and key blocks of 256 for the target pass; the lane offsets
// into one layer's queries must fit 32 bits.
bool kd_target_supported(const Geometry &g, int n_layers) {
    const long long tiles = (long long)g.batch * div_up(g.n_q, kKdTile);
    const long long blocks = (long long)g.batch * div_up(g.n_q, 16);
    return n_layers >= 1 && grid_fits(tiles * n_layers * g.q_heads) &&
           grid_fits((blocks + 7) / 8 * 8 * div_up(g.max_len, 4 * kTgtWaveTiles * kKdTile)) &&
           (long long)g.rows * g.q_heads * kKdDim * 2 < (1LL << 31);
}

size_t kd_target_ws_floats(const Geometry &g, int n_layers) {
    return (size_t)n_layers * g.q_heads * ((size_t)g.rows + 16);
}

hipError_t launch_kd_target(const Geometry &g, int n_layers, const void *q_layers,
                            const void *k_cache, const int32_t *page_table,
                            const int32_t *seq_lens, const int32_t *q_pos, const float *lse_in,
                            float *abar, float *lse2, hipStream_t stream, hipEvent_t between) {
    if (!kd_target_supported(g, n_layers)) return hipErrorInvalidValue;
    KdArgs a;
    a.q_layers = static_cast<const uint16_t *>(q_layers);
    a.k_cache = static_cast<const uint16_t *>(k_cache);
    a.page_table = page_table;
    a.seq_lens = seq_lens;
    a.q_pos = q_pos;
    a.lse2 = lse2;
    a.abar = abar;
    a.n_layers = n_layers;
    a.batch = g.batch;
    a.n_q = g.n_q;
    a.rows = g.rows;
    a.max_len = g.max_len;
    a.page_shift = g.page_shift;
    a.max_pages = g.max_pages;
    a.causal = g.causal;
    a.q_heads = g.q_heads;
    a.kv_heads = g.kv_heads;
    a.group = g.group;
    a.row_tiles = div_up(g.n_q, kKdTile);
    a.key_tiles = div_up(g.max_len, kKdTile);
    a.rows_pad = g.rows + 16;
    a.scale_log2 = g.softmax_scale * kKdLog2e;
    a.inv_lh = 1.0f / ((float)n_layers * (float)g.q_heads);
    // the statistics pass: blocks of 4 waves of `per_wave` (32 rows, query head)
    // items per (KV head, layer)
    const long long items = (long long)div_up(g.n_q, 32) * g.group;
    const int per_wave = (items + 7) / 8 * g.batch * n_layers * g.kv_heads < kLseWide ? 1 : 2;
    a.row_tiles = (int)((items + kLseWaves * per_wave - 1) / (kLseWaves * per_wave));
    const dim3 lse_grid((unsigned)((long long)g.batch * a.row_tiles * n_layers * g.kv_heads));
    const bool paged = g.page_shift >= 0;
    if (lse_in) {  // the caller's log-sum-exps: no statistics pass
        const size_t total = (size_t)n_layers * g.rows * g.q_heads;
        const size_t blocks = (total + 255) / 256;
        kd_lse_import_kernel<<<dim3((unsigned)(blocks < 65536 ? blocks : 65536)), dim3(256), 0,
                               stream>>>(a, lse_in);
    } else {
#define KD_LSE_IT(G, IT)                                                                  \
    (paged ? kd_lse_kernel<G, IT, true><<<lse_grid, dim3(64 * kLseWaves), 0, stream>>>(a) \
           : kd_lse_kernel<G, IT, false><<<lse_grid, dim3(64 * kLseWaves), 0, stream>>>(a))
#define KD_LSE(G) (per_wave == 1 ? KD_LSE_IT(G, 1) : KD_LSE_IT(G, 2))
        switch (g.group) {
            case 1: KD_LSE(1); break;
            case 2: KD_LSE(2); break;
            case 4: KD_LSE(4); break;
            case 5: KD_LSE(5); break;
            case 8: KD_LSE(8); break;
            default: return hipErrorInvalidValue;
        }
#undef KD_LSE
#undef KD_LSE_IT
    }
    if (between && hipEventRecord(between, stream) != hipSuccess) return hipErrorUnknown;
    // the target pass: 16-row blocks x (4 waves x kTgtWaveTiles x 64)-key blocks
    a.row_tiles = div_up(g.n_q, 16);
    a.key_tiles = div_up(g.max_len, 4 * kTgtWaveTiles * kKdTile);
    const long long groups = ((long long)g.batch * a.row_tiles + 7) / 8;
    const dim3 tgt_grid((unsigned)(groups * a.key_tiles * 8));
#define KD_TGT(G)                                                                  \
    (paged ? kd_target_kernel<G, true><<<tgt_grid, dim3(256), 0, stream>>>(a)     \
           : kd_target_kernel<G, false><<<tgt_grid, dim3(256), 0, stream>>>(a))
    switch (g.group) {
        case 1: KD_TGT(1); break;
        case 2: KD_TGT(2); break;
        case 4: KD_TGT(4); break;
        case 5: KD_TGT(5); break;
        case 8: KD_TGT(8); break;
        default: return hipErrorInvalidValue;
    }
#undef KD_TGT
    return hipGetLastError();
}

hipError_t take_device_error_kd(uint32_t *bits) { return take_source_device_error(bits); }

}  // namespace clsa
