// GQA attention of many query rows per sequence over tiles of keys, on the
// matrix cores: dense attention (Eq. 1, every valid key) and, for chunked
// prefill whose rows select a large part of their keys, the sparse attention
// of Eq. 4 as dense tiles with a selection mask.
//
// Work unit: one workgroup of 8 waves, one wave per (32 query rows, query head)
// of one KV head, the heads of a row block next to each other.  The KV head's
// keys and values pass through LDS 64 at a time, double-buffered, one barrier
// per tile, and each staged tile serves all eight waves, instead of being
// gathered again by every row as in the per-row kernel.
//
// Per 64-key tile and wave (v_mfma_f32_32x32x16_bf16; lane l supplies A row /
// B column (l & 31) for contraction indices 8 * (l >> 5) .. + 8, and receives
// C rows 8 * (r >> 2) + 4 * (l >> 5) + (r & 3) of column (l & 31)):
//   * logits transposed, S^T = K Q^T: A = keys (16-byte LDS reads), B = the
//     wave's queries, held in registers for the whole kernel.  A lane then
//     holds 32 keys of ONE query, so the running maximum and sum are one value
//     per lane (the two lanes of a query meet in a permlane swap), and a
//     rescale needs no broadcast;
//   * O^T += V^T P^T: the weights are already in B-operand order (contraction
//     slot (hi, j) of a 16-key step stands for key 4 hi + (j & 3) + 8 (j >> 2)),
//     so they never leave their registers; A = V^T by ds_read_b64_tr_b16, the
//     transposing LDS read, from the row-major value tile.
// The weights enter the second product as bf16, so each tile has its own base: the
// largest logit of the row in that tile (not more than kTaLag below the row's
// largest so far), whose weight is then 1 exactly, and the accumulators move from
// base to base.  The row's first tile adds what rounding takes from its weights as a
// second product, since short rows have few keys and large weights.  Error of the
// outputs against 64 bits (their own rounding alone makes 0.00166), 8192 causal rows /
// 1000 rows of 6000 keys, 2048 selected: 0.00185 / 0.00199; with one base per row that
// lags by up to 2^8 0.0021 / 0.0023; every row gathering its own keys, whose list is
// cut into eight ranges with a base each, 0.00205 / 0.00213.  The sum of the weights
// keeps the row's largest logit as its base, so that it is not rounded at every tile.
// What bounds it: a wave alternates matrix products and the exponentials that
// depend on them, at two waves per SIMD (the accumulators, queries and two
// tiles' logits fill 256 registers).  The loop is therefore pipelined by one
// tile: the products of tile u + 1 stand beside the exponentials of tile u, and
// the weighted values of tile u beside the maximum of tile u + 1.
// Measured, one layer of 8192 causal rows, 20 query and 4 KV heads (3.4e11
// FLOP): every row gathering its own keys 2.7-2.8 ms (127 TFLOP/s); these tiles
// with the steps of a tile one after another, one wave per head, 0.56; pipelined
// with four waves per workgroup 0.46, with eight 0.41, and the key registers
// stored between the two halves (no spill) 0.394; a base per tile 0.410, and with
// the loop unrolled by two, so that a tile's logits are not copied, 0.391 ms:
// 870 TFLOP/s, 72% of what the library GEMM reaches on 8192^3 (1216).
#include "clsa_internal.h"
#include "device_common.h"

#include <math.h>

namespace clsa {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int kTaDim = 128;
constexpr int kTaKeys = 64;              // keys per tile
constexpr int kTaKPitch = kTaDim + 8;    // bf16 per staged key row (272 bytes)
constexpr int kTaVPitch = kTaDim + 16;   // bf16 per staged value row (288 bytes)
constexpr float kTaLag = 8.0f;           // log2 units a tile's base may lie below the row's maximum
constexpr float kTaLn2 = 0.6931471805599453f;

struct TileAttnArgs {
    const uint16_t *q, *k, *v;
    const int32_t *page_table, *seq_lens, *q_pos;
    const uint32_t *mask;  // [rows, mask_pitch] words of 32 keys, or null (dense)
    uint16_t *out;
    float *lse;            // may be null
    float *part_o, *part_ml;
    int batch, n_q, max_len, page_shift, max_pages, causal, kv_heads, q_heads;
    int group, row_blocks; // query heads per KV head, blocks of NW (32 rows, head) pairs per sequence
    int splits, span;      // key ranges per row, keys per range (a multiple of kTaKeys)
    int mask_pitch;        // words per row (two per tile)
    float scale_log2, q_sign;  // scale_log2 > 0: see launch_tile_attn
};

// IEEE maximum (gfx950 v_maximum3_f32; no operand canonicalisation).  A logit that is
// NaN makes its row NaN either way.
__device__ __forceinline__ float ta_max(float x, float y) {
    return __builtin_elementwise_maximum(x, y);
}

// Maximum / sum over the two lanes of a query (l and l ^ 32).
__device__ __forceinline__ float pair_max(float x) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return ta_max(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float pair_sum(float x) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

__device__ __forceinline__ int wave_max_i(int x) {
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) x = max(x, __shfl_xor(x, d));
    return x;
}
// Not an infinity and not a NaN.
__device__ __forceinline__ bool finite(float x) { return x - x == 0.0f; }

__device__ __forceinline__ int wave_min_i(int x) {
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) x = min(x, __shfl_xor(x, d));
    return x;
}

template <int NW, bool PAGED, bool MASK>
__global__ __launch_bounds__(64 * NW, 2) void tile_attn_kernel(TileAttnArgs a) {
    constexpr int NT = 64 * NW;
    constexpr int PER = kTaKeys * kTaDim / 8 / NT;  // 16-byte pieces of a tile per thread
    __shared__ __align__(16) uint16_t s_k[2][kTaKeys][kTaKPitch];
    __shared__ __align__(16) uint16_t s_v[2][kTaKeys][kTaVPitch];
    __shared__ int s_lim[NW];
    int x = blockIdx.x;
    const int g = x % a.kv_heads;
    x /= a.kv_heads;
    const int b = x % a.batch;
    x /= a.batch;
    const int rblk = a.row_blocks - 1 - x % a.row_blocks;  // causal: the longest rows first
    const int split = x / a.row_blocks;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int col = lane & 31, hi = lane >> 5;
    const int pair = rblk * NW + wave;                     // (32-row block, head of the group)
    const int h = g * a.group + pair % a.group;
    const int t0 = (pair / a.group) * 32;                  // the wave's first row
    const int t = t0 + col;                                // this lane's query
    const int len = clamp_len(a.seq_lens[b], a.max_len);
    const int row = b * a.n_q + min(t, a.n_q - 1);
    const int n = t < a.n_q ? valid_keys(a.seq_lens, a.q_pos, a.causal, b, row, a.max_len) : 0;
    const int nmax = __builtin_amdgcn_readfirstlane(wave_max_i(n));
    const int nmin = __builtin_amdgcn_readfirstlane(wave_min_i(n));
    if (lane == 0) s_lim[wave] = nmax;
    bf16x8 qb[8];
    {
        const uint16_t *p = a.q + ((size_t)row * a.q_heads + h) * kTaDim + hi * 8;
#pragma unroll
        for (int s = 0; s < 8; ++s)
            qb[s] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(p + 16 * s));
        if (a.q_sign != 1.0f)  // uniform
#pragma unroll
            for (int s = 0; s < 8; ++s)
#pragma unroll
                for (int e = 0; e < 8; ++e) qb[s][e] = (__bf16)((float)qb[s][e] * a.q_sign);
    }
    __syncthreads();
    int wg_max = s_lim[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) wg_max = max(wg_max, s_lim[w]);
    const int j_begin = split * a.span;
    const int j_end = min(wg_max, j_begin + a.span);
    const int tiles = j_end > j_begin ? div_up(j_end - j_begin, kTaKeys) : 0;

    f32x16 o[4];
#pragma unroll
    for (int d = 0; d < 4; ++d)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[d][r] = 0.0f;
    float m = -INFINITY, top = -INFINITY, l = 0.0f;  // base of o, maximum so far (base of l)

    // staging: thread -> 16-byte piece (tid & 15) of key rows (tid >> 4) + i * NT / 16;
    // keys past len are clamped (and masked)
    const int srow = tid >> 4, spc = (tid & 15) * 8;
    auto vector_at = [&](const uint16_t *base, int j) {  // key or value j (at most the last)
        j = min(j, len - 1);
        size_t tok;
        if (PAGED) {
            const int page = a.page_table[(size_t)b * a.max_pages + (j >> a.page_shift)];
            tok = ((size_t)page << a.page_shift) + (j & ((1 << a.page_shift) - 1));
        } else {
            tok = (size_t)b * a.max_len + j;
        }
        return base + (tok * a.kv_heads + g) * kTaDim;
    };
    auto fetch = [&](const uint16_t *base, int j0, u32x4 (&v)[PER]) {
#pragma unroll
        for (int i = 0; i < PER; ++i)
            v[i] = *reinterpret_cast<const u32x4 *>(vector_at(base, j0 + srow + i * (NT / 16)) + spc);
    };
    auto stage_k = [&](int buf, const u32x4 (&v)[PER]) {
#pragma unroll
        for (int i = 0; i < PER; ++i)
            *reinterpret_cast<u32x4 *>(&s_k[buf][srow + i * (NT / 16)][spc]) = v[i];
    };
    auto stage_v = [&](int buf, const u32x4 (&v)[PER]) {
#pragma unroll
        for (int i = 0; i < PER; ++i)
            *reinterpret_cast<u32x4 *>(&s_v[buf][srow + i * (NT / 16)][spc]) = v[i];
    };
    // transposing V reads: lane i of a 16-lane group q reads row 4 hi + (i >> 2),
    // columns 16 (q & 1) + 4 (i & 3) .. + 4, and receives column i of the 4 x 16 block
    const int vrow = 4 * hi + ((lane & 15) >> 2);
    const int vcol = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
    // the row's selection words of a tile
    const uint2 *mrow = reinterpret_cast<const uint2 *>(MASK ? a.mask + (size_t)row * a.mask_pitch
                                                             : nullptr);
    auto words = [&](int j0) {
        return mrow[min(j0 / kTaKeys, a.mask_pitch / 2 - 1)];
    };
    auto logits = [&](int buf, f32x16 (&s)[2]) {
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
            for (int r = 0; r < 16; ++r) s[kt][r] = 0.0f;
#pragma unroll
        for (int ks = 0; ks < 8; ++ks)
#pragma unroll
            for (int kt = 0; kt < 2; ++kt) {
                const bf16x8 ka = __builtin_bit_cast(
                    bf16x8, *reinterpret_cast<const u32x4 *>(&s_k[buf][32 * kt + col][16 * ks + 8 * hi]));
                s[kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka, qb[ks], s[kt], 0, 0, 0);
            }
    };
    auto drop = [&](int j0, uint2 w, f32x16 (&s)[2]) {  // keys outside a row's set
        if (MASK && __builtin_amdgcn_ballot_w64((w.x & w.y) != ~0u)) {
            w.x >>= 4 * hi;
            w.y >>= 4 * hi;
#pragma unroll
            for (int kt = 0; kt < 2; ++kt)
#pragma unroll
                for (int r = 0; r < 16; ++r) {  // v_bfe_i32 (0 or -1) and v_bfi_b32
                    const uint32_t on = (uint32_t)__builtin_amdgcn_sbfe((int)(kt ? w.y : w.x),
                                                                        8 * (r >> 2) + (r & 3), 1);
                    s[kt][r] = __uint_as_float((__float_as_uint(s[kt][r]) & on) | (0xff800000u & ~on));
                }
        } else if (!MASK && j0 + kTaKeys > nmin) {
#pragma unroll
            for (int kt = 0; kt < 2; ++kt)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    s[kt][r] = j0 + 32 * kt + 8 * (r >> 2) + 4 * hi + (r & 3) < n ? s[kt][r]
                                                                                  : -INFINITY;
        }
    };
    auto largest = [&](const f32x16 (&s)[2]) {
        float mx = ta_max(s[0][0], s[1][0]);
#pragma unroll
        for (int r = 1; r < 16; ++r) mx = ta_max(ta_max(mx, s[0][r]), s[1][r]);
        return pair_max(mx * a.scale_log2);
    };
    auto rebase = [&](float mx, float lag) {  // mx: the next tile's largest logit
        const float old = top;
        top = ta_max(top, mx);
        const float nm = ta_max(mx, top - lag);
        const float f = nm == -INFINITY ? 1.0f : __builtin_amdgcn_exp2f(m - nm);
        l *= top == -INFINITY ? 1.0f : __builtin_amdgcn_exp2f(old - top);
        m = nm;
#pragma unroll
        for (int d = 0; d < 4; ++d)
#pragma unroll
            for (int r = 0; r < 16; ++r) o[d][r] *= f;
    };
    auto weights = [&](const f32x16 (&s)[2], bf16x8 (&pb)[4]) {
        const float base = m == -INFINITY ? 0.0f : m;
        float sum[2] = {0.0f, 0.0f};
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const float p = __builtin_amdgcn_exp2f(fmaf(s[kt][r], a.scale_log2, -base));
                sum[kt] += p;
                pb[2 * kt + (r >> 3)][r & 7] = (__bf16)p;
            }
        l = fmaf(sum[0] + sum[1], m == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(m - top), l);
    };
    auto residues = [&](const f32x16 (&s)[2], bf16x8 (&pb)[4]) {  // what weights() rounds off
        const float base = m == -INFINITY ? 0.0f : m;
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const float p = __builtin_amdgcn_exp2f(fmaf(s[kt][r], a.scale_log2, -base));
                pb[2 * kt + (r >> 3)][r & 7] = (__bf16)(p - (float)(__bf16)p);
            }
    };
    auto weighted = [&](int buf, const bf16x8 (&pb)[4]) {
#pragma unroll
        for (int kb = 0; kb < 4; ++kb)
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                typedef __attribute__((address_space(3))) s16x4 lds4;
                const s16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                    (lds4 *)&s_v[buf][16 * kb + vrow][32 * d + vcol]);
                const s16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                    (lds4 *)&s_v[buf][16 * kb + 8 + vrow][32 * d + vcol]);
                const bf16x8 va = __builtin_bit_cast(
                    bf16x8, __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7));
                o[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va, pb[kb], o[d], 0, 0, 0);
            }
    };
    u32x4 kr[PER], vr[PER];
    if (tiles > 0) {  // uniform over the workgroup
        fetch(a.k, j_begin, kr);
        fetch(a.v, j_begin, vr);
        stage_k(0, kr);
        stage_v(0, vr);
        fetch(a.k, j_begin + kTaKeys, kr);
        stage_k(1, kr);
        __syncthreads();
        f32x16 s[2];
        logits(0, s);
        drop(j_begin, MASK ? words(j_begin) : make_uint2(0u, 0u), s);
        rebase(largest(s), kTaLag);
        {  // the first tile's weights keep 16 bits
            bf16x8 pb[4];
            residues(s, pb);
            weighted(0, pb);
        }
        // A buffer is stored into only after a barrier that follows its last read: in
        // the loop the one that ends the step before, for the first step this one.
        __syncthreads();
        f32x16 sn[2];
        auto step = [&](int u, const f32x16 (&s)[2], f32x16 (&sn)[2]) {
            const int j0 = j_begin + u * kTaKeys, buf = u & 1;
            fetch(a.k, j0 + 2 * kTaKeys, kr);
            fetch(a.v, j0 + kTaKeys, vr);
            const uint2 w = MASK ? words(j0 + kTaKeys) : make_uint2(0u, 0u);
            bf16x8 pb[4];
            __builtin_amdgcn_sched_barrier(0);
            logits(buf ^ 1, sn);
            weights(s, pb);
            __builtin_amdgcn_sched_barrier(0);
            stage_k(buf, kr);
            drop(j0 + kTaKeys, w, sn);
            weighted(buf, pb);
            const float mx = largest(sn);
            __builtin_amdgcn_sched_barrier(0);
            stage_v(buf ^ 1, vr);
            rebase(mx, kTaLag);
            __syncthreads();
        };
        auto last = [&](const f32x16 (&s)[2]) {
            bf16x8 pb[4];
            weights(s, pb);
            weighted((tiles - 1) & 1, pb);
        };
        int u = 0;
        for (; u + 2 < tiles; u += 2) {
            step(u, s, sn);
            step(u + 1, sn, s);
        }
        if (u + 1 < tiles) {
            step(u, s, sn);
            last(sn);
        } else {
            last(s);
        }
    }
    __syncthreads();  // every wave is done with the tiles: see below
    if (t0 >= a.n_q) return;
    // A value that is not finite reaches the products of rows without its key (a
    // weight of zero does not remove it), and one near the largest float can overflow
    // the tiles' lagging base.  A wave with such a result of finite logits makes it
    // again, each value reaching the rows of its key alone: keys straight from memory,
    // values 32 at a time through the wave's own eighth of the tiles, those that are
    // not finite staged as zeros and added by hand, the base always the row's
    // maximum.  8192 causal rows with one infinity 1.9 ms, 64 rows x 131072 keys 1.0
    // (0.4 and 0.19 without); one key at a time it was hundreds of times the usual.
    float odd = 0.0f;
#pragma unroll
    for (int d = 0; d < 4; ++d)
#pragma unroll
        for (int r = 0; r < 16; ++r) odd = fmaf(o[d][r], 0.0f, odd);
    const float l_both = pair_sum(l);
    const bool again = odd != 0.0f && finite(l_both) && (n > j_begin || n == 0) && t < a.n_q;
    if (__builtin_amdgcn_ballot_w64(again)) {
        static_assert(NW == 8, "eight slots of 32 rows in the tiles");
        typedef __attribute__((address_space(3))) u32x4 lds16;
        typedef __attribute__((address_space(3))) s16x4 lds4;
        uint16_t *own = wave < 4 ? &s_k[wave >> 1][32 * (wave & 1)][0]
                                 : &s_v[(wave - 4) >> 1][32 * (wave & 1)][0];
        const int pitch = wave < 4 ? kTaKPitch : kTaVPitch;
#pragma unroll
        for (int d = 0; d < 4; ++d)
#pragma unroll
            for (int r = 0; r < 16; ++r) o[d][r] = 0.0f;
        m = top = -INFINITY;
        l = 0.0f;
        for (int j0 = j_begin; j0 < min(nmax, j_begin + a.span); j0 += kTaKeys) {
            f32x16 s[2];
#pragma unroll
            for (int kt = 0; kt < 2; ++kt) {
                const uint16_t *kp = vector_at(a.k, j0 + 32 * kt + col) + 8 * hi;
#pragma unroll
                for (int r = 0; r < 16; ++r) s[kt][r] = 0.0f;
#pragma unroll
                for (int ks = 0; ks < 8; ++ks)
                    s[kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                        __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(kp + 16 * ks)), qb[ks],
                        s[kt], 0, 0, 0);
            }
            const uint2 w = MASK ? words(j0) : make_uint2(0u, 0u);
            drop(j0, w, s);
            rebase(largest(s), 0.0f);
            bf16x8 pb[4], pr[4];
            weights(s, pb);
            residues(s, pr);
#pragma unroll
            for (int kt = 0; kt < 2; ++kt) {
                uint32_t bad = 0u;  // keys of the half tile with a value that is not finite
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const int r = 4 * i + (lane >> 4);
                    u32x4 x = *reinterpret_cast<const u32x4 *>(vector_at(a.v, j0 + 32 * kt + r) + (lane & 15) * 8);
                    bool some = false;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const bool lo = finite(bf16_lo(x[e])), up = finite(bf16_hi(x[e]));
                        some |= !lo || !up;
                        x[e] &= (lo ? 0x0000ffffu : 0u) | (up ? 0xffff0000u : 0u);
                    }
                    *(lds16 *)(own + r * pitch + (lane & 15) * 8) = x;
                    const uint64_t rows = __builtin_amdgcn_ballot_w64(some);
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        bad |= ((uint32_t)(rows >> (16 * q)) & 0xffffu ? 1u : 0u) << (4 * i + q);
                }
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                    for (int d = 0; d < 4; ++d) {
                        const uint16_t *v = own + (16 * kb + vrow) * pitch + 32 * d + vcol;
                        const s16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4 *)v);
                        const s16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4 *)(v + 8 * pitch));
                        const bf16x8 va = __builtin_bit_cast(
                            bf16x8, __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7));
                        o[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va, pb[2 * kt + kb], o[d], 0, 0, 0);
                        o[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va, pr[2 * kt + kb], o[d], 0, 0, 0);
                    }
                __builtin_amdgcn_wave_barrier();
                for (; bad; bad &= bad - 1u) {  // uniform
                    const int i = __builtin_ctz(bad), j = j0 + 32 * kt + i;
                    const bool in = j < n && (!MASK || (((kt ? w.y : w.x) >> i) & 1u));
                    float z = s[kt][0];  // the key's logit: register 4 (i >> 3) + (i & 3) of lanes hi = (i >> 2) & 1
#pragma unroll
                    for (int r = 1; r < 16; ++r) z = r == 4 * (i >> 3) + (i & 3) ? s[kt][r] : z;
                    const uint32_t p = __float_as_uint(__builtin_amdgcn_exp2f(fmaf(z, a.scale_log2, -m)));
                    const auto both = __builtin_amdgcn_permlane32_swap(p, p, false, false);
                    const float wt = __uint_as_float(both[0]), wu = __uint_as_float(both[1]);
                    const uint16_t *vp = vector_at(a.v, j) + 4 * hi;
#pragma unroll
                    for (int d = 0; d < 4; ++d)
#pragma unroll
                        for (int r = 0; r < 16; r += 4) {
                            const u32x2 x = *reinterpret_cast<const u32x2 *>(vp + 32 * d + 2 * r);
#pragma unroll
                            for (int c = 0; c < 4; ++c) {
                                const float v = c & 1 ? bf16_hi(x[c >> 1]) : bf16_lo(x[c >> 1]);
                                if (in && !finite(v)) o[d][r + c] = fmaf((i >> 2) & 1 ? wu : wt, v, o[d][r + c]);
                            }
                        }
                }
            }
        }
    }
    l = pair_sum(l);
    const float to_top = m == -INFINITY ? 1.0f : __builtin_amdgcn_exp2f(m - top);
#pragma unroll
    for (int d = 0; d < 4; ++d)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[d][r] *= to_top;
    m = top;
    if (t >= a.n_q) return;
    const size_t rh = (size_t)row * a.q_heads + h;
    if (a.splits > 1 && n > 0) {
        const size_t slot = rh * a.splits + split;
        float *dst = a.part_o + slot * kTaDim + 4 * hi;
#pragma unroll
        for (int d = 0; d < 4; ++d)
#pragma unroll
            for (int r = 0; r < 16; r += 4)
                *reinterpret_cast<float4 *>(dst + 32 * d + 2 * r) =
                    make_float4(o[d][r], o[d][r + 1], o[d][r + 2], o[d][r + 3]);
        if (hi == 0) *reinterpret_cast<float2 *>(a.part_ml + slot * 2) = make_float2(m, l);
        return;
    }
    if (split > 0) return;  // an empty row: written once
    const float inv = n == 0 ? 0.0f : 1.0f / l;
    uint16_t *dst = a.out + rh * kTaDim + 4 * hi;
#pragma unroll
    for (int d = 0; d < 4; ++d)
#pragma unroll
        for (int r = 0; r < 16; r += 4) {
            const bf16x2 lo = {(__bf16)(o[d][r] * inv), (__bf16)(o[d][r + 1] * inv)};
            const bf16x2 up = {(__bf16)(o[d][r + 2] * inv), (__bf16)(o[d][r + 3] * inv)};
            *reinterpret_cast<u32x2 *>(dst + 32 * d + 2 * r) =
                u32x2{__builtin_bit_cast(uint32_t, lo), __builtin_bit_cast(uint32_t, up)};
        }
    if (a.lse && hi == 0) a.lse[rh] = (m + log2f(l)) * kTaLn2;
}

struct MaskArgs {
    const int32_t *idx, *n_sel, *seq_lens;  // [rows, top_k], [rows], [batch]
    uint32_t *mask;                         // [rows, pitch]
    int n_q, max_len, top_k, pitch;
};

// The selection mask of tile_attn_kernel from the (ascending) index lists: one
// bit per key, a workgroup per row.  Each thread takes a run of consecutive
// entries and ORs its finished words into LDS, so that dense lists cost few LDS
// operations; a row longer than kMaskKeys takes several passes.
constexpr int kMaskKeys = 65536, kMaskThreads = 256;
__global__ __launch_bounds__(kMaskThreads) void attn_mask_kernel(MaskArgs a) {
    __shared__ uint32_t w[kMaskKeys / 32];
    const size_t row = blockIdx.x;
    const int b = (int)row / a.n_q, tid = threadIdx.x;
    const int len = clamp_len(a.seq_lens[b], a.max_len);
    const int end = div_up(len, kTaKeys) * (kTaKeys / 32);  // words read later
    const int n = min(max(a.n_sel[row], 0), a.top_k);
    const int32_t *sel = a.idx + row * a.top_k;
    const int per = div_up(n, kMaskThreads);
    for (int w0 = 0; w0 < end; w0 += kMaskKeys / 32) {
        const int words = min(kMaskKeys / 32, end - w0);
        __syncthreads();
        for (int i = tid; i < words; i += kMaskThreads) w[i] = 0u;
        __syncthreads();
        uint32_t bits = 0u;
        int at = -1;
        for (int e = tid * per; e < min(n, (tid + 1) * per); ++e) {
            const int j = sel[e], wj = (j >> 5) - w0;
            if (wj != at) {
                if (bits && at >= 0 && at < words) atomicOr(&w[at], bits);
                bits = 0u;
                at = wj;
            }
            bits |= 1u << (j & 31);
        }
        if (bits && at >= 0 && at < words) atomicOr(&w[at], bits);
        __syncthreads();
        for (int i = tid; i < words; i += kMaskThreads) a.mask[row * a.pitch + w0 + i] = w[i];
    }
}

// Workgroups per sequence and KV head: NW waves, one per (32 rows, query head).
constexpr int kTaWaves = 8;
static int tile_blocks(const Geometry &g) { return div_up(div_up(g.n_q, 32) * g.group, kTaWaves); }

void tile_attn_plan(const Geometry &g, int max_splits, int &splits, int &span) {
    const long blocks = (long)g.batch * tile_blocks(g) * g.kv_heads;
    long want = (kTileAttnWorkgroups + blocks - 1) / blocks;
    if (want > max_splits) want = max_splits;
    const int tiles = div_up(g.max_len, kTaKeys);
    if (want > tiles / 2) want = tiles / 2;  // at least two tiles each
    if (want < 1) want = 1;
    span = div_up(tiles, (int)want) * kTaKeys;
    splits = div_up(g.max_len, span);
}

// Keys a row has on average, where every sequence is full (causal: the last n_q rows).
static double mean_keys(const Geometry &g) {
    const int half = g.max_len / 2, mean = g.max_len - g.n_q / 2;
    return !g.causal ? g.max_len : mean > half ? mean : half;
}

// Both sides priced in us with what 3850 shapes measured (16 to 1100 rows, 130 to
// 40000 keys, groups of 1 to 8, contiguous and paged).  Tiles: 3.2 more to start and
// end than gathers, 1.9 a tile and round of the chip, 0.6 a MB of range partials;
// gathers: 17 + 0.75 G ps per (row, KV head, key), 2.5 for the merge and 0.4 a MB of
// partials.  Many query heads over few keys make the tiles' partials large: 4 x 32
// rows x 600 keys, 64 / 8 heads 19.4 us gathered and 33.8 in tiles (by the limits
// alone they were taken), 500 rows x 600 causal keys, 20 / 4 heads 24 and 31, 32 / 8
// 37 and 32 (the price is still wrong here), 3 x 500 x 600 64 / 8 151 and 42.
bool tile_attn_dense(const Geometry &g, int gather_splits) {
    if (g.n_q < kTileAttnMinRows || (double)g.rows * g.kv_heads * g.max_len < kTileAttnMinKeys)
        return false;
    int splits, span;
    tile_attn_plan(g, kMaxSplits, splits, span);
    const double wgs = (double)g.batch * tile_blocks(g) * g.kv_heads * splits;
    const double keys = mean_keys(g), rounds = ceil(wgs / kTileAttnWorkgroups);
    const double split_mb = (double)g.rows * g.q_heads * (kTaDim + 2) * sizeof(float) * 1e-6;
    const double tiles_us = 3.2 + rounds * (span < keys ? span : keys) / kTaKeys * 1.9 +
                            (splits > 1 ? 0.6 * split_mb * splits : 0.0);
    const double gather_us = (double)g.rows * g.kv_heads * keys * (17.0 + 0.75 * g.group) * 1e-6 +
                             (gather_splits > 1 ? 2.5 + 0.4 * split_mb * gather_splits : 0.0);
    return tiles_us < gather_us;
}

static int mask_words(const Geometry &g) { return div_up(g.max_len, kTaKeys) * (kTaKeys / 32); }

hipError_t launch_tile_attn(const Geometry &g, const void *q, const void *k_cache,
                            const void *v_cache, const int32_t *page_table,
                            const int32_t *seq_lens, const int32_t *q_pos, const uint32_t *mask,
                            int splits, int span, void *out, float *lse, float *part_o,
                            float *part_ml, hipStream_t stream) {
    TileAttnArgs a;
    a.q = static_cast<const uint16_t *>(q);
    a.k = static_cast<const uint16_t *>(k_cache);
    a.v = static_cast<const uint16_t *>(v_cache);
    a.page_table = page_table;
    a.seq_lens = seq_lens;
    a.q_pos = q_pos;
    a.mask = mask;
    a.out = static_cast<uint16_t *>(out);
    a.lse = lse;
    a.part_o = part_o;
    a.part_ml = part_ml;
    a.batch = g.batch;
    a.n_q = g.n_q;
    a.max_len = g.max_len;
    a.page_shift = g.page_shift;
    a.max_pages = g.max_pages;
    a.causal = g.causal;
    a.kv_heads = g.kv_heads;
    a.q_heads = g.q_heads;
    a.group = g.group;
    a.row_blocks = tile_blocks(g);
    a.splits = splits;
    a.span = span;
    a.mask_pitch = mask_words(g);
    // The kernel drops keys (-inf) and takes maxima before it scales, so its scale is
    // positive: the sign of the caller's goes into the queries (exact), and a scale of
    // zero makes them zero.
    const float scale = g.softmax_scale;
    a.q_sign = scale > 0.0f ? 1.0f : scale < 0.0f ? -1.0f : 0.0f;
    a.scale_log2 = scale == 0.0f ? 1.0f : fabsf(scale) * 1.4426950408889634f;
    const size_t blocks = (size_t)g.batch * a.row_blocks * g.kv_heads * splits;
    if (blocks == 0) return hipSuccess;
    if (blocks > 0x7fffffffull) return hipErrorInvalidConfiguration;
    const dim3 grid((unsigned)blocks);
    const bool paged = g.page_shift >= 0;
    const dim3 block(64 * kTaWaves);
    if (mask && paged) tile_attn_kernel<kTaWaves, true, true><<<grid, block, 0, stream>>>(a);
    else if (mask) tile_attn_kernel<kTaWaves, false, true><<<grid, block, 0, stream>>>(a);
    else if (paged) tile_attn_kernel<kTaWaves, true, false><<<grid, block, 0, stream>>>(a);
    else tile_attn_kernel<kTaWaves, false, false><<<grid, block, 0, stream>>>(a);
    return hipGetLastError();
}

// Masked tiles cost every key of a row, gathers only the selected ones, so the
// line lies where a row selects about a tenth of its keys (groups of 4; the
// gather serves a whole group, the tiles pay per query head).  Both sides are
// priced with what they measured: a workgroup's tile step (8 waves x 64 keys, one
// workgroup per CU) 3.1 us; a gather 22 + 1.4 G ps per (row, KV head, selected
// token).  Per layer of 4096 rows x 16384 keys, k = 2048, 32 / 8 heads: gathers
// 1.85 ms, tiles 1.1; 4096 x 32768: 1.95 against 2.4.  Where the gathers need no
// merge (one split), the mask's launch counts too: a step of 2 x 137 rows that select
// everything, paged, 29.0 us in tiles and 25.9 gathered (priced 10.2 and 11.6), 2 x 122
// rows, groups of 8 27.2 and 25.5 (6.8 and 8.3); with four splits 4 x 125 rows 27.5
// and 48.2 (6.7 and 7.2).  (Still a little in the tiles' favour for groups of 1: 4 x
// 153 rows of which 243 keys a row 28.4 and 27.2.)
bool tile_attn_masked(const Geometry &g, int gather_splits) {
    if (g.n_q < kTileAttnMinRows || mask_words(g) > g.max_len) return false;  // the scores hold the mask
    const double wgs = (double)g.batch * tile_blocks(g) * g.kv_heads;
    const double keys = wgs > 256 ? mean_keys(g) : g.max_len;
    const double rounds = wgs > 256 ? wgs / 256 + 0.3 : 1.0;  // the last round is partly empty
    const double tiles_us = rounds * (keys / kTaKeys) * 3.1;
    const double sel = g.top_k < keys ? g.top_k : keys;
    const double gather_us = (double)g.rows * g.kv_heads * sel * (22.0 + 1.4 * g.group) * 1e-6;
    return 1.1 * tiles_us + (gather_splits > 1 ? 0.0 : 2.5) < gather_us;
}

hipError_t launch_attn_mask(const Geometry &g, const int32_t *idx, const int32_t *n_sel,
                            const int32_t *seq_lens, uint32_t *mask, hipStream_t stream) {
    MaskArgs a;
    a.idx = idx;
    a.n_sel = n_sel;
    a.seq_lens = seq_lens;
    a.mask = mask;
    a.n_q = g.n_q;
    a.max_len = g.max_len;
    a.top_k = g.top_k;
    a.pitch = mask_words(g);
    attn_mask_kernel<<<dim3((unsigned)g.rows), dim3(kMaskThreads), 0, stream>>>(a);
    return hipGetLastError();
}

hipError_t launch_masked_attn(const Geometry &g, const void *q, const void *k_cache,
                              const void *v_cache, const int32_t *page_table,
                              const int32_t *seq_lens, const int32_t *q_pos, const uint32_t *mask,
                              void *out, float *lse, hipStream_t stream) {
    return launch_tile_attn(g, q, k_cache, v_cache, page_table, seq_lens, q_pos, mask, 1,
                            div_up(g.max_len, kTaKeys) * kTaKeys, out, lse, nullptr, nullptr, stream);
}

hipError_t take_device_error_tile_attn(uint32_t *bits) { return take_source_device_error(bits); }

}  // namespace clsa
