// GQA attention of many query rows per sequence over tiles of keys, on the
// matrix cores: dense attention (Eq. 1, every valid key) and, for chunked
// prefill whose rows select a large part of their keys, the sparse attention
// of Eq. 4 as dense tiles with a selection mask.
//
// Work unit: one workgroup = 32 * RB query rows of one sequence x the G query
// heads of one KV head, one wave per (head, 32 rows).  The KV head's keys and
// values pass through LDS 64 at a time, double-buffered (the next tile's
// global loads are in flight during the current products, one barrier per
// tile), and each staged tile serves every wave, instead of being gathered
// again by every row as in the per-row kernel.
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
// Measured, one layer of 8192 causal rows, 20 query and 4 KV heads: 0.56 ms
// (3.4e11 FLOP, 610 TFLOP/s) against 2.7-2.8 ms with every row gathering its
// own keys (127 TFLOP/s, held by the L2).
// The running maximum moves lazily: only when a logit exceeds it by 2^kLazy
// (a wave-uniform branch), so that the steady state rescales nothing.
#include "clsa_internal.h"
#include "device_common.h"

namespace clsa {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int kTaDim = 128;
constexpr int kTaKeys = 64;              // keys per tile
constexpr int kTaKPitch = kTaDim + 8;    // bf16 per staged key row (272 bytes)
constexpr int kTaVPitch = kTaDim + 16;   // bf16 per staged value row (288 bytes)
constexpr float kTaLazy = 8.0f;          // log2 units the maximum may lag behind
constexpr float kTaLn2 = 0.6931471805599453f;

struct TileAttnArgs {
    const uint16_t *q, *k, *v;
    const int32_t *page_table, *seq_lens, *q_pos;
    const uint64_t *mask;  // [batch * mask_blocks, mask_pitch] lane masks, or null (dense)
    uint16_t *out;
    float *lse;            // may be null
    float *part_o, *part_ml;
    int batch, n_q, max_len, page_shift, max_pages, causal, kv_heads, q_heads;
    int row_blocks;        // blocks of 32 * RB rows per sequence
    int splits, span;      // key ranges per row, keys per range (a multiple of kTaKeys)
    int mask_blocks, mask_pitch;  // 32-row blocks per sequence, 64-bit masks per block
    float scale_log2;
};

// Maximum / sum over the two lanes of a query (l and l ^ 32).
__device__ __forceinline__ float pair_max(float x) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
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
__device__ __forceinline__ int wave_min_i(int x) {
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) x = min(x, __shfl_xor(x, d));
    return x;
}

// Position of key j of a 32-key block among the block's 32 mask words: word
// 2 r + hi belongs to the key that lanes of half hi hold in C register r, so
// that a 64-bit word is the lane mask of one register.
__host__ __device__ constexpr int mask_word(int j) {
    return 2 * (4 * (j >> 3) + (j & 3)) + ((j >> 2) & 1);
}

// The wave's queries one by one, one key at a time (2 dimensions per lane),
// every value exactly as selected: taken only when a tile product met an
// infinity or a NaN, which a weight of zero does not remove from a product, so
// that a key outside a row's set never reaches its result.
template <bool PAGED, bool MASK>
__device__ __forceinline__ void tile_attn_rows(const TileAttnArgs &a, int b, int t0, int g, int h,
                                            int split) {
    const int lane = threadIdx.x & 63;
    for (int i = 0; i < 32 && t0 + i < a.n_q; ++i) {
        const int row = b * a.n_q + t0 + i;
        const int n = valid_keys(a.seq_lens, a.q_pos, a.causal, b, row, a.max_len);
        const int j_end = min(n, (split + 1) * a.span);
        const uint32_t qw = *reinterpret_cast<const uint32_t *>(
            a.q + ((size_t)row * a.q_heads + h) * kTaDim + 2 * lane);
        float m = -INFINITY, l = 0.0f, ox = 0.0f, oy = 0.0f;
        for (int j = split * a.span; j < j_end; ++j) {
            if (MASK) {
                const uint32_t *w = reinterpret_cast<const uint32_t *>(
                    a.mask + ((size_t)b * a.mask_blocks + (t0 >> 5)) * a.mask_pitch);
                if (!((w[(j & ~31) + mask_word(j & 31)] >> i) & 1u)) continue;  // uniform
            }
            const size_t off = token_offset(a.page_table, a.page_shift, a.max_pages, a.max_len, b, j,
                                            a.kv_heads * kTaDim) + (size_t)g * kTaDim + 2 * lane;
            const uint32_t kw = *reinterpret_cast<const uint32_t *>(a.k + off);
            const uint32_t vw = *reinterpret_cast<const uint32_t *>(a.v + off);
            const float z = wave_sum(fmaf(bf16_lo(kw), bf16_lo(qw), bf16_hi(kw) * bf16_hi(qw))) *
                            a.scale_log2;
            const float nm = fmaxf(m, z), base = nm == -INFINITY ? 0.0f : nm;
            const float f = __builtin_amdgcn_exp2f(m - base), w = __builtin_amdgcn_exp2f(z - base);
            l = fmaf(l, f, w);
            ox = fmaf(w, bf16_lo(vw), ox * f);
            oy = fmaf(w, bf16_hi(vw), oy * f);
            m = nm;
        }
        const size_t rh = (size_t)row * a.q_heads + h;
        if (a.splits > 1 && n > 0) {
            const size_t slot = rh * a.splits + split;
            *reinterpret_cast<float2 *>(a.part_o + slot * kTaDim + 2 * lane) = make_float2(ox, oy);
            if (lane == 0) *reinterpret_cast<float2 *>(a.part_ml + slot * 2) = make_float2(m, l);
        } else if (split == 0) {
            const float inv = n == 0 ? 0.0f : 1.0f / l;
            const bf16x2 o = {(__bf16)(ox * inv), (__bf16)(oy * inv)};
            *reinterpret_cast<uint32_t *>(a.out + rh * kTaDim + 2 * lane) = __builtin_bit_cast(uint32_t, o);
            if (a.lse && lane == 0) a.lse[rh] = (m + log2f(l)) * kTaLn2;
        }
    }
}

template <int G, int RB, bool PAGED, bool MASK>
__global__ __launch_bounds__(64 * G * RB, 2) void tile_attn_kernel(TileAttnArgs a) {
    constexpr int NW = G * RB, NT = 64 * NW;
    constexpr int PIECES = kTaKeys * kTaDim / 8;          // 16-byte pieces of a tile
    constexpr int PER = (PIECES + NT - 1) / NT;           // per thread
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
    const int h = g * G + wave % G;
    const int t0 = rblk * 32 * RB + (wave / G) * 32;       // the wave's first row
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
    float m = -INFINITY, l = 0.0f;

    u32x4 kr[PER], vr[PER];
    auto fetch = [&](int j0) {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int pc = tid + i * NT;
            const int j = min(j0 + min(pc >> 4, kTaKeys - 1), len - 1);  // keys past len: masked
            size_t tok;
            if (PAGED) {
                const int page = a.page_table[(size_t)b * a.max_pages + (j >> a.page_shift)];
                tok = ((size_t)page << a.page_shift) + (j & ((1 << a.page_shift) - 1));
            } else {
                tok = (size_t)b * a.max_len + j;
            }
            const size_t off = (tok * a.kv_heads + g) * kTaDim + (pc & 15) * 8;
            kr[i] = *reinterpret_cast<const u32x4 *>(a.k + off);
            vr[i] = *reinterpret_cast<const u32x4 *>(a.v + off);
        }
    };
    auto stage = [&](int buf) {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int pc = tid + i * NT;
            if (PIECES % NT == 0 || pc < PIECES) {
                *reinterpret_cast<u32x4 *>(&s_k[buf][pc >> 4][(pc & 15) * 8]) = kr[i];
                *reinterpret_cast<u32x4 *>(&s_v[buf][pc >> 4][(pc & 15) * 8]) = vr[i];
            }
        }
    };
    if (tiles > 0) {
        fetch(j_begin);
        stage(0);
    }
    __syncthreads();
    // transposing V reads: lane i of a 16-lane group q reads row 4 hi + (i >> 2),
    // columns 16 (q & 1) + 4 (i & 3) .. + 4, and receives column i of the 4 x 16 block
    const int vrow = 4 * hi + ((lane & 15) >> 2);
    const int vcol = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
    const uint64_t *mrow = MASK ? a.mask + ((size_t)b * a.mask_blocks + min(t0 >> 5, a.mask_blocks - 1)) *
                                               a.mask_pitch
                                : nullptr;
    for (int u = 0; u < tiles; ++u) {
        const int j0 = j_begin + u * kTaKeys, buf = u & 1;
        if (u + 1 < tiles) fetch(j0 + kTaKeys);
        if (j0 < nmax) {  // uniform per wave
            f32x16 s[2];
#pragma unroll
            for (int kt = 0; kt < 2; ++kt) {
#pragma unroll
                for (int r = 0; r < 16; ++r) s[kt][r] = 0.0f;
#pragma unroll
                for (int ks = 0; ks < 8; ++ks) {
                    const bf16x8 ka = __builtin_bit_cast(
                        bf16x8, *reinterpret_cast<const u32x4 *>(&s_k[buf][32 * kt + col][16 * ks + 8 * hi]));
                    s[kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka, qb[ks], s[kt], 0, 0, 0);
                }
            }
            if (MASK) {
#pragma unroll
                for (int kt = 0; kt < 2; ++kt)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        s[kt][r] = __builtin_amdgcn_inverse_ballot_w64(mrow[(j0 >> 1) + 16 * kt + r])
                                       ? s[kt][r]
                                       : -INFINITY;
            } else if (j0 + kTaKeys > nmin) {
#pragma unroll
                for (int kt = 0; kt < 2; ++kt)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        s[kt][r] = j0 + 32 * kt + 8 * (r >> 2) + 4 * hi + (r & 3) < n ? s[kt][r]
                                                                                      : -INFINITY;
            }
            float mx = fmaxf(s[0][0], s[1][0]);
#pragma unroll
            for (int r = 1; r < 16; ++r) mx = fmaxf(mx, fmaxf(s[0][r], s[1][r]));
            mx = pair_max(mx * a.scale_log2);
            if (__builtin_amdgcn_ballot_w64(mx > m + kTaLazy)) {
                const float nm = fmaxf(m, mx);
                const float f = nm == -INFINITY ? 1.0f : __builtin_amdgcn_exp2f(m - nm);
                m = nm;
                l *= f;
#pragma unroll
                for (int d = 0; d < 4; ++d)
#pragma unroll
                    for (int r = 0; r < 16; ++r) o[d][r] *= f;
            }
            const float base = m == -INFINITY ? 0.0f : m;
            bf16x8 pb[4];
#pragma unroll
            for (int kt = 0; kt < 2; ++kt)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const float p = __builtin_amdgcn_exp2f(fmaf(s[kt][r], a.scale_log2, -base));
                    l += p;
                    pb[2 * kt + (r >> 3)][r & 7] = (__bf16)p;
                }
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
        }
        if (u + 1 < tiles) stage(buf ^ 1);
        __syncthreads();
    }
    if (t0 >= a.n_q) return;
    l = pair_sum(l);
    // a value that is not finite in any result of the wave: see tile_attn_rows
    float odd = 0.0f;
#pragma unroll
    for (int d = 0; d < 4; ++d)
#pragma unroll
        for (int r = 0; r < 16; ++r) odd = fmaf(o[d][r], 0.0f, odd);
    if (__builtin_amdgcn_ballot_w64(odd != 0.0f || l != l)) {
        tile_attn_rows<PAGED, MASK>(a, b, t0, g, h, split);
        return;
    }
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

// Rows per workgroup: 32 per head and wave, four waves or one per head.
static int tile_rows(int group) { return group == 1 ? 128 : group == 2 ? 64 : 32; }

bool tile_attn_dense(const Geometry &g) { return g.n_q >= kTileAttnMinRows; }

void tile_attn_plan(const Geometry &g, int max_splits, int &splits, int &span) {
    const long blocks = (long)g.batch * div_up(g.n_q, tile_rows(g.group)) * g.kv_heads;
    long want = (kTileAttnWorkgroups + blocks - 1) / blocks;
    if (want > max_splits) want = max_splits;
    const int tiles = div_up(g.max_len, kTaKeys);
    if (want > tiles / 4) want = tiles / 4;  // at least four tiles each
    if (want < 1) want = 1;
    span = div_up(tiles, (int)want) * kTaKeys;
    splits = div_up(g.max_len, span);
}

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
    a.mask = reinterpret_cast<const uint64_t *>(mask);
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
    a.row_blocks = div_up(g.n_q, tile_rows(g.group));
    a.splits = splits;
    a.span = span;
    a.mask_blocks = div_up(g.n_q, 32);
    a.mask_pitch = div_up(g.max_len, kTaKeys) * (kTaKeys / 2);
    a.scale_log2 = g.softmax_scale * 1.4426950408889634f;
    const size_t blocks = (size_t)g.batch * a.row_blocks * g.kv_heads * splits;
    if (blocks == 0) return hipSuccess;
    if (blocks > 0x7fffffffull) return hipErrorInvalidConfiguration;
    const dim3 grid((unsigned)blocks);
    const bool paged = g.page_shift >= 0;
#define TILE_ATTN(G, RB)                                                                        \
    if (mask && paged) tile_attn_kernel<G, RB, true, true><<<grid, dim3(64 * G * RB), 0, stream>>>(a); \
    else if (mask) tile_attn_kernel<G, RB, false, true><<<grid, dim3(64 * G * RB), 0, stream>>>(a);    \
    else if (paged) tile_attn_kernel<G, RB, true, false><<<grid, dim3(64 * G * RB), 0, stream>>>(a);   \
    else tile_attn_kernel<G, RB, false, false><<<grid, dim3(64 * G * RB), 0, stream>>>(a);             \
    break
    switch (g.group) {
        case 1: TILE_ATTN(1, 4);
        case 2: TILE_ATTN(2, 2);
        case 4: TILE_ATTN(4, 1);
        case 5: TILE_ATTN(5, 1);
        case 8: TILE_ATTN(8, 1);
        default: return hipErrorInvalidValue;
    }
#undef TILE_ATTN
    return hipGetLastError();
}

hipError_t take_device_error_tile_attn(uint32_t *bits) { return take_source_device_error(bits); }

}  // namespace clsa
