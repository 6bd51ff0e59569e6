// Eq. 2 for the new tokens of a step (Q_idx = H W_idx^Q, K_idx = H W_idx^K),
// together with the shared key and value of the same hidden states
// (K = H W^K, V = H W^V), fused with the cache write: the index query goes to
// its own buffer, the index key, key and value rows are written into the
// caches at each token's position.  One matrix product over the stacked
// weights [256 + 256 + 2 * kv_heads * 128, d_model] (each output feature's
// weight vector contiguous), bf16 inputs, fp32 accumulation, bf16 results
// rounded to nearest even.
//
// MFMA mapping (v_mfma_f32_16x16x32_bf16): A = 16 rows of h x 32 dims,
// B = 32 dims x 16 output features; lane l supplies row / feature (l & 15) for
// dims (l >> 4) * 8 .. +8 of each 32-dim step and receives C rows
// 4 * (l >> 4) + r (r = 0..3) of feature (l & 15).  A wave owns 16 rows x 64
// features (four feature tiles).
//   * few rows (decode): a workgroup of 8 waves splits d_model eight ways for
//     one tile of 16 or 32 rows x 16 features, each wave issuing all of its loads
//     before its first product (in two batches past d_model 3072), and the eight
//     partial tiles are added in LDS: the weights (13 MB at d_model 2560, the
//     bytes that bound this case) are then read by 160 workgroups at once.
//     Models wider than 3072 had gone to the tiled product, 20 workgroups that
//     walk d_model alone: 16 rows, d_model 4096 37 us, now 10; 8192 70, now 17;
//   * many rows (prefill): a tiled product, 128 rows x 128 features per
//     workgroup of 4 waves (64 x 64 each, 4 x 4 tiles of 16 x 16), d_model in
//     steps of 64 staged through LDS (double-buffered: the next step's global
//     loads are in flight during the current products); the 128-feature tile
//     lies in one destination (index query, index key, K or V), so the bf16
//     results go back through LDS and leave as whole 256-byte rows.
#include "clsa_internal.h"
#include "device_common.h"

namespace clsa {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kSplitWaves = 8;     // d_model split of the few-rows kernel
// Rows up to which the weights' bytes bound the product.  Against the tiled
// product (2560 features): 96 rows, d_model 2560 15.8 us against 28.4; 128 rows 22.2
// against 30.1, d_model 4096 33.9 against 42.6; 192 rows, 4096 44.7 against 41.5.
constexpr int kSplitMaxRows = 128;

struct ProjArgs {
    const uint16_t *h;         // [rows, d]
    const uint16_t *w;         // [n_feat, d]
    const int32_t *pos;        // [rows]
    const int32_t *page_table;
    uint16_t *q_idx;           // [rows, 256]
    uint16_t *k_idx;           // index-key cache
    uint16_t *k_cache, *v_cache;
    int rows, d, n_q, max_len, page_shift, max_pages, kvw;  // kvw = kv_heads * 128
    int rtiles, ftiles, band;  // tiled kernel: 128-row and 128-feature tiles, row tiles per band
};

__device__ __forceinline__ bf16x8 ld8(const uint16_t *p) {
    return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(p));
}

// Writes output feature f of row r (rows past the end are dropped; cache rows
// only for positions inside [0, max_len)).
template <bool PAGED>
__device__ __forceinline__ void store_feature(const ProjArgs &a, int r, int f, float v) {
    if (r >= a.rows) return;
    const uint16_t bits = (uint16_t)f32_to_bf16_bits(v);
    if (f < 256) {
        a.q_idx[(size_t)r * 256 + f] = bits;
        return;
    }
    const int p = a.pos[r];
    if (p < 0 || p >= a.max_len) return;
    const int b = r / a.n_q;
    size_t row;
    if (PAGED) {
        const int page = a.page_table[(size_t)b * a.max_pages + (p >> a.page_shift)];
        row = ((size_t)page << a.page_shift) + (p & ((1 << a.page_shift) - 1));
    } else {
        row = (size_t)b * a.max_len + p;
    }
    if (f < 512) a.k_idx[row * 256 + (f - 256)] = bits;
    else if (f < 512 + a.kvw) a.k_cache[row * a.kvw + (f - 512)] = bits;
    else a.v_cache[row * a.kvw + (f - 512 - a.kvw)] = bits;
}

// Few rows: one 16 RT-row x 16-feature tile per workgroup, d_model split over 8
// waves of NB * KS 32-dim steps each (d_model = 256 * NB * KS), KS at a time.
// RT = 2: a weight is read once for 32 rows (launch_splitk: when).
template <int KS, int NB, int RT, bool PAGED>
__global__ __launch_bounds__(512) void project_splitk_kernel(ProjArgs a) {
    __shared__ float part[kSplitWaves][16 * RT][16 + 1];
    const int ft = blockIdx.x, rt = blockIdx.y;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int col = lane & 15, grp = lane >> 4;
    const int k0 = wave * NB * KS * 32 + grp * 8;
    const uint16_t *hp[RT];
#pragma unroll
    for (int t = 0; t < RT; ++t)
        hp[t] = a.h + (size_t)min((rt * RT + t) * 16 + col, a.rows - 1) * a.d + k0;
    const uint16_t *wp = a.w + (size_t)(ft * 16 + col) * a.d + k0;
    f32x4 c[RT];
#pragma unroll
    for (int t = 0; t < RT; ++t) c[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        bf16x8 av[RT][KS], bv[KS];
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            bv[s] = ld8(wp + (nb * KS + s) * 32);
#pragma unroll
            for (int t = 0; t < RT; ++t) av[t][s] = ld8(hp[t] + (nb * KS + s) * 32);
        }
        __builtin_amdgcn_sched_barrier(0);  // every load in flight before the first product
#pragma unroll
        for (int s = 0; s < KS; ++s)
#pragma unroll
            for (int t = 0; t < RT; ++t)
                c[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[t][s], bv[s], c[t], 0, 0, 0);
    }
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) part[wave][16 * t + 4 * grp + r][col] = c[t][r];
    __syncthreads();
    if (threadIdx.x < 256 * RT) {  // 16 RT x 16 outputs
        const int rr = threadIdx.x >> 4, f = threadIdx.x & 15;
        float sum = 0.0f;
#pragma unroll
        for (int w = 0; w < kSplitWaves; ++w) sum += part[w][rr][f];
        store_feature<PAGED>(a, rt * 16 * RT + rr, ft * 16 + f, sum);
    }
}

// Many rows: the tiled product.
constexpr int kGemmM = 128, kGemmN = 128, kGemmK = 64;
// A staged row is 8 pieces of 16 bytes; piece p of row r lies at p ^ ((r >> 1) & 7):
// the 16 rows of an operand read and the two rows of a store then fall on all 64
// banks once (rows padded by 16 bytes: a third of the LDS cycles were conflicts of
// the stores).
constexpr int kGemmPitch = kGemmK;           // bf16 per staged row
constexpr int kGemmOutPitch = kGemmN + 8;    // bf16 per staged output row
constexpr size_t kGemmLds = sizeof(uint16_t) * 2 * 2 * kGemmM * kGemmPitch;

template <bool PAGED>
__global__ __launch_bounds__(256, 2) void project_gemm_kernel(ProjArgs a) {
    // two stages of A (rows of h) and B (features of w), 128 x 64 bf16 each
    // (dynamic LDS, kGemmLds bytes); the output tile (128 x 128 bf16) reuses it
    extern __shared__ __align__(16) uint16_t s_lds[];
    uint16_t(*s_ab)[2][kGemmM][kGemmPitch] =
        reinterpret_cast<uint16_t(*)[2][kGemmM][kGemmPitch]>(s_lds);
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int col = lane & 15, grp = lane >> 4;
    const int wm = wave >> 1, wn = wave & 1;  // the wave's 64 x 64 quadrant
    // Tile order: workgroups are dealt to the 8 XCDs in turn (L mod 8); XCD x
    // takes bands of `band` row tiles (8, fewer when there are few rows) and
    // walks, for each band, the feature tiles with the band's row tiles next to
    // each other, so that the workgroups in flight on an XCD share a few row
    // tiles and feature tiles per 64-wide step of d_model (their slices meet in
    // its L2).
    int rt, ft;
    {
        const int L = blockIdx.x, x = L & 7, q = L >> 3;
        const int per_band = a.band * a.ftiles;          // workgroups of one band
        const int band = 8 * (q / per_band) + x;         // bands dealt to the XCDs in turn
        const int qi = q % per_band;
        rt = a.band * band + qi % a.band;
        ft = qi / a.band;
    }
    if (rt >= a.rtiles) return;  // uniform: padding workgroups of the last bands
    const int f0 = ft * kGemmN, r0 = rt * kGemmM;
    // staging: thread t moves 16-byte pieces t + 256 i (i < 4) of each 128 x 64
    // tile: row (t >> 3) + 32 i, columns 8 (t & 7) .. + 8
    const int lrow = tid >> 3, lcol = (tid & 7) * 8;
    const int wcol = ((tid & 7) ^ ((lrow >> 1) & 7)) * 8, rswz = (col >> 1) & 7;
    const uint16_t *hp[4], *wp[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        hp[i] = a.h + (size_t)min(r0 + lrow + 32 * i, a.rows - 1) * a.d + lcol;  // tail rows: never stored
        wp[i] = a.w + (size_t)(f0 + lrow + 32 * i) * a.d + lcol;
    }
    // two register sets: the loads for step k + 2 are issued while step k is
    // computed, and step k + 1 (loaded a step earlier) goes to LDS after it;
    // every step issues its loads (the last two reload a valid step that is
    // never stored), so that the compiler's wait before each LDS store leaves
    // the newest 8 loads in flight
    u32x4 ra[2][4], rb[2][4];
    auto gload = [&](int set, int k0) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            ra[set][i] = *reinterpret_cast<const u32x4 *>(hp[i] + k0);
            rb[set][i] = *reinterpret_cast<const u32x4 *>(wp[i] + k0);
        }
    };
    auto lstore = [&](int set, int st) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            *reinterpret_cast<u32x4 *>(&s_ab[st][0][lrow + 32 * i][wcol]) = ra[set][i];
            *reinterpret_cast<u32x4 *>(&s_ab[st][1][lrow + 32 * i][wcol]) = rb[set][i];
        }
    };
    f32x4 c[4][4];
#pragma unroll
    for (int mt = 0; mt < 4; ++mt)
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) c[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int nk = a.d / kGemmK;  // even (d_model is a multiple of 512)
    gload(0, 0);
    gload(1, kGemmK);
    lstore(0, 0);
    __syncthreads();
    for (int kt = 0; kt < nk; kt += 2) {
      for (int h = 0; h < 2; ++h) {   // unrolled by two so that register sets are static
        const int k = kt + h;
        const int st = h;
        gload(h, min(k + 2, nk - 1) * kGemmK);  // unconditional (the last steps reload a valid step, never stored): a static load count
        // operand o of 32-wide half ks: A rows (o < 4) and B features of the wave's quadrant
        bf16x8 op[2][8];
        auto read_op = [&](int ks, int o) {
            const int r = (o < 4 ? wm * 64 + o * 16 : wn * 64 + (o - 4) * 16) + col;
            op[ks][o] = __builtin_bit_cast(
                bf16x8, *reinterpret_cast<const u32x4 *>(&s_ab[st][o >> 2][r][((ks * 4 + grp) ^ rswz) * 8]));
        };
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int o = 0; o < 8; ++o) read_op(0, o < 4 ? o + 4 : o - 4);
        // 16 parts of two products whose order is pinned: the first eight each read
        // an operand of the second half, the others each store a piece of the next
        // step (the last step stores an old piece that is not read).  8192 rows x 2560
        // features x 2560: 127.6 us with padded rows and the compiler's order, 124.0
        // swizzled, 117.4 in this order; 32-wide steps (three workgroups per CU) 139.6.
        // What bounds it now: 1280 tiles on 512 resident workgroups are 2.5 rounds, and
        // the step's own chain of barrier, operand reads and products at two waves per
        // SIMD.
#pragma unroll
        for (int p = 0; p < 16; ++p) {
            const int ks = p >> 3;
            if (ks == 0) read_op(1, p < 4 ? p + 4 : p - 4);
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int m = 2 * (p & 7) + e, mt = m >> 2, nt = m & 3;
                c[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(op[ks][mt], op[ks][4 + nt], c[mt][nt], 0, 0, 0);
            }
            if (ks == 1) {
                const int i = (p & 7) >> 1;
                if (p & 1) *reinterpret_cast<u32x4 *>(&s_ab[st ^ 1][1][lrow + 32 * i][wcol]) = rb[h ^ 1][i];
                else *reinterpret_cast<u32x4 *>(&s_ab[st ^ 1][0][lrow + 32 * i][wcol]) = ra[h ^ 1][i];
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        __syncthreads();
      }
    }
    // bf16 results into LDS: C tile (mt, nt) row 4 grp + r, column col
    uint16_t(*s_out)[kGemmOutPitch] = reinterpret_cast<uint16_t(*)[kGemmOutPitch]>(&s_ab[0][0][0][0]);
    static_assert(kGemmLds >= sizeof(uint16_t) * kGemmM * kGemmOutPitch, "output tile fits");
#pragma unroll
    for (int mt = 0; mt < 4; ++mt)
#pragma unroll
        for (int nt = 0; nt < 4; ++nt)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                s_out[wm * 64 + mt * 16 + 4 * grp + r][wn * 64 + nt * 16 + col] =
                    (uint16_t)f32_to_bf16_bits(c[mt][nt][r]);
    __syncthreads();
    // whole rows out: 16 pieces of 16 bytes per row, 8 rows per pass of 128 threads
    const int piece = tid & 15;
    int dst_kind, width, fo;  // 0: index query, 1: index key, 2: K, 3: V
    if (f0 < 256) { dst_kind = 0; width = 256; fo = f0; }
    else if (f0 < 512) { dst_kind = 1; width = 256; fo = f0 - 256; }
    else if (f0 < 512 + a.kvw) { dst_kind = 2; width = a.kvw; fo = f0 - 512; }
    else { dst_kind = 3; width = a.kvw; fo = f0 - 512 - a.kvw; }
    for (int rr = tid >> 4; rr < kGemmM; rr += 16) {
        const int r = r0 + rr;
        if (r >= a.rows) break;
        const u32x4 v = *reinterpret_cast<const u32x4 *>(&s_out[rr][piece * 8]);
        uint16_t *dst;
        if (dst_kind == 0) {
            dst = a.q_idx + (size_t)r * 256;
        } else {
            const int p = a.pos[r];
            if (p < 0 || p >= a.max_len) continue;
            const int b = r / a.n_q;
            size_t row;
            if (PAGED) {
                const int page = a.page_table[(size_t)b * a.max_pages + (p >> a.page_shift)];
                row = ((size_t)page << a.page_shift) + (p & ((1 << a.page_shift) - 1));
            } else {
                row = (size_t)b * a.max_len + p;
            }
            dst = (dst_kind == 1 ? a.k_idx : dst_kind == 2 ? a.k_cache : a.v_cache) + row * width;
        }
        *reinterpret_cast<u32x4 *>(dst + fo + piece * 8) = v;
    }
}

bool project_supported(int d_model) {
    return d_model >= 512 && d_model <= 8192 && d_model % 512 == 0;
}

template <int KS, int NB = 1>
static void launch_splitk(const ProjArgs &a, bool paged, int n_feat, hipStream_t stream) {
    // 32 rows a workgroup where 16 would not fit the chip in one round but 32 do
    // (32 rows x 2560 features, d_model 2560: 9.1 us against 11.3; 4096: 13.2 against
    // 16.5), and from 65 rows on; 32 rows x 1536 features fit with 16 (9.3 against 12.8
    // at 4096), 48 x 2560 fit with neither (11.3 against 13.9)
    const int tiles = n_feat / 16;
    const bool two = tiles * div_up(a.rows, 16) > 256 && (tiles * div_up(a.rows, 32) <= 256 || a.rows > 64);
    const dim3 grid(tiles, div_up(a.rows, two ? 32 : 16)), block(512);
    if (two && paged) project_splitk_kernel<KS, NB, 2, true><<<grid, block, 0, stream>>>(a);
    else if (two) project_splitk_kernel<KS, NB, 2, false><<<grid, block, 0, stream>>>(a);
    else if (paged) project_splitk_kernel<KS, NB, 1, true><<<grid, block, 0, stream>>>(a);
    else project_splitk_kernel<KS, NB, 1, false><<<grid, block, 0, stream>>>(a);
}

hipError_t launch_project(const Geometry &g, int d_model, const void *h, const void *w,
                          const int32_t *pos, const int32_t *page_table, void *q_idx,
                          void *k_idx, void *k_cache, void *v_cache, hipStream_t stream) {
    if (!project_supported(d_model)) return hipErrorInvalidValue;
    ProjArgs a;
    a.h = static_cast<const uint16_t *>(h);
    a.w = static_cast<const uint16_t *>(w);
    a.pos = pos;
    a.page_table = page_table;
    a.q_idx = static_cast<uint16_t *>(q_idx);
    a.k_idx = static_cast<uint16_t *>(k_idx);
    a.k_cache = static_cast<uint16_t *>(k_cache);
    a.v_cache = static_cast<uint16_t *>(v_cache);
    a.rows = g.rows;
    a.d = d_model;
    a.n_q = g.n_q;
    a.max_len = g.max_len;
    a.page_shift = g.page_shift;
    a.max_pages = g.max_pages;
    a.kvw = g.kv_heads * 128;
    if (g.rows == 0) return hipSuccess;
    const int n_feat = 512 + 2 * a.kvw;  // a multiple of 256 (kv_heads * 128 per K and V)
    const bool paged = g.page_shift >= 0;
    if (g.rows <= kSplitMaxRows) {
        switch (d_model / 512) {
            case 1: launch_splitk<2>(a, paged, n_feat, stream); break;
            case 2: launch_splitk<4>(a, paged, n_feat, stream); break;
            case 3: launch_splitk<6>(a, paged, n_feat, stream); break;
            case 4: launch_splitk<8>(a, paged, n_feat, stream); break;
            case 5: launch_splitk<10>(a, paged, n_feat, stream); break;
            case 6: launch_splitk<12>(a, paged, n_feat, stream); break;
            // past 3072 (96 operand registers) in two batches
            case 7: launch_splitk<7, 2>(a, paged, n_feat, stream); break;
            case 8: launch_splitk<8, 2>(a, paged, n_feat, stream); break;
            case 9: launch_splitk<9, 2>(a, paged, n_feat, stream); break;
            case 10: launch_splitk<10, 2>(a, paged, n_feat, stream); break;
            case 11: launch_splitk<11, 2>(a, paged, n_feat, stream); break;
            case 12: launch_splitk<12, 2>(a, paged, n_feat, stream); break;
            case 13: launch_splitk<13, 2>(a, paged, n_feat, stream); break;
            case 14: launch_splitk<14, 2>(a, paged, n_feat, stream); break;
            case 15: launch_splitk<15, 2>(a, paged, n_feat, stream); break;
            case 16: launch_splitk<16, 2>(a, paged, n_feat, stream); break;
            default: return hipErrorInvalidValue;
        }
        return hipGetLastError();
    }
    a.rtiles = div_up(g.rows, kGemmM);
    a.ftiles = n_feat / kGemmN;
    // bands of up to 8 row tiles, dealt to the 8 XCDs in turn (the last round
    // padded); fewer row tiles per band when that still leaves XCDs idle
    a.band = a.rtiles >= 64 ? 8 : div_up(a.rtiles, 8);
    const long bands = div_up(a.rtiles, a.band);
    const long blocks = div_up((int)bands, 8) * 8 * (long)a.band * a.ftiles;
    if (blocks > 0x7fffffffL) return hipErrorInvalidConfiguration;
    const dim3 grid((unsigned)blocks);
    const void *fn = paged ? reinterpret_cast<const void *>(&project_gemm_kernel<true>)
                           : reinterpret_cast<const void *>(&project_gemm_kernel<false>);
    hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kGemmLds);
    if (e != hipSuccess) return e;
    if (paged) project_gemm_kernel<true><<<grid, dim3(256), kGemmLds, stream>>>(a);
    else project_gemm_kernel<false><<<grid, dim3(256), kGemmLds, stream>>>(a);
    return hipGetLastError();
}

}  // namespace clsa
