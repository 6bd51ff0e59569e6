// A kernel source of this library as ordinary C++: every lane of a workgroup is a
// fibre, the lanes of a wave meet at each wave-wide operation, and the waves of a
// workgroup meet at its barriers only.  The waves run one after another, each as
// far as the next barrier, in an order that the test chooses, so that a missing
// barrier gives a wrong result every time.  For tests: sizes of a few tiles.
#pragma once
#include <hip/hip_runtime_api.h>
#include <math.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <ucontext.h>

#include <functional>
#include <vector>

#define __global__
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __shared__ static
#define __align__(n) __attribute__((aligned(n)))
#define HIP_SYMBOL(x) (&(x))

struct dim3 {
    unsigned x, y, z;
    dim3(unsigned x_ = 1, unsigned y_ = 1, unsigned z_ = 1) : x(x_), y(y_), z(z_) {}
};
struct uint2 { uint32_t x, y; };
struct uint4 { uint32_t x, y, z, w; };
struct float2 { float x, y; };
struct alignas(16) float4 { float x, y, z, w; };
inline uint2 make_uint2(uint32_t x, uint32_t y) { return {x, y}; }
inline uint4 make_uint4(uint32_t x, uint32_t y, uint32_t z, uint32_t w) { return {x, y, z, w}; }
inline float2 make_float2(float x, float y) { return {x, y}; }
inline float4 make_float4(float x, float y, float z, float w) { return {x, y, z, w}; }
template <class T> inline T min(T a, T b) { return b < a ? b : a; }
template <class T> inline T max(T a, T b) { return a < b ? b : a; }
inline uint32_t __float_as_uint(float x) { return __builtin_bit_cast(uint32_t, x); }
inline float __uint_as_float(uint32_t x) { return __builtin_bit_cast(float, x); }
inline int __float_as_int(float x) { return __builtin_bit_cast(int, x); }
inline float __int_as_float(int x) { return __builtin_bit_cast(float, x); }
inline uint32_t atomicOr(uint32_t *p, uint32_t v) { const uint32_t o = *p; *p |= v; return o; }
template <class... A> inline hipError_t hipMemcpyFromSymbol(A...) { return hipSuccess; }
template <class... A> inline hipError_t hipMemcpyToSymbol(A...) { return hipSuccess; }

namespace emu {

struct Fibre {
    ucontext_t ctx;
    std::vector<char> stack;
    enum { kRun, kWave, kBarrier, kDone } state = kRun;
    void *arg = nullptr;                // of the wave operation it waits in
    void (*op)(void *const *) = nullptr;
};
inline std::vector<Fibre> fibres;
inline ucontext_t home;
inline int current = 0;
inline dim3 thread_idx, block_idx, grid_dim;
inline std::function<void()> body;
inline int wave_order = 0;              // 0: first wave first, 1: last wave first
inline long wave_ops = 0;               // wave-wide operations since it was last cleared

inline void yield_as(decltype(Fibre::state) s) {
    Fibre &f = fibres[current];
    f.state = s;
    swapcontext(&f.ctx, &home);
}
// The lanes of the wave meet; op sees every lane's argument (NULL: a lane that has returned).
template <class A> inline void wave_op(A &arg, void (*op)(void *const *)) {
    Fibre &f = fibres[current];
    f.arg = &arg;
    f.op = op;
    yield_as(Fibre::kWave);
}
inline void entry() {
    body();
    yield_as(Fibre::kDone);
}
inline void run_wave(int w, int threads) {
    const int lo = w * 64, hi = lo + 64 < threads ? lo + 64 : threads;
    for (;;) {
        for (int i = lo; i < hi; ++i)
            if (fibres[i].state == Fibre::kRun) {
                current = i;
                thread_idx.x = i;
                swapcontext(&home, &fibres[i].ctx);
            }
        void *args[64] = {};
        int waits = 0, barriers = 0;
        Fibre *any = nullptr;
        for (int i = lo; i < hi; ++i) {
            Fibre &f = fibres[i];
            if (f.state == Fibre::kWave) {
                ++waits;
                if (any && any->op != f.op) abort();  // lanes of a wave in different operations
                any = &f;
                args[i - lo] = f.arg;
            }
            barriers += f.state == Fibre::kBarrier;
        }
        if (!waits) return;                            // at a barrier, or done
        if (barriers) abort();                         // part of a wave at a barrier
        ++wave_ops;
        any->op(args);
        for (int i = lo; i < hi; ++i)
            if (fibres[i].state == Fibre::kWave) fibres[i].state = Fibre::kRun;
    }
}
template <class F> inline void launch(F f, dim3 grid, dim3 block, size_t = 0, hipStream_t = nullptr) {
    const int threads = block.x, waves = (threads + 63) / 64;
    grid_dim = grid;
    body = f;
    if ((int)fibres.size() < threads) fibres.resize(threads);
    for (unsigned b = 0; b < grid.x; ++b) {
        block_idx.x = b;
        for (int i = 0; i < threads; ++i) {
            Fibre &x = fibres[i];
            x.stack.resize(64 << 10);
            getcontext(&x.ctx);
            x.ctx.uc_stack.ss_sp = x.stack.data();
            x.ctx.uc_stack.ss_size = x.stack.size();
            x.ctx.uc_link = nullptr;
            makecontext(&x.ctx, entry, 0);
            x.state = Fibre::kRun;
        }
        for (bool more = true; more;) {
            for (int w = 0; w < waves; ++w) run_wave(wave_order ? waves - 1 - w : w, threads);
            more = false;
            for (int i = 0; i < threads; ++i)  // waves that have ended no longer count
                if (fibres[i].state == Fibre::kBarrier) {
                    fibres[i].state = Fibre::kRun;
                    more = true;
                }
        }
    }
}

typedef uint32_t pair_u32 __attribute__((ext_vector_type(2)));
typedef float acc16 __attribute__((ext_vector_type(16)));
typedef short s4 __attribute__((ext_vector_type(4)));

template <class T> inline T shfl_xor(T v, int d) {
    struct A { T v; int d; T r; } a{v, d, v};
    wave_op(a, [](void *const *l) {
        for (int i = 0; i < 64; ++i)
            if (A *x = (A *)l[i])
                if (A *y = (A *)l[i ^ x->d]) x->r = y->v;
    });
    return a.r;
}
template <int M> inline pair_u32 permlane_swap(uint32_t x, uint32_t y) {
    struct A { uint32_t x, y; pair_u32 r; } a{x, y, {}};
    wave_op(a, [](void *const *l) {
        for (int i = 0; i < 64; ++i)
            if (A *p = (A *)l[i]) {
                const A *q = l[i ^ M] ? (A *)l[i ^ M] : p;
                p->r = i & M ? pair_u32{q->y, p->y} : pair_u32{p->x, q->x};
            }
    });
    return a.r;
}
inline uint64_t ballot(bool v) {
    struct A { bool v; uint64_t r; } a{v, 0};
    wave_op(a, [](void *const *l) {
        uint64_t m = 0;
        for (int i = 0; i < 64; ++i) m |= (uint64_t)(l[i] && ((A *)l[i])->v) << i;
        for (int i = 0; i < 64; ++i)
            if (l[i]) ((A *)l[i])->r = m;
    });
    return a.r;
}
inline int readfirstlane(int v) {
    struct A { int v, r; } a{v, 0};
    wave_op(a, [](void *const *l) {
        int i = 0;
        while (!l[i]) ++i;
        const int r = ((A *)l[i])->v;
        for (i = 0; i < 64; ++i)
            if (l[i]) ((A *)l[i])->r = r;
    });
    return a.r;
}
inline void converge() {
    struct A {} a;
    wave_op(a, [](void *const *) {});
}
inline int mov_dpp(int v, int ctrl) {
    struct A { int v, ctrl, r; } a{v, ctrl, 0};
    wave_op(a, [](void *const *l) {
        for (int i = 0; i < 64; ++i)
            if (A *x = (A *)l[i]) {
                const int s = i & 15, base = i & 48;
                const int from = x->ctrl == 0x140 ? 15 - s : x->ctrl == 0x141 ? (s & 8) | (7 - (s & 7))
                               : x->ctrl == 0x4E ? s ^ 2 : s ^ 1;
                x->r = ((A *)l[base + from])->v;
            }
    });
    return a.r;
}
// Four rows of 16 values per 16 lanes, lane i holding values 4 (i & 3) .. + 4 of row
// i >> 2: lane i receives column i.
inline s4 read_tr16(const void *p) {
    struct A { s4 v, r; } a;
    memcpy(&a.v, p, sizeof a.v);
    wave_op(a, [](void *const *l) {
        for (int i = 0; i < 64; ++i)
            for (int j = 0; j < 4; ++j)
                ((A *)l[i])->r[j] = ((A *)l[(i & 48) + 4 * j + ((i & 15) >> 2)])->v[i & 3];
    });
    return a.r;
}
// v_mfma_f32_32x32x16_bf16
template <class V> inline acc16 mfma_32x32x16(V av, V bv, acc16 c) {
    struct A { uint16_t a[8], b[8]; acc16 c; } x;
    memcpy(x.a, &av, 16);
    memcpy(x.b, &bv, 16);
    x.c = c;
    wave_op(x, [](void *const *l) {
        auto f = [](uint16_t h) { return __uint_as_float((uint32_t)h << 16); };
        for (int i = 0; i < 64; ++i) {
            A *me = (A *)l[i];
            for (int r = 0; r < 16; ++r) {
                const int row = 8 * (r >> 2) + 4 * (i >> 5) + (r & 3);
                float s = me->c[r];
                for (int k = 0; k < 16; ++k)
                    s += f(((A *)l[row + 32 * (k >> 3)])->a[k & 7]) * f(((A *)l[(i & 31) + 32 * (k >> 3)])->b[k & 7]);
                me->c[r] = s;
            }
        }
    });
    return x.c;
}
inline uint32_t perm(uint32_t hi, uint32_t lo, uint32_t sel) {
    const uint64_t v = ((uint64_t)hi << 32) | lo;
    uint32_t r = 0;
    for (int i = 0; i < 4; ++i) r |= (uint32_t)((v >> (8 * ((sel >> (8 * i)) & 7))) & 255) << (8 * i);
    return r;
}

}  // namespace emu

#define threadIdx emu::thread_idx
#define blockIdx emu::block_idx
#define gridDim emu::grid_dim
#define __syncthreads() emu::yield_as(emu::Fibre::kBarrier)
#define __shfl_xor emu::shfl_xor
#define __ballot emu::ballot
#define __lane_id() (emu::thread_idx.x & 63)
#define __builtin_amdgcn_ballot_w64 emu::ballot
#define __builtin_amdgcn_readfirstlane emu::readfirstlane
#define __builtin_amdgcn_permlane32_swap(x, y, f, b) emu::permlane_swap<32>(x, y)
#define __builtin_amdgcn_permlane16_swap(x, y, f, b) emu::permlane_swap<16>(x, y)
#define __builtin_amdgcn_mov_dpp(x, c, r, b, z) emu::mov_dpp(x, c)
#define __builtin_amdgcn_ds_read_tr16_b64_v4i16(p) emu::read_tr16((const void *)(p))
#define __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, x, y, z) emu::mfma_32x32x16(a, b, c)
#define __builtin_amdgcn_sched_barrier(m) ((void)0)
#define __builtin_amdgcn_wave_barrier emu::converge
#define __builtin_amdgcn_perm emu::perm
#define __builtin_amdgcn_mbcnt_lo(m, a) (a)
#define __builtin_amdgcn_mbcnt_hi(m, a) ((int)(emu::thread_idx.x & 63))
#define __builtin_amdgcn_exp2f exp2f
#define __builtin_amdgcn_logf log2f
#define __builtin_amdgcn_sbfe(v, o, w) ((int)((uint32_t)(v) << (32 - (w) - (o))) >> (32 - (w)))
#define __builtin_amdgcn_fdot2_f32_bf16(a, b, c, k) ((float)(a)[0] * (float)(b)[0] + (float)(a)[1] * (float)(b)[1] + (c))
