// kernels.hip -- gfx950 device code of libtsspin.
//
// Kernel families:
//   sweep_reg_kernel   one pass over a state larger than a tile.  Each workgroup owns one
//                      closed set of 2^T amplitudes (Sec. 3.3: fixing the spins outside a
//                      group of bits leaves a set closed under flipping the spins inside it)
//                      and runs a host-planned stage program on it: butterflies on the
//                      bits of one layer, the phase step, butterflies of the next layer.
//                      Each thread holds 2^RB amplitudes along a window of RB tile bits in
//                      registers; changing window is one transpose through LDS.  The low
//                      index bits always stay in the tile, so every workgroup moves
//                      contiguous runs (Sec. 3.4), and the phase is fused with the rotations
//                      (Sec. 3.1).
//   sweep_pipe_kernel  the same stages with a grid of resident workgroups that prefetch
//                      their next tile into a second register set.
//   sweep_kernel       the same pass with the tile staged in LDS (kept for tuning).
//   resident_kernel    a state that fits one workgroup's registers: a whole recording
//                      segment in one launch, one workgroup per state (or per chain of a
//                      batch).
//   reduce_kernel, batch_reduce_kernel, finalize_kernel
//                      FP64 observables of Sec. 4.2 (norm, spin components, correlations,
//                      magnetisation, overlaps) and the energy <H> of Eq. 1, with a
//                      fixed-order compensated final sum.
//   apply_obs_kernel, apply_ham_kernel, grad_reduce_kernel
//                      the adjoint: lambda = O psi (O = H for the energy), and the gradient
//                      sums in a phase frame.
//
// Phase step.  The energy of axis a is D(b) = sum_j h_j s_j + sum_(i,j) J_ij s_i s_j with
// s = +-1/2 (Sec. 2, Eqs. 1 and ZZ-Phases).  It is split by who fixes which bits:
//   workgroup  the bits outside the tile: a host table holds per tile the phase factors of
//              the outside energy and of the effective field on each tile bit;
//   thread     the tile bits outside its register window: a host table per thread pattern
//              holds the pair phases among them and the fields they put on window bits;
//   element    a Gray-code walk over the window bits times a table of the couplings
//              inside the window.
// Every phase argument and phase factor is FP64 for both storage precisions.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>
#include <type_traits>

#include "kernels.hpp"

namespace tsk {

template <typename R> struct Vec;
template <> struct Vec<double> { using T = double2; };
template <> struct Vec<float> { using T = float2; };

constexpr int kThreads = 256;
constexpr int kFixedBits = 8;  // log2(kThreads): tile bits fixed per thread

__device__ __forceinline__ uint64_t dep(uint64_t x, const Run *r, int n)
{
    uint64_t out = 0;
    for (int i = 0; i < n; ++i) out |= ((x >> r[i].src) & ((1ull << r[i].len) - 1ull)) << r[i].dst;
    return out;
}

// insert a zero bit at position k
__device__ __forceinline__ uint32_t ins0(uint32_t g, int k)
{
    return ((g >> k) << (k + 1)) | (g & ((1u << k) - 1u));
}

template <typename V>
__device__ __forceinline__ void bfly(V &a, V &b)
{
    V u = a, v = b;
    a.x = u.x + v.x;
    a.y = u.y + v.y;
    b.x = u.x - v.x;
    b.y = u.y - v.y;
}

// Walsh-Hadamard butterflies on 1, 2 or 3 tile bits over the LDS tile of ne amplitudes.
template <typename V>
__device__ void wht_pass(V *tile, int ne, int nk, int k0, int k1, int k2)
{
    if (nk == 3) {
        const int ng = ne >> 3;
        const uint32_t d0 = 1u << k0, d1 = 1u << k1, d2 = 1u << k2;
        for (int g = threadIdx.x; g < ng; g += kThreads) {
            const uint32_t t = ins0(ins0(ins0((uint32_t)g, k0), k1), k2);
            V x[8];
#pragma unroll
            for (int i = 0; i < 8; ++i)
                x[i] = tile[t + ((i & 1) ? d0 : 0) + ((i & 2) ? d1 : 0) + ((i & 4) ? d2 : 0)];
#pragma unroll
            for (int s = 1; s < 8; s <<= 1)
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    if (!(i & s)) bfly(x[i], x[i + s]);
#pragma unroll
            for (int i = 0; i < 8; ++i)
                tile[t + ((i & 1) ? d0 : 0) + ((i & 2) ? d1 : 0) + ((i & 4) ? d2 : 0)] = x[i];
        }
    } else if (nk == 2) {
        const int ng = ne >> 2;
        const uint32_t d0 = 1u << k0, d1 = 1u << k1;
        for (int g = threadIdx.x; g < ng; g += kThreads) {
            const uint32_t t = ins0(ins0((uint32_t)g, k0), k1);
            V x0 = tile[t], x1 = tile[t + d0], x2 = tile[t + d1], x3 = tile[t + d0 + d1];
            bfly(x0, x1);
            bfly(x2, x3);
            bfly(x0, x2);
            bfly(x1, x3);
            tile[t] = x0;
            tile[t + d0] = x1;
            tile[t + d1] = x2;
            tile[t + d0 + d1] = x3;
        }
    } else {
        const int ng = ne >> 1;
        const uint32_t d0 = 1u << k0;
        for (int g = threadIdx.x; g < ng; g += kThreads) {
            const uint32_t t = ins0((uint32_t)g, k0);
            V x0 = tile[t], x1 = tile[t + d0];
            bfly(x0, x1);
            tile[t] = x0;
            tile[t + d0] = x1;
        }
    }
}

// All butterflies of a layer restricted to the tile bits in `mask`, three bits per pass.
template <typename V>
__device__ void wht_layer(V *tile, int ne, uint32_t mask)
{
    while (mask) {
        int k[3] = {0, 0, 0};
        int nk = 0;
        while (mask && nk < 3) {
            k[nk++] = __builtin_ctz(mask);
            mask &= mask - 1;
        }
        wht_pass(tile, ne, nk, k[0], k[1], k[2]);
        __syncthreads();
    }
}

// Complex products with explicit FMAs: the rounding is then the same in every kernel,
// whatever the compiler would otherwise contract in the surrounding code.
__device__ __forceinline__ double2 cmul(double2 a, double2 b)
{
    return make_double2(__builtin_fma(a.x, b.x, -(a.y * b.y)), __builtin_fma(a.x, b.y, a.y * b.x));
}

// multiply by i^m
__device__ __forceinline__ double2 qturn(double2 a, int m)
{
    switch (m & 3) {
    case 1: return make_double2(-a.y, a.x);
    case 2: return make_double2(-a.x, -a.y);
    case 3: return make_double2(a.y, -a.x);
    default: return a;
    }
}

__device__ __forceinline__ double2 expi(double phi)
{
    double s, c;
    sincos(phi, &s, &c);
    return make_double2(c, s);
}

// complex64: the product with the FP64 factor is formed in FP64 and rounded once.  Rounding
// the factor to FP32 first would give it a modulus 1 + O(2^-24) that every amplitude sharing
// it picks up alike: a systematic drift of the norm (about 3e-7 per fourth-order step in the
// Loschmidt echo of a 14-spin ring), where one rounding of each product leaves only
// independent errors.
__device__ __forceinline__ void apply_phase(double2 &x, double2 z) { x = cmul(x, z); }
__device__ __forceinline__ void apply_phase(float2 &x, double2 z)
{
    const double xr = x.x, xi = x.y;
    x.x = (float)__builtin_fma(xr, z.x, -(xi * z.y));
    x.y = (float)__builtin_fma(xr, z.y, xi * z.x);
}

// Per-launch table over the var bits: i^(c*popcount(j)) * exp(-i tau Q(j)), Q = the
// couplings among var bits (tile bits 8..T-1).  Built by threads j < 2^V.
template <int T>
__device__ void build_qtab(double2 *qtab, const DiagArgs &d, const double *jt)
{
    constexpr int V = (T > kFixedBits) ? T - kFixedBits : 0;
    const int j = threadIdx.x;
    if (j < (1 << V)) {
        double q = 0.0;
        if (d.axis < 3) {
#pragma unroll
            for (int v1 = 0; v1 < V; ++v1)
#pragma unroll
                for (int v2 = v1 + 1; v2 < V; ++v2) {
                    const double c = jt[(kFixedBits + v1) * T + kFixedBits + v2];
                    const double s = (((j >> v1) ^ (j >> v2)) & 1) ? -0.25 : 0.25;
                    q += c * s;
                }
        }
        qtab[j] = qturn(expi(-d.tau * q), d.qturn * __builtin_popcount(j));
    }
}

// Factors z of a phase step for the thread's 2^(T-8) amplitudes t = tid + 256*j of a tile, use(t, z).
// wg = [C, geff_0 .. geff_{T-1}] of this workgroup, jt = tile couplings (upper triangle),
// b_thread = global index of element j = 0.
template <int T, typename F>
__device__ __forceinline__ void diag_factors(int ne, const DiagArgs &d, const double *wg, const double *jt,
                                             const double2 *qtab, uint64_t b_thread, F use)
{
    constexpr int NV = (T > kFixedBits) ? T - kFixedBits : 0;
    constexpr int EPT = 1 << NV;
    constexpr int FB = (T < kFixedBits) ? T : kFixedBits;
    const int tid = threadIdx.x;
    if (tid >= ne) return;
    double C = 0.0;
    double g[NV > 0 ? NV : 1];
#pragma unroll
    for (int v = 0; v < NV; ++v) g[v] = 0.0;
    if (d.axis < 3) {
        C = wg[0];
#pragma unroll
        for (int k = 0; k < FB; ++k) C += (((tid >> k) & 1) ? 0.5 : -0.5) * wg[1 + k];
#pragma unroll
        for (int k1 = 0; k1 < FB; ++k1)
#pragma unroll
            for (int k2 = k1 + 1; k2 < FB; ++k2)
                C += jt[k1 * T + k2] * ((((tid >> k1) ^ (tid >> k2)) & 1) ? -0.25 : 0.25);
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            double gv = wg[1 + kFixedBits + v];
#pragma unroll
            for (int k = 0; k < kFixedBits; ++k)
                gv += jt[k * T + kFixedBits + v] * (((tid >> k) & 1) ? 0.5 : -0.5);
            g[v] = gv;
        }
    }
    // energy of element j = 0 (all var bits down) without the var-var part (in qtab)
    double e0 = C;
#pragma unroll
    for (int v = 0; v < NV; ++v) e0 -= 0.5 * g[v];
    double2 p = cmul(make_double2(d.kre, d.kim), expi(-d.tau * e0));
    p = qturn(p, d.qturn * __popcll(b_thread));
    double2 w[NV > 0 ? NV : 1];
#pragma unroll
    for (int v = 0; v < NV; ++v) w[v] = expi(-d.tau * g[v]);
#pragma unroll
    for (int k = 0; k < EPT; ++k) {
        const int j = k ^ (k >> 1);
        if (k > 0) {
            const int v = __builtin_ctz(k);
            const double2 wv = ((j >> v) & 1) ? w[v] : make_double2(w[v].x, -w[v].y);
            p = cmul(p, wv);
        }
        use(tid + kThreads * j, cmul(p, qtab[j]));
    }
}

// Phase step on the thread's amplitudes of the LDS tile.
template <int T, typename V>
__device__ void diag_step(V *tile, int ne, const DiagArgs &d, const double *wg, const double *jt,
                          const double2 *qtab, uint64_t b_thread)
{
    diag_factors<T>(ne, d, wg, jt, qtab, b_thread, [&](int t, double2 z) {
        V x = tile[t];
        apply_phase(x, z);
        tile[t] = x;
    });
}

template <typename R, int T>
__global__ __launch_bounds__(kThreads) void sweep_kernel(typename Vec<R>::T *__restrict__ psi,
                                                         SweepArgs a)
{
    using V = typename Vec<R>::T;
    constexpr int NE = 1 << T;
    constexpr int EPT = NE / kThreads;
    constexpr int NV = T - kFixedBits;
    __shared__ V tile[NE];
    __shared__ double2 qtab[1 << NV];
    const int tid = threadIdx.x;
    const uint64_t base = dep(blockIdx.x, a.out_runs, a.n_out_runs);
    const uint64_t bt = base | dep((uint64_t)tid, a.tile_runs, a.n_tile_runs);
    {
        V r[EPT];
#pragma unroll
        for (int j = 0; j < EPT; ++j)
            r[j] = psi[bt | dep((uint64_t)j << kFixedBits, a.tile_runs, a.n_tile_runs)];
#pragma unroll
        for (int j = 0; j < EPT; ++j) tile[tid + kThreads * j] = r[j];
    }
    if (a.d.axis >= 0) build_qtab<T>(qtab, a.d, a.jt);
    __syncthreads();
    wht_layer(tile, NE, a.pre_mask);
    if (a.d.axis >= 0) {
        const double *wg = (a.d.axis < 3) ? a.wg + (size_t)blockIdx.x * (T + 1) : nullptr;
        diag_step<T>(tile, NE, a.d, wg, a.jt, qtab, bt);
        __syncthreads();
    }
    wht_layer(tile, NE, a.post_mask);
    {
        V r[EPT];
#pragma unroll
        for (int j = 0; j < EPT; ++j) r[j] = tile[tid + kThreads * j];
#pragma unroll
        for (int j = 0; j < EPT; ++j)
            psi[bt | dep((uint64_t)j << kFixedBits, a.tile_runs, a.n_tile_runs)] = r[j];
    }
}

// --------------------------------------------------------- register-window sweep
//
// Each of the 2^(T-RB) threads holds 2^RB amplitudes of the tile in registers: the ones
// whose tile indices differ only in a window of RB consecutive tile bits [w, w+RB).
// Butterflies on window bits need no LDS; moving to another window is one transpose
// through a padded LDS buffer.  The stage list (window, butterfly mask, phase step) is
// planned on the host; loads and stores use windows that keep the low index bits on the
// lanes, so every wavefront instruction moves whole 128-byte lines.

// tile index of element r = 0 of thread tid in the layout with window w
template <int RB>
__device__ __forceinline__ uint32_t thread_part(uint32_t tid, int w)
{
    return (tid & ((1u << w) - 1u)) | ((tid >> w) << (w + RB));
}

__device__ __forceinline__ uint32_t lds_pos(uint32_t t) { return t + (t >> 4); }

template <int RB, typename V>
__device__ __forceinline__ void reg_bfly(V (&x)[1 << RB], uint32_t mask)
{
#pragma unroll
    for (int v = 0; v < RB; ++v) {
        if (!((mask >> v) & 1u)) continue;
#pragma unroll
        for (int r = 0; r < (1 << RB); ++r)
            if (!(r & (1 << v))) bfly(x[r], x[r | (1 << v)]);
    }
}

// Workgroup barrier that orders LDS traffic only: it waits for this wave's LDS operations
// (lgkmcnt) but not for its outstanding global loads, so prefetches stay in flight.
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

template <int RB, typename V>
__device__ __forceinline__ void reg_transpose(V (&x)[1 << RB], V *lds, int from, int to)
{
    const uint32_t tid = threadIdx.x;
    lds_barrier();
    const uint32_t tf = thread_part<RB>(tid, from);
#pragma unroll
    for (int r = 0; r < (1 << RB); ++r) lds[lds_pos(tf | ((uint32_t)r << from))] = x[r];
    lds_barrier();
    const uint32_t tt = thread_part<RB>(tid, to);
#pragma unroll
    for (int r = 0; r < (1 << RB); ++r) x[r] = lds[lds_pos(tt | ((uint32_t)r << to))];
}

// The same transpose for complex128 through an LDS buffer of doubles: real parts first,
// then imaginary parts.  Half the LDS of reg_transpose, at the cost of two more barriers.
template <int RB>
__device__ __forceinline__ void reg_transpose_half(double2 (&x)[1 << RB], double *lds, int from, int to)
{
    const uint32_t tid = threadIdx.x;
    const uint32_t tf = thread_part<RB>(tid, from);
    const uint32_t tt = thread_part<RB>(tid, to);
    lds_barrier();
#pragma unroll
    for (int r = 0; r < (1 << RB); ++r) lds[lds_pos(tf | ((uint32_t)r << from))] = x[r].x;
    lds_barrier();
#pragma unroll
    for (int r = 0; r < (1 << RB); ++r) x[r].x = lds[lds_pos(tt | ((uint32_t)r << to))];
    lds_barrier();
#pragma unroll
    for (int r = 0; r < (1 << RB); ++r) lds[lds_pos(tf | ((uint32_t)r << from))] = x[r].y;
    lds_barrier();
#pragma unroll
    for (int r = 0; r < (1 << RB); ++r) x[r].y = lds[lds_pos(tt | ((uint32_t)r << to))];
}

template <int RB, typename V>
__device__ __forceinline__ void any_transpose(V (&x)[1 << RB], V *lds, int from, int to)
{
    reg_transpose<RB>(x, lds, from, to);
}
template <int RB>
__device__ __forceinline__ void any_transpose(double2 (&x)[1 << RB], double *lds, int from, int to)
{
    reg_transpose_half<RB>(x, lds, from, to);
}

// A read-only table whose entries every lane reads at the same address: through the
// constant address space the loads become scalar loads into SGPRs, which the complex
// products then take as operands (no LDS staging, no LDS reads, no vector registers).
typedef const __attribute__((address_space(4))) double *ctab;
__device__ __forceinline__ ctab as_const(const double *p)
{
    return (ctab)(const __attribute__((address_space(4))) void *)p;
}
__device__ __forceinline__ double2 ld2(ctab t, uint32_t i) { return make_double2(t[2 * i], t[2 * i + 1]); }
// One word of every 64-byte line of the `bytes` bytes at t (L lines at most), through the
// scalar data cache: the table's later scalar loads then hit there.  The lines run from the
// one holding the first byte to the one holding the last (clamped there).
template <int L>
__device__ __forceinline__ uint32_t ctab_touch(ctab t, uint32_t bytes)
{
    typedef const __attribute__((address_space(4))) uint32_t *cword;
    const uint64_t first = (uint64_t)t & ~63ull, last = ((uint64_t)t + bytes - 1) & ~63ull;
    uint32_t acc = 0;
#pragma unroll
    for (int l = 0; l < L; ++l) {
        const uint64_t at = first + 64 * l;
        acc ^= *(cword)(at < last ? at : last);
    }
    return acc;
}

// Streaming access to the state, which a sweep reads and writes once: loads and stores
// with the non-temporal hint (the light-cone sweeps at N = 27 ran 2% faster with it).
__device__ __forceinline__ double2 ntload(const double2 *p)
{
    return make_double2(__builtin_nontemporal_load(&p->x), __builtin_nontemporal_load(&p->y));
}
__device__ __forceinline__ float2 ntload(const float2 *p)
{
    return make_float2(__builtin_nontemporal_load(&p->x), __builtin_nontemporal_load(&p->y));
}
__device__ __forceinline__ void ntstore(double2 *p, double2 v)
{
    __builtin_nontemporal_store(v.x, &p->x);
    __builtin_nontemporal_store(v.y, &p->y);
}
__device__ __forceinline__ void ntstore(float2 *p, float2 v)
{
    __builtin_nontemporal_store(v.x, &p->x);
    __builtin_nontemporal_store(v.y, &p->y);
}

// entry i of a table of (re, im) pairs in LDS or, read with scalar loads, in memory
__device__ __forceinline__ double2 tab2(const double2 *t, uint32_t i) { return t[i]; }
__device__ __forceinline__ double2 tab2(ctab t, uint32_t i) { return ld2(t, i); }
// exp(0) on every entry: the workgroup row of a phase step without energy
__constant__ double kUnitRow[2 * 16] = {1, 0, 1, 0, 1, 0, 1, 0, 1, 0, 1, 0, 1, 0, 1, 0,
                                        1, 0, 1, 0, 1, 0, 1, 0, 1, 0, 1, 0, 1, 0, 1, 0};

// Workgroup phase factors in LDS: wgf[0] = kappa exp(-i tau C), wgf[1+k] = exp(-i tau geff_k/2)
// for every tile bit k (C, geff: the outside-bit energy and fields of this workgroup).
// Thread k <= T passes entry k of its tile's row of the host factor table ((1, 0) when the
// phase step has no energy).
template <int T>
__device__ __forceinline__ void put_wgf(double2 *wgf, const DiagArgs &d, double2 f)
{
    const int k = threadIdx.x;
    if (k <= T) wgf[k] = k == 0 ? cmul(make_double2(d.kre, d.kim), f) : f;
}

// Phase step on the registers in the layout with window w.  With s = bit - 1/2 and the
// tile bits split into the thread's bits (outside the window) and the window bits v,
//   E = C + sum_thr s_k geff_k + sum_(thr pairs) J s s + sum_v s_v (geff_{w+v} + h_v) + Q(r),
//   h_v = sum_thr J_{k,w+v} s_k,  Q = couplings inside the window,
// so exp(-i tau E) is a product of: the workgroup factors wgf; a host table per thread
// pattern (thread pairs with their quarter turns, and exp(-i tau h_v/2)); and, per element,
// a Gray-code walk over the window bits times the window table q[r].  wgf and q are in LDS
// or read with scalar loads (W, Q); w0 is entry 0 of wgf (with the step's scalar kappa).
template <int T, int RB, typename V, typename W, typename Q>
__device__ void reg_diag_tab(V (&x)[1 << RB], const DiagArgs &d, W wgf, double2 w0,
                             const double2 (&th)[1 + RB], Q q, uint32_t t0, uint64_t base, int w)
{
    double2 p = qturn(cmul(w0, th[0]), d.qturn * __popcll(base));
#pragma unroll
    for (int k = 0; k < T; ++k) {
        if ((unsigned)(k - w) < (unsigned)RB) continue;
        const double2 G = tab2(wgf, 1 + k);
        p = cmul(p, ((t0 >> k) & 1) ? G : make_double2(G.x, -G.y));
    }
    double2 wv[RB];
#pragma unroll
    for (int v = 0; v < RB; ++v) {
        const double2 u = cmul(tab2(wgf, 1 + w + v), th[1 + v]);
        p = cmul(p, make_double2(u.x, -u.y));  // window bits start down: s = -1/2
        wv[v] = cmul(u, u);
    }
#pragma unroll
    for (int k = 0; k < (1 << RB); ++k) {
        const int j = k ^ (k >> 1);
        if (k > 0) {
            const int v = __builtin_ctz(k);
            p = cmul(p, ((j >> v) & 1) ? wv[v] : make_double2(wv[v].x, -wv[v].y));
        }
        apply_phase(x[j], cmul(p, tab2(q, j)));
    }
}

// One tile per workgroup; overlap of memory and ALU comes from the other resident
// workgroups of the CU.  L is the LDS element of the transposes (the amplitude type, or
// double for the half-buffer complex128 variant).
// sin and cos of x for |x| < 2^20 (the host checks the bound), to a few ulp: Cody and
// Waite's reduction by pi/2 (pi/2 = P1 + P2, P1 holding 27 significant bits so that k * P1 is
// exact) to |r| <= pi/4, then the Taylor series of sin r and cos r through r^17 and r^16
// (truncation below 1e-18 there), in Horner form in r^2.  The library sincos carries a
// path for arbitrary arguments whose registers the sweep cannot spare.
__device__ __forceinline__ void sincos_bounded(double x, double *sn, double *cs)
{
    constexpr double P1 = 1.570796325802803, P2 = 9.920935796805404e-10;
    const double k = rint(x * 0.63661977236758134);   // 2 / pi
    double r = __builtin_fma(-k, P1, x);
    r = __builtin_fma(-k, P2, r);
    const double z = r * r;
    double ps = 1.0 / 355687428096000.0;                // 1/17!
    ps = __builtin_fma(ps, z, -1.0 / 1307674368000.0);  // 1/15!
    ps = __builtin_fma(ps, z, 1.0 / 6227020800.0);
    ps = __builtin_fma(ps, z, -1.0 / 39916800.0);
    ps = __builtin_fma(ps, z, 1.0 / 362880.0);
    ps = __builtin_fma(ps, z, -1.0 / 5040.0);
    ps = __builtin_fma(ps, z, 1.0 / 120.0);
    ps = __builtin_fma(ps, z, -1.0 / 6.0);
    const double s0 = __builtin_fma(ps * z, r, r);
    double pc = 1.0 / 20922789888000.0;                 // 1/16!
    pc = __builtin_fma(pc, z, -1.0 / 87178291200.0);    // 1/14!
    pc = __builtin_fma(pc, z, 1.0 / 479001600.0);
    pc = __builtin_fma(pc, z, -1.0 / 3628800.0);
    pc = __builtin_fma(pc, z, 1.0 / 40320.0);
    pc = __builtin_fma(pc, z, -1.0 / 720.0);
    pc = __builtin_fma(pc, z, 1.0 / 24.0);
    pc = __builtin_fma(pc, z, -0.5);
    const double c0 = __builtin_fma(pc, z, 1.0);
    const int q = (int)k & 3;
    *sn = q == 0 ? s0 : q == 1 ? c0 : q == 2 ? -s0 : -c0;
    *cs = q == 0 ? c0 : q == 1 ? -s0 : q == 2 ? -c0 : s0;
}

// Phase step from an energy table: register r holds basis index b = gd | off[r], whose
// energy D_axis(b) is read from HBM; the factor kappa i^(c popcount(b)) exp(-i tau D) is
// formed in FP64 (argument and sin/cos) and applied with one rounding.
template <int RB, typename V, typename ET>
__device__ __forceinline__ void reg_diag_etab(V (&x)[1 << RB], const DiagArgs &d, const ET *et, uint64_t gd,
                                              const uint64_t *off, bool energy)
{
    ET e[1 << RB];
    if (energy) {
#pragma unroll
        for (int r = 0; r < (1 << RB); ++r) e[r] = et[gd | off[r]];
    }
#pragma unroll
    for (int r = 0; r < (1 << RB); ++r) {
        double sn = 0.0, cs = 1.0;
        if (energy) sincos_bounded(d.tau * (double)e[r], &sn, &cs);
        const double2 z = qturn(cmul(make_double2(d.kre, d.kim), make_double2(cs, -sn)),
                                d.qturn * __popcll(gd | off[r]));
        apply_phase(x[r], z);
    }
}

template <typename R, int T, int RB, typename L, bool ETAB = false>
__device__ __forceinline__ void reg_sweep(typename Vec<R>::T *__restrict__ psi, const RegSweepArgs &a, L *lds)
{
    using V = typename Vec<R>::T;
    constexpr int E = 1 << RB;
    const uint32_t tid = threadIdx.x;
    uint64_t tile = blockIdx.x;
    const double *wgp = a.wgf;
    const double *dtp = a.dtab;
    if (a.chains) {  // batched: this workgroup's chain
        const uint64_t c = tile / a.tiles_per_chain;
        tile -= c * a.tiles_per_chain;
        const ChainPtrs cp = a.chains[c];
        psi = static_cast<V *>(cp.psi);
        wgp = cp.wgf;
        dtp = cp.dtab;
    } else {
        if (a.psi2 && tile >= a.n_tiles) {  // second state of a pair launch
            psi = static_cast<V *>(a.psi2);
            tile -= a.n_tiles;
        }
        if (a.reverse) tile = a.n_tiles - 1 - tile;
        // Rotated order: workgroups launched together then take tiles spread over the top
        // bits of the tile index instead of neighbouring ones.  A strided tile reads short
        // runs far apart; neighbouring strided tiles read neighbouring runs at the same far
        // offsets.  Spreading them over the address space ran about 5% faster on an 8 GiB
        // state (the host sets rot for large states' strided groups only).
        if (a.rot) {
            const int nb = 63 - __builtin_clzll(a.n_tiles);
            tile = (tile >> a.rot) | ((tile & ((1ull << a.rot) - 1)) << (nb - a.rot));
        }
    }
    const bool has_diag = a.diag_win >= 0;
    const uint64_t base = dep(tile, a.out_runs, a.n_out_runs);
    V x[E];
    {
        const uint64_t gb = base | dep(thread_part<RB>(tid, a.load_win), a.tile_runs, a.n_tile_runs);
#pragma unroll
        for (int r = 0; r < E; ++r) x[r] = ntload(&psi[gb | a.load_off[r]]);
    }
    // this thread's row of the host phase table; the workgroup's row of factors (exp(0)
    // everywhere for a step without energy) and the window table, read with scalar loads at
    // the phase step
    double2 th[1 + RB];
    ctab wrow = as_const(kUnitRow), qtab = as_const(kUnitRow);
    if (!ETAB && has_diag) {
        const double2 *dt = reinterpret_cast<const double2 *>(dtp);
#pragma unroll
        for (int v = 0; v <= RB; ++v) th[v] = dt[(size_t)tid * (1 + RB) + v];
        qtab = as_const(dtp) + 2 * ((size_t)1 << (T - RB)) * (1 + RB);
        if (a.d.axis < 3) wrow = as_const(wgp) + 2 * tile * (T + 1);
        // bring both into the scalar cache behind the tile's loads
        const uint32_t t = ctab_touch<((T + 1) * 16 + 63) / 64 + 1>(wrow, 16 * (T + 1)) ^
                           ctab_touch<(16 << RB) / 64>(qtab, 16 << RB);
        asm volatile("" ::"s"(t));
    }
    int cur = a.load_win;
    for (int s = 0; s < a.n_stages; ++s) {
        const uint64_t word = s < kStagesPerWord ? a.st_code[0] : a.st_code[1];
        const uint32_t code = (uint32_t)(word >> (9 * (s % kStagesPerWord))) & 0x1FFu;
        const int w = (int)(code & 15u);
        if (w != cur) {
            any_transpose<RB>(x, lds, cur, w);
            cur = w;
        }
        if (!((code >> 4) & 1u)) {
            reg_bfly<RB>(x, code >> 5);
        } else if constexpr (ETAB) {
            const uint64_t gd = base | dep(thread_part<RB>(tid, w), a.tile_runs, a.n_tile_runs);
            reg_diag_etab<RB>(x, a.d, static_cast<const R *>(a.etab), gd, a.diag_off,
                              a.etab != nullptr && a.d.axis < 3);
        } else {
            const double2 w0 = cmul(make_double2(a.d.kre, a.d.kim), ld2(wrow, 0));
            reg_diag_tab<T, RB>(x, a.d, wrow, w0, th, qtab, thread_part<RB>(tid, w), base, w);
        }
    }
    if (cur != a.store_win) any_transpose<RB>(x, lds, cur, a.store_win);
    {
        const uint64_t gb = base | dep(thread_part<RB>(tid, a.store_win), a.tile_runs, a.n_tile_runs);
#pragma unroll
        for (int r = 0; r < E; ++r) ntstore(&psi[gb | a.store_off[r]], x[r]);
    }
}

template <typename R, int T, int RB>
__global__ __launch_bounds__(1 << (T - RB)) void sweep_reg_kernel(typename Vec<R>::T *__restrict__ psi,
                                                                  RegSweepArgs a)
{
    constexpr int NE = 1 << T;
    __shared__ typename Vec<R>::T lds[NE + NE / 16];
    reg_sweep<R, T, RB>(psi, a, lds);
}

// The register-window sweep with the phase step from an energy table in HBM.
template <typename R, int T, int RB>
__global__ __launch_bounds__(1 << (T - RB)) void sweep_etab_kernel(typename Vec<R>::T *__restrict__ psi,
                                                                   RegSweepArgs a)
{
    constexpr int NE = 1 << T;
    __shared__ typename Vec<R>::T lds[NE + NE / 16];
    reg_sweep<R, T, RB, typename Vec<R>::T, true>(psi, a, lds);
}

// Energy table of one axis: out[b] = sum_i h_i s_i(b) + sum_bonds J s_i(b) s_j(b), the bonds
// read as uniform (scalar) values, each term +-J/4 by the parity of its two bits.
template <typename ET>
__global__ __launch_bounds__(kThreads) void energy_table_kernel(ET *__restrict__ out, int n,
                                                                const double *__restrict__ h,
                                                                const HamBond *__restrict__ bonds, int nb,
                                                                int axis, uint64_t count)
{
    for (uint64_t b = (uint64_t)blockIdx.x * kThreads + threadIdx.x; b < count;
         b += (uint64_t)gridDim.x * kThreads) {
        double e = 0.0;
        for (int i = 0; i < n; ++i) e += ((b >> i) & 1) ? 0.5 * h[3 * i + axis] : -0.5 * h[3 * i + axis];
        for (int k = 0; k < nb; ++k) {
            const HamBond hb = bonds[k];
            const double J = axis == 0 ? hb.jx : axis == 1 ? hb.jy : hb.jz;
            e += (((b >> hb.i) ^ (b >> hb.j)) & 1) ? -0.25 * J : 0.25 * J;
        }
        out[b] = (ET)e;
    }
}

// ------------------------------------------------------------ adjoint pair sweep
//
// One reverse sweep of the adjoint on psi (x) and lambda (y) in the same workgroup: every
// stage runs on both; the phase step forms each factor once and applies it to both, then
// takes the gradient sums of its axis in registers.  The amplitudes then sit in the frame
// of that phase step, scaled as the split-phase plan would store them, so the sums are the
// ones that plan's separate pass formed.

template <int T, int RB, typename V>
__device__ __forceinline__ void reg_diag_pair(V (&x)[1 << RB], V (&y)[1 << RB], const DiagArgs &d,
                                              const double2 *wgf, const double2 (&th)[1 + RB],
                                              const double2 *q, uint32_t t0, uint64_t base, int w)
{
    double2 p = qturn(cmul(wgf[0], th[0]), d.qturn * __popcll(base));
#pragma unroll
    for (int k = 0; k < T; ++k) {
        if ((unsigned)(k - w) < (unsigned)RB) continue;
        const double2 G = wgf[1 + k];
        p = cmul(p, ((t0 >> k) & 1) ? G : make_double2(G.x, -G.y));
    }
    double2 wv[RB];
#pragma unroll
    for (int v = 0; v < RB; ++v) {
        const double2 u = cmul(wgf[1 + w + v], th[1 + v]);
        p = cmul(p, make_double2(u.x, -u.y));
        wv[v] = cmul(u, u);
    }
#pragma unroll
    for (int k = 0; k < (1 << RB); ++k) {
        const int j = k ^ (k >> 1);
        if (k > 0) {
            const int v = __builtin_ctz(k);
            p = cmul(p, ((j >> v) & 1) ? wv[v] : make_double2(wv[v].x, -wv[v].y));
        }
        const double2 z = cmul(p, q[j]);
        apply_phase(x[j], z);
        apply_phase(y[j], z);
    }
}

// Gradient sums of one phase step from the registers of the window w: per thread the Walsh
// sums M[m] of w_j = Im(conj(y_j) x_j) over the subsets m of the window bits; each wave's
// lanes then take one parameter each and sum its sign times M over the wave's 64 lanes
// (through LDS), and one thread per parameter adds the workgroup's total to its slot.
// gm holds [waves][16][65] doubles, red [waves][64].
template <int T, int RB, typename V>
__device__ __forceinline__ void pair_grad(const V (&x)[1 << RB], const V (&y)[1 << RB], const PairGradArgs &g,
                                          uint64_t base, int w, double *gm, double *red)
{
    constexpr int E = 1 << RB;
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    constexpr int NW = (1 << (T - RB)) / 64 > 0 ? (1 << (T - RB)) / 64 : 1;
    constexpr int WL = (1 << (T - RB)) < 64 ? (1 << (T - RB)) : 64;   // threads per wave
    double M[E];
#pragma unroll
    for (int j = 0; j < E; ++j) M[j] = (double)y[j].x * (double)x[j].y - (double)y[j].y * (double)x[j].x;
#pragma unroll
    for (int k = 0; k < RB; ++k)
#pragma unroll
        for (int j = 0; j < E; ++j)
            if (!(j & (1 << k))) {
                const double w0 = M[j], w1 = M[j | (1 << k)];
                M[j] = w0 + w1;
                M[j | (1 << k)] = 0.5 * (w1 - w0);
            }
    lds_barrier();   // the transpose buffer is free: every wave is past its last transpose
    double *gw = gm + (size_t)wave * (E * 65);
#pragma unroll
    for (int m = 0; m < E; ++m) gw[m * 65 + lane] = M[m];
    lds_barrier();
    const uint32_t wbase = wave * 64u;
    for (int p0 = 0; p0 < g.np; p0 += WL) {
        const int p = p0 + (int)lane;
        double acc = 0.0;
        if (p < g.np) {
            const int i = g.pi[p], j = g.pj[p];
            int m = 0, ki = -1, kj = -1;
            double s = 1.0;
            const int bi = g.tile_bit[i];
            if (bi < 0) s = ((base >> i) & 1) ? 0.5 : -0.5;
            else if ((unsigned)(bi - w) < (unsigned)RB) m |= 1 << (bi - w);
            else ki = bi;
            if (j >= 0) {
                const int bj = g.tile_bit[j];
                if (bj < 0) s *= ((base >> j) & 1) ? 0.5 : -0.5;
                else if ((unsigned)(bj - w) < (unsigned)RB) m |= 1 << (bj - w);
                else kj = bj;
            }
            for (int t = 0; t < WL; ++t) {
                const uint32_t tp = thread_part<RB>(wbase + (uint32_t)t, w);
                double f = gw[m * 65 + t];
                if (ki >= 0) f *= ((tp >> ki) & 1) ? 0.5 : -0.5;
                if (kj >= 0) f *= ((tp >> kj) & 1) ? 0.5 : -0.5;
                acc += f;
            }
            acc *= s;
        }
        red[wave * 64 + lane] = acc;
        lds_barrier();
        if (wave == 0 && p < g.np) {
            double tot = 0.0;
            for (int v = 0; v < NW; ++v) tot += red[v * 64 + lane];
            g.slots[(size_t)blockIdx.x * g.stride + g.off + g.col[p]] += g.coef * tot;
        }
        lds_barrier();
    }
}

template <typename R, int T, int RB, typename L>
__device__ __forceinline__ void reg_sweep_pair(typename Vec<R>::T *__restrict__ psi, typename Vec<R>::T *__restrict__ lam,
                                               const RegSweepArgs &a, const PairGradArgs &g, L *lds,
                                               double2 *wgf, double2 *q, double *red)
{
    using V = typename Vec<R>::T;
    constexpr int E = 1 << RB;
    const uint32_t tid = threadIdx.x;
    uint64_t tile = blockIdx.x;
    if (a.reverse) tile = a.n_tiles - 1 - tile;
    const bool has_diag = a.diag_win >= 0;
    const uint64_t base = dep(tile, a.out_runs, a.n_out_runs);
    V x[E], y[E];
    {
        const uint64_t gb = base | dep(thread_part<RB>(tid, a.load_win), a.tile_runs, a.n_tile_runs);
#pragma unroll
        for (int r = 0; r < E; ++r) {
            x[r] = psi[gb | a.load_off[r]];
            y[r] = lam[gb | a.load_off[r]];
        }
    }
    double2 th[1 + RB];
    if (has_diag) {
        const double2 *dt = reinterpret_cast<const double2 *>(a.dtab);
#pragma unroll
        for (int v = 0; v <= RB; ++v) th[v] = dt[(size_t)tid * (1 + RB) + v];
        if (tid < (uint32_t)E) q[tid] = dt[((size_t)1 << (T - RB)) * (1 + RB) + tid];
        double2 f = make_double2(1.0, 0.0);
        if (a.d.axis < 3 && tid <= (uint32_t)T) f = reinterpret_cast<const double2 *>(a.wgf)[tile * (T + 1) + tid];
        put_wgf<T>(wgf, a.d, f);
        lds_barrier();
    }
    int cur = a.load_win;
    for (int s = 0; s < a.n_stages; ++s) {
        const uint64_t word = s < kStagesPerWord ? a.st_code[0] : a.st_code[1];
        const uint32_t code = (uint32_t)(word >> (9 * (s % kStagesPerWord))) & 0x1FFu;
        const int w = (int)(code & 15u);
        if (w != cur) {
            any_transpose<RB>(x, lds, cur, w);
            any_transpose<RB>(y, lds, cur, w);
            cur = w;
        }
        if (!((code >> 4) & 1u)) {
            reg_bfly<RB>(x, code >> 5);
            reg_bfly<RB>(y, code >> 5);
        } else {
            reg_diag_pair<T, RB>(x, y, a.d, wgf, th, q, thread_part<RB>(tid, w), base, w);
            if (a.d.axis >= 0 && a.d.axis < 3 && g.np > 0)
                pair_grad<T, RB>(x, y, g, base, w, reinterpret_cast<double *>(lds), red);
        }
    }
    if (cur != a.store_win) {
        any_transpose<RB>(x, lds, cur, a.store_win);
        any_transpose<RB>(y, lds, cur, a.store_win);
    }
    {
        const uint64_t gb = base | dep(thread_part<RB>(tid, a.store_win), a.tile_runs, a.n_tile_runs);
#pragma unroll
        for (int r = 0; r < E; ++r) {
            psi[gb | a.store_off[r]] = x[r];
            lam[gb | a.store_off[r]] = y[r];
        }
    }
}

// LDS: the transpose buffer (real and imaginary parts in turn for complex128), at least the
// gradient pass's [waves][16][65] doubles.
template <typename R, int T, int RB>
__global__ __launch_bounds__(1 << (T - RB)) void sweep_pair_kernel(typename Vec<R>::T *__restrict__ psi,
                                                                   typename Vec<R>::T *__restrict__ lam,
                                                                   RegSweepArgs a, PairGradArgs g)
{
    constexpr int NE = 1 << T;
    constexpr int NW = (1 << (T - RB)) / 64 > 0 ? (1 << (T - RB)) / 64 : 1;
    constexpr int NBUF = NE + NE / 16 > NW * 16 * 65 ? NE + NE / 16 : NW * 16 * 65;
    using L = typename std::conditional<sizeof(R) == 8, double, float2>::type;
    __shared__ L lds[NBUF];
    __shared__ double2 wgf[T + 1];
    __shared__ double2 q[1 << RB];
    __shared__ double red[NW * 64];
    reg_sweep_pair<R, T, RB>(psi, lam, a, g, lds, wgf, q, red);
}

// complex128 with half the LDS per workgroup and a register budget for three waves per SIMD:
// three workgroups per CU instead of two at T = 12.
template <int T, int RB>
__global__ __launch_bounds__(1 << (T - RB)) __attribute__((amdgpu_waves_per_eu(3)))
void sweep_half_kernel(double2 *__restrict__ psi, RegSweepArgs a)
{
    constexpr int NE = 1 << T;
    __shared__ double lds[NE + NE / 16];
    reg_sweep<double, T, RB>(psi, a, lds);
}

// Butterflies of the light-cone stage loop, written in place: (u, v) -> (u + v, (u + v) - 2v).
// A fresh register for u - v would have to be copied back at the end of every masked bit
// (the loop carries the register array): 16 moves per 32 adds.  The difference then carries
// up to one more rounding of the sum (unbiased, like the first), far inside the FP64 error
// budget; for complex64 the 1000-step C(t) error against complex128 stays at the level of
// the exact form (2e-9 at N = 24, GPU test bound 1e-5).
template <typename V>
__device__ __forceinline__ void bfly_inplace(V &a, V &b);
template <>
__device__ __forceinline__ void bfly_inplace(double2 &a, double2 &b)
{
    a.x += b.x;
    a.y += b.y;
    b.x = __builtin_fma(-2.0, b.x, a.x);
    b.y = __builtin_fma(-2.0, b.y, a.y);
}
template <>
__device__ __forceinline__ void bfly_inplace(float2 &a, float2 &b)
{
    a.x += b.x;
    a.y += b.y;
    b.x = __builtin_fmaf(-2.0f, b.x, a.x);
    b.y = __builtin_fmaf(-2.0f, b.y, a.y);
}

template <int RB, typename V>
__device__ __forceinline__ void cone_bfly(V (&x)[1 << RB], uint32_t mask)
{
#pragma unroll
    for (int v = 0; v < RB; ++v) {
        if (!((mask >> v) & 1u)) continue;
#pragma unroll
        for (int r = 0; r < (1 << RB); ++r)
            if (!(r & (1 << v))) bfly_inplace(x[r], x[r | (1 << v)]);
    }
}

// Light-cone transposes.  For disjoint bit fields lds_pos(a | b) = lds_pos(a) + lds_pos(b)
// (no carry out of the low four bits), so an element's LDS slot is the thread's base plus a
// per-register offset that is uniform (scalar) for the window.  The light-cone windows start
// at bit 0 or at a bit >= 4, where lds_pos(r << w) = r * lds_pos(1 << w): the offsets are
// multiples of one scalar stride (forming each from lds_pos took ~8 scalar instructions).  One code path for every pair
// of windows: the stage loop then keeps the register array in place (separate compiled
// variants per window pair made the compiler copy it between registers at every stage).
template <int RB, typename V>
__device__ __forceinline__ void cone_transpose(V (&x)[1 << RB], V *lds, int from, int to)
{
    const uint32_t tid = threadIdx.x;
    const uint32_t bf = lds_pos(thread_part<RB>(tid, from)), bt = lds_pos(thread_part<RB>(tid, to));
    const uint32_t mf = lds_pos(1u << from), mt = lds_pos(1u << to);
    V *pf = lds + bf, *pt = lds + bt;
    lds_barrier();
#pragma unroll
    for (int r = 0; r < (1 << RB); ++r) pf[r * mf] = x[r];
    lds_barrier();
#pragma unroll
    for (int r = 0; r < (1 << RB); ++r) x[r] = pt[r * mt];
}

// Elements of a transpose buffer, and whether two full ones leave room for a second workgroup on
// the CU (160 KB).
__host__ __device__ constexpr int cone_buffer(int T) { return (1 << T) + (1 << T) / 16; }
template <int T, typename L>
__host__ __device__ constexpr bool cone_two_buffers()
{
    return 2 * cone_buffer(T) * sizeof(L) <= 80 * 1024 - 1024;
}

// The same through two full buffers in turn (`lds`: the one that the transpose before did not
// use): the barrier between has seen every wave past its reads of it, so one barrier is enough.
template <int RB, typename V>
__device__ __forceinline__ void cone_transpose_next(V (&x)[1 << RB], V *lds, int from, int to)
{
    const uint32_t tid = threadIdx.x;
    const uint32_t bf = lds_pos(thread_part<RB>(tid, from)), bt = lds_pos(thread_part<RB>(tid, to));
    const uint32_t mf = lds_pos(1u << from), mt = lds_pos(1u << to);
    V *pf = lds + bf, *pt = lds + bt;
#pragma unroll
    for (int r = 0; r < (1 << RB); ++r) pf[r * mf] = x[r];
    lds_barrier();
#pragma unroll
    for (int r = 0; r < (1 << RB); ++r) x[r] = pt[r * mt];
}

// complex128 through the half buffer: real parts, then imaginary parts
template <int RB>
__device__ __forceinline__ void cone_transpose(double2 (&x)[1 << RB], double *lds, int from, int to)
{
    const uint32_t tid = threadIdx.x;
    const uint32_t bf = lds_pos(thread_part<RB>(tid, from)), bt = lds_pos(thread_part<RB>(tid, to));
    const uint32_t mf = lds_pos(1u << from), mt = lds_pos(1u << to);
    double *pf = lds + bf, *pt = lds + bt;
    lds_barrier();
#pragma unroll
    for (int r = 0; r < (1 << RB); ++r) pf[r * mf] = x[r].x;
    lds_barrier();
#pragma unroll
    for (int r = 0; r < (1 << RB); ++r) x[r].x = pt[r * mt];
    lds_barrier();
#pragma unroll
    for (int r = 0; r < (1 << RB); ++r) pf[r * mf] = x[r].y;
    lds_barrier();
#pragma unroll
    for (int r = 0; r < (1 << RB); ++r) x[r].y = pt[r * mt];
}

// Both vectors of the adjoint pair through two buffers at once: half the barriers of two
// transposes in turn.
template <int RB>
__device__ __forceinline__ void cone_transpose_pair(double2 (&x)[1 << RB], double2 (&y)[1 << RB], double *lx,
                                                    double *ly, int from, int to)
{
    const uint32_t tid = threadIdx.x;
    const uint32_t bf = lds_pos(thread_part<RB>(tid, from)), bt = lds_pos(thread_part<RB>(tid, to));
    const uint32_t mf = lds_pos(1u << from), mt = lds_pos(1u << to);
    double *fx = lx + bf, *tx = lx + bt, *fy = ly + bf, *ty = ly + bt;
    lds_barrier();
#pragma unroll
    for (int r = 0; r < (1 << RB); ++r) {
        fx[r * mf] = x[r].x;
        fy[r * mf] = y[r].x;
    }
    lds_barrier();
#pragma unroll
    for (int r = 0; r < (1 << RB); ++r) {
        x[r].x = tx[r * mt];
        y[r].x = ty[r * mt];
    }
    lds_barrier();
#pragma unroll
    for (int r = 0; r < (1 << RB); ++r) {
        fx[r * mf] = x[r].y;
        fy[r * mf] = y[r].y;
    }
    lds_barrier();
#pragma unroll
    for (int r = 0; r < (1 << RB); ++r) {
        x[r].y = tx[r * mt];
        y[r].y = ty[r * mt];
    }
}
template <int RB, typename V>
__device__ __forceinline__ void cone_transpose_pair(V (&x)[1 << RB], V (&y)[1 << RB], V *lx, V *ly, int from,
                                                    int to)
{
    const uint32_t tid = threadIdx.x;
    const uint32_t bf = lds_pos(thread_part<RB>(tid, from)), bt = lds_pos(thread_part<RB>(tid, to));
    const uint32_t mf = lds_pos(1u << from), mt = lds_pos(1u << to);
    V *fx = lx + bf, *tx = lx + bt, *fy = ly + bf, *ty = ly + bt;
    lds_barrier();
#pragma unroll
    for (int r = 0; r < (1 << RB); ++r) {
        fx[r * mf] = x[r];
        fy[r * mf] = y[r];
    }
    lds_barrier();
#pragma unroll
    for (int r = 0; r < (1 << RB); ++r) {
        x[r] = tx[r * mt];
        y[r] = ty[r * mt];
    }
}

// apply_phase in place: the same four operations, with the results tied to the amplitude's
// registers.  Left to itself the compiler writes the products of a whole phase step to other
// registers and copies them back at the end of the stage (32 moves, and 64 registers more).
__device__ __forceinline__ void apply_cone(double2 &x, double2 z)
{
    const double t = x.y * z.y, u = x.y * z.x;
    asm("v_fma_f64 %0, %1, %2, %3" : "+v"(x.y) : "v"(x.x), "v"(z.y), "v"(u));
    asm("v_fma_f64 %0, %0, %1, -%2" : "+v"(x.x) : "v"(z.x), "v"(t));
}
__device__ __forceinline__ void apply_cone(float2 &x, double2 z) { apply_phase(x, z); }

// Row of a phase step's workgroup table that this tile selects (its outside spins).
__device__ __forceinline__ uint64_t cone_row(const ConePhaseArgs &ph, uint64_t tile)
{
    const uint32_t *rb = reinterpret_cast<const uint32_t *>(ph.row_bit);
    uint64_t row = 0;
    for (int b = 0; b < ph.n_row_bits; ++b)
        row |= ((tile >> ((rb[b >> 2] >> (8 * (b & 3))) & 0xffu)) & 1ull) << b;
    return row;
}

// The phase tables are reached through pointers stored in the sweep arguments; these name
// global memory, which lets the compiler use global (not flat) loads for them.
typedef const __attribute__((address_space(1))) double *gtab;
__device__ __forceinline__ gtab as_global(const double *p)
{
    return (gtab)(const __attribute__((address_space(1))) void *)p;
}
// a 64-bit value that is the same in every lane, held in scalar registers
__device__ __forceinline__ uint64_t uniform64(uint64_t v)
{
    return ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(v >> 32)) << 32) |
           (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
}
// complex entry i of a global table of (re, im) pairs
__device__ __forceinline__ double2 gload2(gtab t, size_t i)
{
    return make_double2(t[2 * i], t[2 * i + 1]);
}

// Phase step of a light-cone sweep in window w.  Each step holds few terms, so the product is
// built only from its non-trivial parts: the thread table entry and the workgroup row entry
// (which already hold the couplings and row fields of the window bits with every window bit
// down), the row-dependent fields of the thread bits in xmask, per window bit the factor that
// flips it up (exactly 1 + 0i for a bit without thread or row couplings), and one window-table
// factor per register.  Most light-cone steps of a chain couple the lowest or the highest
// window bit, or both, to the rest of the tile (bonds at the window's edges): register j takes
// P[lowest bit of j, highest bit of j] * q[j].  One code path serves every such mask, and the
// inner bits of other masks come in beside it: with a copy of the loop per mask the
// compiler moved the amplitudes to other registers and back around them (32 to 64 moves per
// step, and as many registers more).  wgf is the workgroup's row of the step (w0: its entry 0 times the step's
// scalar), q the window table, row the thread's table row.
template <int T, int RB, bool FEW, typename V>
__device__ __forceinline__ void cone_diag(V (&x)[1 << RB], ctab wgf, double2 w0, ctab q, const double2 (&th)[3],
                                          uint32_t cmask, uint32_t xmask, gtab row, int w)
{
    constexpr uint32_t HI = 1u << (RB - 1);
    const uint32_t t0 = thread_part<RB>(threadIdx.x, w);
    double2 P[4];
    P[0] = cmul(w0, th[0]);
    uint32_t m = xmask & ~(((1u << RB) - 1u) << w);
    while (m) {
        const int k = __builtin_ctz(m);
        m &= m - 1u;
        const double2 G = ld2(wgf, 1 + k);
        P[0] = cmul(P[0], ((t0 >> k) & 1) ? G : make_double2(G.x, -G.y));
    }
    P[1] = P[0];
    if (cmask & 1u) P[1] = cmul(P[0], cmul(ld2(wgf, 1 + w), th[1]));
    P[2] = P[0];
    P[3] = P[1];
    if (cmask & HI) {
        const double2 f = cmul(ld2(wgf, RB + w), th[2]);
        P[2] = cmul(P[0], f);
        P[3] = cmul(P[1], f);
    }
    const bool inner = (cmask & ~(1u | HI)) != 0;
    auto bit_factor = [&](int v) { return cmul(ld2(wgf, 1 + w + v), gload2(row, 1 + v)); };
    if constexpr (std::is_same<V, double2>::value) {
        // complex128: the inner bits' factors first (113 registers: four waves per SIMD)
        if (inner) {
#pragma unroll
            for (int v = 1; v < RB - 1; ++v) {
                if (!((cmask >> v) & 1u)) continue;
                const double2 f = bit_factor(v);
#pragma unroll
                for (int j = 0; j < (1 << RB); ++j)
                    if ((j >> v) & 1) apply_cone(x[j], f);
            }
        }
#pragma unroll
        for (int j = 0; j < (1 << RB); ++j) {
            apply_cone(x[j], cmul(P[(j & 1) | ((j >> (RB - 1)) << 1)], ld2(q, j)));
            if (!FEW && (j & 3) == 3) __builtin_amdgcn_sched_barrier(0);
        }
    } else {
        // complex64 of few tiles: one product and one rounding per amplitude whatever the mask, by
        // the operations of cone_diag_cm and cone_diag_walk for that mask: the registers in
        // Gray-code order, and other masks walk along, P[0] the walk's factor
        double2 z[1 << RB];
        if (inner) {
#pragma unroll
            for (int k = 0; k < (1 << RB); ++k) {
                const int j = k ^ (k >> 1), v = k ? __builtin_ctz(k) : 0;
                if (k > 0) {
                    const double2 f = bit_factor(v);
                    P[0] = cmul(P[0], ((j >> v) & 1) ? f : make_double2(f.x, -f.y));
                }
                z[k] = cmul(P[0], ld2(q, j));
            }
        } else {
#pragma unroll
            for (int k = 0; k < (1 << RB); ++k) {
                const int j = k ^ (k >> 1);
                z[k] = cmul(P[(j & 1) | ((j >> (RB - 1)) << 1)], ld2(q, j));
            }
        }
#pragma unroll
        for (int k = 0; k < (1 << RB); ++k) apply_cone(x[k ^ (k >> 1)], z[k]);
    }
}

// The phase step of complex64 sweeps of many tiles: a copy of the products per mask.  The
// amplitudes take half the registers of complex128, so four waves per SIMD fit anyway (110
// registers), and the one path above, four products at a time to keep its registers, is slower:
// N = 27 chain 10.56 against 10.82 ms per fourth-order step, N = 26 with next-nearest bonds 6.31
// and 7.44.  First any mask, as a Gray-code walk over the registers (flipping bit v up multiplies
// by the square of its two factors; exactly 1 + 0i for a bit without couplings).
template <int T, int RB, typename V>
__device__ __forceinline__ void cone_diag_walk(V (&x)[1 << RB], ctab wgf, double2 w0, ctab q,
                                               const double2 (&th)[1 + RB], uint32_t xmask, int w)
{
    const uint32_t tid = threadIdx.x;
    const uint32_t t0 = thread_part<RB>(tid, w);
    double2 p = cmul(w0, th[0]);
    uint32_t m = xmask & ~(((1u << RB) - 1u) << w);
    while (m) {
        const int k = __builtin_ctz(m);
        m &= m - 1u;
        const double2 G = ld2(wgf, 1 + k);
        p = cmul(p, ((t0 >> k) & 1) ? G : make_double2(G.x, -G.y));
    }
    double2 wv[RB];
#pragma unroll
    for (int v = 0; v < RB; ++v) wv[v] = cmul(ld2(wgf, 1 + w + v), th[1 + v]);
#pragma unroll
    for (int k = 0; k < (1 << RB); ++k) {
        const int j = k ^ (k >> 1);
        if (k > 0) {
            const int v = __builtin_ctz(k);
            p = cmul(p, ((j >> v) & 1) ? wv[v] : make_double2(wv[v].x, -wv[v].y));
        }
        apply_cone(x[j], cmul(p, ld2(q, j)));
    }
}
// ... and the masks in which only the window bits in CM (known when compiling) have walk
// factors other than exactly 1 + 0i: the products P[s] = p * prod_{v in s} wv[v] over the
// subsets s of CM (2^|CM| - 1 complex products), and register j takes P[j & CM] * q[j].
template <int T, int RB, uint32_t CM, typename V>
__device__ __forceinline__ void cone_diag_cm(V (&x)[1 << RB], ctab wgf, double2 w0, ctab q,
                                             const double2 (&th)[1 + RB], uint32_t xmask, int w)
{
    const uint32_t t0 = thread_part<RB>(threadIdx.x, w);
    double2 P[1 << RB];
    P[0] = cmul(w0, th[0]);
    uint32_t m = xmask & ~(((1u << RB) - 1u) << w);
    while (m) {
        const int k = __builtin_ctz(m);
        m &= m - 1u;
        const double2 G = ld2(wgf, 1 + k);
        P[0] = cmul(P[0], ((t0 >> k) & 1) ? G : make_double2(G.x, -G.y));
    }
#pragma unroll
    for (int v = 0; v < RB; ++v) {
        if (!((CM >> v) & 1u)) continue;
        const double2 f = cmul(ld2(wgf, 1 + w + v), th[1 + v]);
        const uint32_t lower = CM & ((1u << v) - 1u);
#pragma unroll
        for (uint32_t s = 0; s < (1u << RB); ++s)
            if ((s & ~lower) == 0) P[s | (1u << v)] = cmul(P[s], f);
    }
#pragma unroll
    for (int j = 0; j < (1 << RB); ++j) apply_cone(x[j], cmul(P[j & CM], ld2(q, j)));
}

// ... on two vectors (the adjoint's psi and lambda), each factor formed once; the row and the
// window table are in LDS.
template <int T, int RB, typename V>
__device__ __forceinline__ void cone_phase_pair(V (&x)[1 << RB], V (&y)[1 << RB], const ConePhaseArgs &ph,
                                                const double2 *wgf, const double2 *q,
                                                const double2 (&th)[1 + RB], int w)
{
    constexpr uint32_t HI = 1u << (RB - 1);
    const uint32_t t0 = thread_part<RB>(threadIdx.x, w), cmask = ph.cmask;
    double2 P[4];
    P[0] = cmul(wgf[0], th[0]);
    uint32_t m = ph.xmask & ~(((1u << RB) - 1u) << w);
    while (m) {
        const int k = __builtin_ctz(m);
        m &= m - 1u;
        const double2 G = wgf[1 + k];
        P[0] = cmul(P[0], ((t0 >> k) & 1) ? G : make_double2(G.x, -G.y));
    }
    P[1] = P[0];
    if (cmask & 1u) P[1] = cmul(P[0], cmul(wgf[1 + w], th[1]));
    P[2] = P[0];
    P[3] = P[1];
    if (cmask & HI) {
        const double2 f = cmul(wgf[RB + w], th[RB]);
        P[2] = cmul(P[0], f);
        P[3] = cmul(P[1], f);
    }
    const bool inner = (cmask & ~(1u | HI)) != 0;
#pragma unroll
    for (int i = 0; i < (1 << (RB - 2)); ++i) {
        double2 z[4] = {P[0], P[1], P[2], P[3]};
        if (i > 0 && inner) {  // the set bits' factors in ascending order
#pragma unroll
            for (int v = 1; v < RB - 1; ++v) {
                if (!((i >> (v - 1)) & 1)) continue;
                const double2 f = cmul(wgf[1 + w + v], th[1 + v]);
                z[0] = cmul(z[0], f);
                z[1] = cmul(z[1], f);
            }
            const double2 f = cmul(wgf[RB + w], th[RB]);
            z[2] = cmul(z[0], f);
            z[3] = cmul(z[1], f);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) z[e] = cmul(z[e], q[(e & 1) | (i << 1) | ((e >> 1) << (RB - 1))]);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int j = (e & 1) | (i << 1) | ((e >> 1) << (RB - 1));
            apply_cone(x[j], z[e]);
            apply_cone(y[j], z[e]);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

__device__ __forceinline__ double wave_sum(double v);

// Observables of a recorded segment from the tile the last light-cone sweep of a vector is
// about to store (its addresses gb | off[r] are the basis indices): one observable at a time,
// FP64 sums over the thread's amplitudes (four bra amplitudes in flight: the register budget
// of the sweep), then a wave reduction and one row of partials per workgroup.  (The kinds'
// code once per register and observable was 60 KB of instructions that no cache kept.)  At
// most kConeRecMax observables per vector.
template <typename R, int RB>
__device__ __forceinline__ void cone_record(const typename Vec<R>::T (&x)[1 << RB], uint64_t gb,
                                            const uint64_t *off, const ConeRec &rec, double *red)
{
    using V = typename Vec<R>::T;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nw = blockDim.x >> 6;
#pragma unroll 1
    for (int o = 0; o < rec.n_obs; ++o) {
        const ObsDev ob = rec.obs[o];
        double a0 = 0.0, a1 = 0.0;
        if (obs_complex(ob.kind)) {
            const V *bra = static_cast<const V *>(rec.bra[o]);
#pragma unroll
            for (int r = 0; r < (1 << RB); r += 4) {
                V w[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) w[e] = bra[gb | off[r + e]];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const double cr = x[r + e].x, ci = x[r + e].y;
                    const double s = ob.kind == kObsOverlap ? 1.0 : (((gb | off[r + e]) >> ob.i) & 1) ? 0.5 : -0.5;
                    a0 += s * ((double)w[e].x * cr + (double)w[e].y * ci);
                    a1 += s * ((double)w[e].x * ci - (double)w[e].y * cr);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        } else {
#pragma unroll
            for (int r = 0; r < (1 << RB); ++r) {
                const uint64_t b = gb | off[r];
                const double cr = x[r].x, ci = x[r].y;
                double f = 1.0;
                if (ob.kind == 3) f = ((b >> ob.i) & 1) ? 0.5 : -0.5;
                if (ob.kind == 4) f = (((b >> ob.i) ^ (b >> ob.j)) & 1) ? -0.25 : 0.25;
                if (ob.kind == 5) f = (double)__popcll(b) - 0.5 * rec.n;
                a0 += f * (cr * cr + ci * ci);
            }
        }
        a0 = wave_sum(a0);
        a1 = wave_sum(a1);
        if (lane == 0) {
            red[2 * wv] = a0;
            red[2 * wv + 1] = a1;
        }
        __syncthreads();
        if (threadIdx.x < 2) {
            double sum = 0.0;
            for (int w = 0; w < nw; ++w) sum += red[2 * w + threadIdx.x];
            rec.partials[(size_t)blockIdx.x * (2 * kMaxObs) + 2 * ob.slot + threadIdx.x] = sum;
        }
        __syncthreads();
    }
}

// Every phase step's workgroup row (T + 1 entries) and window table (2^RB entries) into LDS
// (the adjoint's pair sweep, which ran 3% slower with the one-vector sweep's scalar loads).
// Wave v takes the steps v, v + NW, ...: a step's arguments are then uniform (scalar loads;
// the row bits are read as whole words, since scalar loads of single bytes do not exist and
// a vector load would wait behind the tile's), lanes 0..T load its row entries and lanes
// T+1..T+2^RB its window entries, and every step's loads are issued before any is written,
// so they go out right behind the tile's own loads instead of one dependent round trip after
// another.  The caller's barrier makes them visible.
template <int T, int RB>
__device__ __forceinline__ void cone_tables(const ConeArgs *__restrict__ a, uint64_t tile, double2 *wgf,
                                            double2 *qt)
{
    constexpr int E = 1 << RB;
    constexpr uint32_t kThr = 1u << (T - RB);
    const uint32_t tid = threadIdx.x;
    const int nph = a->n_phases;
    constexpr int NW = (int)(kThr / 64);
    constexpr int K = (kConePhases + NW - 1) / NW;
    static_assert(NW >= 1 && T + 1 + E <= 64, "one wave holds a step's tables");
    const int wv = __builtin_amdgcn_readfirstlane((int)(tid >> 6));
    const int lane = (int)(tid & 63);
    const bool row_lane = lane <= T, win_lane = lane > T && lane <= T + E;
    double2 f[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int p = wv + k * NW;
        if (p >= nph) break;
        const ConePhaseArgs &ph = a->ph[p];
        const uint32_t *rb = reinterpret_cast<const uint32_t *>(ph.row_bit);
        uint64_t row = 0;
        for (int b = 0; b < ph.n_row_bits; ++b)
            row |= ((tile >> ((rb[b >> 2] >> (8 * (b & 3))) & 0xffu)) & 1ull) << b;
        // one load instruction for both kinds of lanes (two would share the destination
        // registers, and the second would wait for the first), from uniform table pointers
        const uint64_t pw = uniform64((uint64_t)ph.wgf), pd = uniform64((uint64_t)ph.dtab);
        const uint64_t at = row_lane ? pw + 16 * (row * (T + 1) + lane)
                                     : pd + 16 * ((uint64_t)kThr * (1 + RB) + (lane - T - 1));
        if (row_lane || win_lane) f[k] = gload2(as_global(reinterpret_cast<const double *>(at)), 0);
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int p = wv + k * NW;
        if (p >= nph) break;
        if (lane == 0) {
            const ConePhaseArgs &ph = a->ph[p];
            wgf[p * (T + 1)] = cmul(make_double2(ph.kre, ph.kim), f[k]);
        } else if (row_lane) {
            wgf[p * (T + 1) + lane] = f[k];
        } else if (win_lane) {
            qt[p * E + (lane - T - 1)] = f[k];
        }
    }
}

// The thread's row of a phase step's thread table: entry 0 always, entry 1 + v only where
// the step's walk factor for window bit v is not exactly 1 (the stage code lists them).
template <int RB>
__device__ __forceinline__ void cone_thread_row(const ConeArgs *__restrict__ a, uint32_t code, double2 (&th)[1 + RB])
{
    const gtab dt = as_global(a->ph[(code >> 9) & 63u].dtab);
    const uint32_t need = (code >> 15) & 15u;
    // the row offset is formed here, per stage: held across the stage loop it is one register
    // more than the complex128 kernel has, and the compiler spills it
    uint32_t row = threadIdx.x;
    asm volatile("" : "+v"(row));
    th[0] = gload2(dt, (size_t)row * (1 + RB));
#pragma unroll
    for (int v = 0; v < RB; ++v)
        if ((need >> v) & 1u) th[1 + v] = gload2(dt, (size_t)row * (1 + RB) + 1 + v);
}

// The same for cone_diag: the row's address, entry 0, and the entries of the lowest
// and the highest window bit where the step's walk mask is one of those two (or both); any
// other mask loads its entries when it gets there (cone_diag).
template <int RB>
__device__ __forceinline__ gtab cone_thread_ends(const ConeArgs *__restrict__ a, uint32_t code, double2 (&th)[3])
{
    const uint32_t need = (code >> 15) & 15u;
    uint32_t row = threadIdx.x;
    asm volatile("" : "+v"(row));
    const gtab dt = as_global(a->ph[(code >> 9) & 63u].dtab) + 2 * (size_t)row * (1 + RB);
    th[0] = gload2(dt, 0);
    if (need & 1u) th[1] = gload2(dt, 1);
    if ((need >> (RB - 1)) & 1u) th[2] = gload2(dt, RB);
    return dt;
}

// Reads one word of every 64-byte line of every phase step's workgroup row and window table,
// right behind the tile's loads: the steps' own scalar loads then hit the scalar cache.  (A
// launch of few workgroups per CU has too few waves to hide a trip to L2 at every step.)
// Wave v takes the steps v, v + NW, ...; every load is issued before any result is used.
template <int T, int RB>
__device__ __forceinline__ void cone_warm(const ConeArgs *__restrict__ a, uint64_t tile)
{
    constexpr int NW = (1 << (T - RB)) / 64;
    constexpr int K = (kConePhases + NW - 1) / NW;
    constexpr int RL = ((T + 1) * 16 + 63) / 64 + 1;   // lines a row can touch
    constexpr int QL = (16 << RB) / 64;                // lines of a window table
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int nph = a->n_phases;
    uint32_t acc = 0;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int p = wv + k * NW;
        if (p >= nph) break;
        const ConePhaseArgs &ph = a->ph[p];
        acc ^= ctab_touch<RL>(as_const(ph.wgf) + 2 * cone_row(ph, tile) * (T + 1), 16 * (T + 1)) ^
               ctab_touch<QL>(as_const(ph.dtab) + 2 * (1u << (T - RB)) * (1 + RB), 16 << RB);
    }
    asm volatile("" ::"s"(acc));
}

// The forms of the light-cone kernel (below).
constexpr int kConeMany = 0, kConeMid = 1, kConeFew = 2;

// Light-cone sweep.  The same register windows, transposes and phase arithmetic as the
// register-window sweep, with many phase steps per pass (each restricted to the terms that
// the host assigned to it, with its own workgroup row and tables) and separate tile-bit maps
// for the load and the store.  L is the LDS element of the transposes (double: the half
// buffer for complex128; KIND kConeFew: a full buffer, or two).  The workgroup row and the window table of a
// phase step are the same for every lane: the step reads them with scalar loads where it uses them.
template <typename R, int T, int RB, typename L, bool REC = false, int KIND = kConeMany>
__device__ __forceinline__ void cone_sweep(typename Vec<R>::T *__restrict__ psi,
                                           const ConeArgs *__restrict__ a, uint64_t tile, L *lds,
                                           const ConeRec *rec = nullptr, double *red = nullptr)
{
    using V = typename Vec<R>::T;
    constexpr int E = 1 << RB;
    const uint32_t tid = threadIdx.x;
    const uint64_t base = dep(tile, a->out_runs, a->n_out_runs);
    V x[E];
    {
        const uint64_t gb = base | dep(thread_part<RB>(tid, a->load_win), a->load_runs, a->n_load_runs);
#pragma unroll
        for (int r = 0; r < E; ++r) x[r] = ntload(&psi[gb | a->load_off[r]]);
    }
    cone_warm<T, RB>(a, tile);
    // the tile is complete (s_waitcnt vmcnt(0)): the first stage needs it anyway, and the
    // stage loop's waits then cover only the loads it issues itself
    __builtin_amdgcn_s_waitcnt(0x0F70);
    int cur = a->load_win, half = 0;
    auto transpose = [&](int to) {
        if constexpr (KIND == kConeFew && cone_two_buffers<T, L>()) {
            cone_transpose_next<RB>(x, lds + half, cur, to);
            half = cone_buffer(T) - half;
        } else {
            cone_transpose<RB>(x, lds, cur, to);
        }
    };
    const int ns = a->n_stages;
    for (int s = 0; s < ns; ++s) {
        const uint32_t code = a->st[s];
        const int w = (int)(code & 15u);
        const bool has_phase = (code >> 4) & 1u;
        const int p = (int)((code >> 9) & 63u);
        // the thread's phase-table row is loaded first: its latency then hides behind the
        // transpose and the butterflies of the stage
        constexpr bool MASKS = sizeof(R) == 4 && KIND == kConeMany;
        double2 th[MASKS ? 1 + RB : 3];
        gtab row = nullptr;
        if (has_phase) {
            if constexpr (MASKS)
                cone_thread_row<RB>(a, code, th);
            else
                row = cone_thread_ends<RB>(a, code, th);
        }
        if (w != cur) {
            transpose(w);
            cur = w;
        }
        // butterflies, then (if any) the phase step, in one stage: fewer trips through the
        // stage loop, each of which the compiler ends with copies of the register array
        const uint32_t mask = (code >> 5) & 15u;
        if (mask) cone_bfly<RB>(x, mask);
        if (has_phase) {
            const ConePhaseArgs &ph = a->ph[p];
            const ctab wp = as_const(ph.wgf) + 2 * cone_row(ph, tile) * (T + 1);
            const double2 w0 = cmul(make_double2(ph.kre, ph.kim), ld2(wp, 0));
            const ctab qp = as_const(ph.dtab) + 2 * (1u << (T - RB)) * (1 + RB);
            if constexpr (MASKS) {
                switch (ph.cmask) {
                case 0: cone_diag_cm<T, RB, 0u>(x, wp, w0, qp, th, ph.xmask, w); break;
                case 1: cone_diag_cm<T, RB, 1u>(x, wp, w0, qp, th, ph.xmask, w); break;
                case 8: cone_diag_cm<T, RB, 8u>(x, wp, w0, qp, th, ph.xmask, w); break;
                case 9: cone_diag_cm<T, RB, 9u>(x, wp, w0, qp, th, ph.xmask, w); break;
                default: cone_diag_walk<T, RB>(x, wp, w0, qp, th, ph.xmask, w); break;
                }
            } else {
                cone_diag<T, RB, KIND != kConeMany>(x, wp, w0, qp, th, ph.cmask, ph.xmask, row, w);
            }
        }
    }
    if (cur != a->store_win) transpose(a->store_win);
    {
        const uint64_t gb = base | dep(thread_part<RB>(tid, a->store_win), a->store_runs, a->n_store_runs);
        if constexpr (REC) cone_record<R, RB>(x, gb, a->store_off, *rec, red);
#pragma unroll
        for (int r = 0; r < E; ++r) ntstore(&psi[gb | a->store_off[r]], x[r]);
    }
}

// The adjoint's pair sweep stages the phase tables of a sweep (per phase step: T + 1
// workgroup-row entries, then 2^RB window entries) in dynamic LDS sized by the launch for the
// sweep's own phase steps.
template <int T, int RB>
__host__ __device__ constexpr size_t cone_tab_bytes(int n_phases)
{
    return (size_t)n_phases * ((T + 1) + (1 << RB)) * sizeof(double2);
}

// complex128 transposes through the half buffer, so that four workgroups share a CU (four waves
// per SIMD, as complex64 with its full buffer).  A launch of few workgroups leaves each CU one of
// them; its time is the latency of the chain of stages, which more registers (the phase products
// of a step all at once) and a full buffer, or two (one barrier per transpose), shorten.  But
// launches on other streams should run beside it, up to four (the hardware queues of a process):
// kConeFew, of at most half as many workgroups as CUs, stays within half a CU; kConeMid (complex128,
// up to one workgroup per CU) keeps the half buffer, and has the registers of three waves per SIMD
// (it needs 113, as kConeMany: only the order of its phase products differs).
// Eight fourth-order steps of a complex128 chain, us: N = 18 1140 as kConeFew and 1266 otherwise,
// N = 19 1205 and 1336 (four streams at once 2730 and 3100); N = 20 as kConeMid 1465 (2290
// on four streams), as kConeMany 1500 (2300), as kConeFew 1353 (3100).  Two full buffers in
// complex128 (139 KB, one workgroup per CU) took 1209 at N = 19 and 3220 on four streams.
template <typename R, int KIND>
using ConeLds = typename std::conditional<
    sizeof(R) == 8, typename std::conditional<KIND == kConeFew, double2, double>::type, float2>::type;
template <typename R, int T, int KIND>
__host__ __device__ constexpr int cone_lds()
{
    return KIND == kConeFew && cone_two_buffers<T, ConeLds<R, KIND>>() ? 2 * cone_buffer(T) : cone_buffer(T);
}
__host__ __device__ constexpr int cone_waves(int T, int kind, int many)
{
    return kind == kConeFew ? T - 10 : kind == kConeMid ? 3 : many;
}
template <typename R, int T, int RB, int KIND>
__global__ __launch_bounds__(1 << (T - RB)) __attribute__((amdgpu_waves_per_eu(cone_waves(T, KIND, 4))))
void cone_kernel(typename Vec<R>::T *__restrict__ psi, const ConeArgs *__restrict__ a, uint64_t n_tiles,
                 int reverse)
{
    __shared__ ConeLds<R, KIND> lds[cone_lds<R, T, KIND>()];
    const uint64_t tile = reverse ? n_tiles - 1 - blockIdx.x : blockIdx.x;
    cone_sweep<R, T, RB, ConeLds<R, KIND>, false, KIND>(psi, a, tile, lds);
}

// The last sweep of a vector's recorded segment, with the segment's observables (at four waves per
// SIMD its registers would spill; complex64 N = 21 511 against 527 us per two recorded steps).
template <typename R, int T, int RB, int KIND>
__global__ __launch_bounds__(1 << (T - RB)) __attribute__((amdgpu_waves_per_eu(cone_waves(T, KIND, 3))))
void cone_rec_kernel(typename Vec<R>::T *__restrict__ psi, const ConeArgs *__restrict__ a, uint64_t n_tiles,
                     int reverse, ConeRec rec)
{
    __shared__ ConeLds<R, KIND> lds[cone_lds<R, T, KIND>()];
    __shared__ double red[2 << (T - RB - 6)];
    const uint64_t tile = reverse ? n_tiles - 1 - blockIdx.x : blockIdx.x;
    cone_sweep<R, T, RB, ConeLds<R, KIND>, true, KIND>(psi, a, tile, lds, &rec, red);
}

// ------------------------------------------------------------ adjoint light-cone sweep
//
// psi (x) and lambda (y) through one stage program in the same workgroup.  Each phase step
// forms its factors once and applies them to both, then takes the gradient sums of its own
// terms (the fields and bonds of the level that the step applies): per thread the Walsh
// sums M[m] of w_j = Im(conj(y_j) x_j) over the subsets m of the register window (spin
// values +-1/2), and for each term whose window spins form m, M[m] times the spin values of
// its other spins (bits of the thread's index, or of the workgroup's tile index) times the
// step's coefficient, added to the term's accumulator acc[slot][lane] in LDS.  At the end of
// the sweep one thread per accumulator sums its 64 lanes into the workgroup's gradient row.

template <int T, int RB, typename V>
__device__ __forceinline__ void cone_pair_grad(const V (&x)[1 << RB], const V (&y)[1 << RB], double coef,
                                               uint32_t sv, uint32_t tv0, uint32_t tv1, uint32_t t0,
                                               uint32_t tile, double *acc)
{
    constexpr int E = 1 << RB;
    const uint32_t lane = threadIdx.x & 63u;
    double M[E];
#pragma unroll
    for (int j = 0; j < E; ++j) M[j] = (double)y[j].x * (double)x[j].y - (double)y[j].y * (double)x[j].x;
#pragma unroll
    for (int k = 0; k < RB; ++k)
#pragma unroll
        for (int j = 0; j < E; ++j)
            if (!(j & (1 << k))) {
                const double w0 = M[j], w1 = M[j | (1 << k)];
                M[j] = w0 + w1;
                M[j | (1 << k)] = 0.5 * (w1 - w0);
            }
    // a spin that is down contributes -1/2, one that is up +1/2: the sign is the parity of the
    // term's masked bits that are 0, set directly in the sign bit
    const uint32_t nt0 = ~t0, ntile = ~tile;
    auto term = [&](double base, int t) {
        const uint32_t w0 = (uint32_t)__builtin_amdgcn_readlane((int)tv0, t);
        const uint32_t w1 = (uint32_t)__builtin_amdgcn_readlane((int)tv1, t);
        const uint32_t par = __popc((w0 >> 12) & nt0) + __popc(w1 & ntile);
        const double v = __builtin_ldexp(base, -(int)((w0 >> 8) & 3u));
        atomicAdd(&acc[(w0 & 0xffu) * 64 + lane],
                  __hiloint2double(__double2hiint(v) ^ (int)(par << 31), __double2loint(v)));
    };
#pragma unroll
    for (int m = 0; m < E; ++m) {
        const int t1 = __builtin_amdgcn_readlane((int)sv, m + 1);
        const double base = coef * M[m];
        for (int t = __builtin_amdgcn_readlane((int)sv, m); t < t1; ++t) term(base, t);
    }
}

template <typename R, int T, int RB, typename L>
__device__ __forceinline__ void cone_pair_sweep(typename Vec<R>::T *__restrict__ psi,
                                                typename Vec<R>::T *__restrict__ lam,
                                                const ConeArgs *__restrict__ a,
                                                const ConeGradArgs *__restrict__ g, double *slots,
                                                int stride, uint64_t tile, L *lds, double2 *wgf,
                                                double2 *qt, double *acc)
{
    using V = typename Vec<R>::T;
    constexpr int E = 1 << RB;
    constexpr uint32_t kThr = 1u << (T - RB);
    constexpr int HB = (1 << T) + (1 << T) / 16;   // one transpose buffer; lds holds two
    const uint32_t tid = threadIdx.x;
    const uint64_t base = dep(tile, a->out_runs, a->n_out_runs);
    V x[E], y[E];
    {
        const uint64_t gb = base | dep(thread_part<RB>(tid, a->load_win), a->load_runs, a->n_load_runs);
#pragma unroll
        for (int r = 0; r < E; ++r) {
            x[r] = ntload(&psi[gb | a->load_off[r]]);
            y[r] = ntload(&lam[gb | a->load_off[r]]);
        }
    }
    cone_tables<T, RB>(a, tile, wgf, qt);
    const int n_slots = g->n_slots;
    for (int i = (int)tid; i < n_slots * 64; i += (int)kThr) acc[i] = 0.0;
    lds_barrier();
    __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): as in cone_sweep
    int cur = a->load_win;
    const int ns = a->n_stages;
    for (int s = 0; s < ns; ++s) {
        const uint32_t code = a->st[s];
        const int w = (int)(code & 15u);
        const bool has_phase = (code >> 4) & 1u;
        const int p = (int)((code >> 9) & 63u);
        double2 th[1 + RB];
        uint32_t sv = 0, tv0 = 0, tv1 = 0;   // the step's term offsets and terms, one per lane
        if (has_phase) {
            cone_thread_row<RB>(a, code, th);
            const uint32_t lane = tid & 63u;
            sv = (uint32_t)g->start[p][lane & 31u];
            tv0 = g->term[p][0][lane];
            tv1 = g->term[p][1][lane];
        }
        if (w != cur) {
            cone_transpose_pair<RB>(x, y, lds, lds + HB, cur, w);
            cur = w;
        }
        const uint32_t mask = (code >> 5) & 15u;
        if (mask) {
            cone_bfly<RB>(x, mask);
            cone_bfly<RB>(y, mask);
        }
        if (has_phase) {
            cone_phase_pair<T, RB>(x, y, a->ph[p], wgf + p * (T + 1), qt + p * E, th, w);
            cone_pair_grad<T, RB>(x, y, g->coef[p], sv, tv0, tv1, thread_part<RB>(tid, w), (uint32_t)tile, acc);
        }
    }
    if (cur != a->store_win) cone_transpose_pair<RB>(x, y, lds, lds + HB, cur, a->store_win);
    {
        const uint64_t gb = base | dep(thread_part<RB>(tid, a->store_win), a->store_runs, a->n_store_runs);
#pragma unroll
        for (int r = 0; r < E; ++r) {
            ntstore(&psi[gb | a->store_off[r]], x[r]);
            ntstore(&lam[gb | a->store_off[r]], y[r]);
        }
    }
    __syncthreads();
    for (int i = (int)tid; i < n_slots; i += (int)kThr) {
        double sum = 0.0;
        for (int l = 0; l < 64; ++l) sum += acc[i * 64 + l];
        slots[(size_t)blockIdx.x * stride + g->col[i]] += sum;
    }
}

// Static LDS: a transpose buffer per vector; dynamic LDS: the phase tables (cone_tab_bytes),
// then the accumulators.
template <int T, int RB>
__global__ __launch_bounds__(1 << (T - RB)) void cone_pair_c128_kernel(double2 *__restrict__ psi,
                                                                       double2 *__restrict__ lam,
                                                                       const ConeArgs *__restrict__ a,
                                                                       const ConeGradArgs *__restrict__ g,
                                                                       double *slots, int stride,
                                                                       uint64_t n_tiles, int reverse)
{
    constexpr int NE = 1 << T;
    __shared__ double lds[2 * (NE + NE / 16)];
    extern __shared__ double2 cone_dyn[];
    const uint64_t tile = reverse ? n_tiles - 1 - blockIdx.x : blockIdx.x;
    const int nph = a->n_phases;
    double2 *qt = cone_dyn + nph * (T + 1);
    cone_pair_sweep<double, T, RB>(psi, lam, a, g, slots, stride, tile, lds, cone_dyn, qt,
                                   reinterpret_cast<double *>(qt + (nph << RB)));
}

template <int T, int RB>
__global__ __launch_bounds__(1 << (T - RB)) void cone_pair_c64_kernel(float2 *__restrict__ psi,
                                                                      float2 *__restrict__ lam,
                                                                      const ConeArgs *__restrict__ a,
                                                                      const ConeGradArgs *__restrict__ g,
                                                                      double *slots, int stride,
                                                                      uint64_t n_tiles, int reverse)
{
    constexpr int NE = 1 << T;
    __shared__ float2 lds[2 * (NE + NE / 16)];
    extern __shared__ double2 cone_dyn[];
    const uint64_t tile = reverse ? n_tiles - 1 - blockIdx.x : blockIdx.x;
    const int nph = a->n_phases;
    double2 *qt = cone_dyn + nph * (T + 1);
    cone_pair_sweep<float, T, RB>(psi, lam, a, g, slots, stride, tile, lds, cone_dyn, qt,
                                  reinterpret_cast<double *>(qt + (nph << RB)));
}

// Batched: workgroup b works on tile b % tiles_per_chain of chain c = b / tiles_per_chain: its
// state starts at element off[c] of the packed buffer and its arguments for this sweep are
// args[c].  (Both are derived from kernel arguments, so the stage loop keeps its scalar
// loads and the state accesses stay global ones; pointers read from memory lose both.)
template <typename R, int T, int RB>
__global__ __launch_bounds__(1 << (T - RB)) __attribute__((amdgpu_waves_per_eu(4)))
void cone_batch_kernel(typename Vec<R>::T *__restrict__ packed, const int64_t *__restrict__ off,
                       const ConeArgs *__restrict__ args, uint64_t tiles_per_chain, int reverse)
{
    constexpr int NE = 1 << T;
    using L = typename std::conditional<sizeof(R) == 8, double, float2>::type;
    __shared__ L lds[NE + NE / 16];
    const uint64_t c = blockIdx.x / tiles_per_chain;
    uint64_t tile = blockIdx.x - c * tiles_per_chain;
    if (reverse) tile = tiles_per_chain - 1 - tile;
    cone_sweep<R, T, RB>(packed + off[c], args + c, tile, lds);
}

// Marks registers as produced here: the compiler then waits for their loads once, at this
// point, instead of conservatively inside the stage loop (where it would also wait for the
// next tile's prefetch).  Each amplitude passes through the empty asm as one whole vector
// register tuple (splitting it into its two halves as separate operands miscompiles the
// complex128 case: the store address was allocated over the imaginary half).
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));
template <int RB>
__device__ __forceinline__ void settle(double2 (&x)[1 << RB])
{
#pragma unroll
    for (int r = 0; r < (1 << RB); ++r) {
        u32x4_t t = __builtin_bit_cast(u32x4_t, x[r]);
        asm volatile("" : "+v"(t));
        x[r] = __builtin_bit_cast(double2, t);
    }
}
template <int RB>
__device__ __forceinline__ void settle(float2 (&x)[1 << RB])
{
#pragma unroll
    for (int r = 0; r < (1 << RB); ++r) {
        u32x2_t t = __builtin_bit_cast(u32x2_t, x[r]);
        asm volatile("" : "+v"(t));
        x[r] = __builtin_bit_cast(float2, t);
    }
}

// Stages and store of one tile held in registers (shared by the pipelined sweep).
template <int T, int RB, typename V>
__device__ __forceinline__ void pipe_tile(V (&x)[1 << RB], V *__restrict__ psi, const RegSweepArgs &a,
                                          V *lds, double2 *wgf, const double2 (&th)[1 + RB],
                                          const double2 *q, uint64_t base, uint64_t spart)
{
    const uint32_t tid = threadIdx.x;
    int cur = a.load_win;
    for (int s = 0; s < a.n_stages; ++s) {
        const uint64_t word = s < kStagesPerWord ? a.st_code[0] : a.st_code[1];
        const uint32_t code = (uint32_t)(word >> (9 * (s % kStagesPerWord))) & 0x1FFu;
        const int w = (int)(code & 15u);
        if (w != cur) {
            reg_transpose<RB>(x, lds, cur, w);
            cur = w;
        }
        if (!((code >> 4) & 1u)) {
            reg_bfly<RB>(x, code >> 5);
        } else {
            reg_diag_tab<T, RB>(x, a.d, wgf, wgf[0], th, q, thread_part<RB>(tid, w), base, w);
        }
    }
    if (cur != a.store_win) reg_transpose<RB>(x, lds, cur, a.store_win);
#pragma unroll
    for (int r = 0; r < (1 << RB); ++r) (psi + (base | a.store_off[r]))[spart] = x[r];
}

// Pipelined register-window sweep: a grid of resident workgroups walks the tiles with a
// stride of gridDim.x, alternating two register sets.  The global loads of the next tile
// (and its row of workgroup phase factors) are issued before the current tile's stages
// run, so each workgroup keeps HBM busy while it computes even when the LDS footprint
// allows only one or two workgroups per CU.  Stores are fire-and-forget.  Single state
// only (no batched chains).
template <typename R, int T, int RB>
__global__ __launch_bounds__(1 << (T - RB)) void sweep_pipe_kernel(typename Vec<R>::T *__restrict__ psi,
                                                                   RegSweepArgs a)
{
    using V = typename Vec<R>::T;
    constexpr int E = 1 << RB;
    constexpr int NE = 1 << T;
    __shared__ V lds[NE + NE / 16];
    __shared__ double2 wgf[2][T + 1];   // one per register set: no barrier needed before refilling
    __shared__ double2 q[E];
    const uint32_t tid = threadIdx.x;
    const uint64_t stride = gridDim.x;
    uint64_t tile = blockIdx.x;   // walk index; the tile itself is phys(tile)
    if (tile >= a.n_tiles) return;
    const uint64_t last = a.reverse ? a.n_tiles - 1 : 0;
    auto phys = [&](uint64_t t) { return a.reverse ? last - t : t; };
    const bool has_diag = a.diag_win >= 0;
    // a.wgf is never NULL here (the host passes a one-entry unit row for phase steps without
    // energy), so the loads below need no branch and stay global loads
    const bool has_wg = has_diag && a.d.axis < 3 && tid <= (uint32_t)T;
    const double2 *wgt = reinterpret_cast<const double2 *>(a.wgf);
    // Addresses: the tile base and the register offsets are uniform (scalar); only the
    // thread part is per lane, so no per-register 64-bit addresses stay live in VGPRs.
    const uint64_t lpart = dep(thread_part<RB>(tid, a.load_win), a.tile_runs, a.n_tile_runs);
    const uint64_t spart = dep(thread_part<RB>(tid, a.store_win), a.tile_runs, a.n_tile_runs);
    V xa[E], xb[E];
    double2 fa, fb;
    {
        const uint64_t tb = dep(phys(tile), a.out_runs, a.n_out_runs);
        fa = wgt[has_wg ? phys(tile) * (T + 1) + tid : 0];
#pragma unroll
        for (int r = 0; r < E; ++r) xa[r] = (psi + (tb | a.load_off[r]))[lpart];
    }
    double2 th[1 + RB];
    if (has_diag) {
        const double2 *dt = reinterpret_cast<const double2 *>(a.dtab);
#pragma unroll
        for (int v = 0; v <= RB; ++v) th[v] = dt[(size_t)tid * (1 + RB) + v];
        if (tid < (uint32_t)E) q[tid] = dt[((size_t)1 << (T - RB)) * (1 + RB) + tid];
    }
    // The prefetch is unconditional (past the end it re-reads the current tile and the data
    // is never used): a branch around it would make the compiler wait for it before the
    // stages, where the paths merge.
    for (;;) {
        // set A holds `tile` (loads in flight); prefetch the next tile into set B
        uint64_t next = tile + stride;
        {
            const uint64_t pf = phys(next < a.n_tiles ? next : tile);
            const uint64_t tb = dep(pf, a.out_runs, a.n_out_runs);
            fb = wgt[has_wg ? pf * (T + 1) + tid : 0];
#pragma unroll
            for (int r = 0; r < E; ++r) xb[r] = (psi + (tb | a.load_off[r]))[lpart];
        }
        settle<RB>(xa);
        if (has_diag) {
            put_wgf<T>(wgf[0], a.d, has_wg ? fa : make_double2(1.0, 0.0));
            lds_barrier();
        }
        pipe_tile<T, RB>(xa, psi, a, lds, wgf[0], th, q, dep(phys(tile), a.out_runs, a.n_out_runs), spart);
        tile = next;
        if (tile >= a.n_tiles) break;
        // set B holds `tile`; prefetch the next tile into set A
        next = tile + stride;
        {
            const uint64_t pf = phys(next < a.n_tiles ? next : tile);
            const uint64_t tb = dep(pf, a.out_runs, a.n_out_runs);
            fa = wgt[has_wg ? pf * (T + 1) + tid : 0];
#pragma unroll
            for (int r = 0; r < E; ++r) xa[r] = (psi + (tb | a.load_off[r]))[lpart];
        }
        settle<RB>(xb);
        if (has_diag) {
            put_wgf<T>(wgf[1], a.d, has_wg ? fb : make_double2(1.0, 0.0));
            lds_barrier();
        }
        pipe_tile<T, RB>(xb, psi, a, lds, wgf[1], th, q, dep(phys(tile), a.out_runs, a.n_out_runs), spart);
        tile = next;
        if (tile >= a.n_tiles) break;
    }
}

// ------------------------------------------------------------------ resident states
//
// A state that fits the registers of one workgroup (N <= 13, complex64 14): the whole
// segment in one launch.  One workgroup on one CU waits for no memory: its time is the
// layers' arithmetic and the exchange of amplitudes between threads, one layer after the
// other.  Each thread holds 2^RB amplitudes along a window of RB index bits, as in the
// register sweeps; a layer visits the windows from the highest to the lowest, the next layer
// from the lowest to the highest, so a layer of W windows needs W - 1 transposes through LDS
// and the phase steps run at the two end windows (complex64: always from the lowest, W
// transposes; see resident_ascending).  Windows, masks and LDS offsets are known when
// compiling.  Up to 64 threads (N <= 9) the workgroup is one wave, whose LDS operations are
// in order without barriers.
//
// Measured, per fourth-order step (20 layers) of one complex128 vector: N = 12 180 -> 48 us,
// N = 9 56 -> 17 us against the state kept in LDS (three bits per pass and a barrier after
// each).  A layer at N = 12 is then 5800 cycles: 3072 of LDS (three transposes of 64 KB each
// way at 128 bytes a cycle), 2000 of vector arithmetic, and latency at the barriers.  Eight
// amplitudes per thread (512 threads, two waves per SIMD) instead of sixteen: 48 against
// 53 us at N = 12, 25 against 31 at N = 10, although a layer then takes one transpose more.
// Real and imaginary parts exchanged apart, so that one part's butterflies run while the
// other is under way: 55 us (8-byte LDS accesses move half the bytes per cycle of 16-byte
// ones).

// Phase tables (resident_phase_entries): for the thread's bits outside the window, with every
// window bit down, th[0] = kappa i^(c popcount) exp(-i tau E); per window bit th[1 + v] =
// exp(-i tau g_v), the factor that flips it up; and the table over the window's bits of its
// own couplings and quarter turns.  Block (phase, chain), one thread per thread pattern.
__global__ void resident_phase_kernel(ResidentPhaseArgs a)
{
    const int n = a.n, T = n < 8 ? 8 : n, RB = resident_reg_bits(n), nt = 1 << (n - RB);
    const ResidentPhase ph = a.phases[blockIdx.x];
    const int w = ph.top ? n - RB : 0, tid = threadIdx.x;
    const int ax = ph.d.axis;
    const double *wg = nullptr, *jt = nullptr;
    if (ax >= 0 && ax < 3) {
        wg = a.chains ? a.chains[blockIdx.y].wg[ax] : a.wg[ax];
        jt = a.chains ? a.chains[blockIdx.y].jt[ax] : a.jt[ax];
    }
    double2 *out = reinterpret_cast<double2 *>(a.tab) +
                   ((size_t)blockIdx.y * a.n_phases + blockIdx.x) * resident_phase_entries(n);
    const uint32_t t0 = (tid & ((1u << w) - 1u)) | (((uint32_t)tid >> w) << (w + RB));
    auto spin = [&](uint32_t b, int k) { return ((b >> k) & 1u) ? 0.5 : -0.5; };
    auto inside = [&](int k) { return k >= w && k < w + RB; };
    if (tid < nt) {
        double E = wg ? wg[0] : 0.0, g[kRegBits] = {0.0, 0.0, 0.0, 0.0};
        if (wg) {
            for (int k = 0; k < n; ++k) {
                if (inside(k)) {
                    g[k - w] += wg[1 + k];
                    continue;
                }
                E += spin(t0, k) * wg[1 + k];
                for (int m = k + 1; m < n; ++m)
                    if (!inside(m)) E += spin(t0, k) * spin(t0, m) * jt[k * T + m];
            }
            for (int v = 0; v < RB; ++v) {
                for (int k = 0; k < n; ++k)
                    if (!inside(k)) g[v] += spin(t0, k) * jt[k < w ? k * T + w + v : (w + v) * T + k];
                E -= 0.5 * g[v];
            }
        }
        out[tid] = qturn(cmul(make_double2(ph.d.kre, ph.d.kim), expi(-ph.d.tau * E)), ph.d.qturn * __popc(t0));
        for (int v = 0; v < RB; ++v) out[(1 + v) * nt + tid] = expi(-ph.d.tau * g[v]);
    }
    if (tid < (1 << RB)) {
        double Q = 0.0;
        if (wg)
            for (int v = 0; v < RB; ++v)
                for (int u = v + 1; u < RB; ++u)
                    Q += spin(tid, v) * spin(tid, u) * jt[(w + v) * T + w + u];
        out[(1 + RB) * nt + tid] = qturn(expi(-ph.d.tau * Q), ph.d.qturn * __popc((uint32_t)tid));
    }
}

// Orders this workgroup's LDS operations; one wave's are in order by themselves.
template <int NT>
__device__ __forceinline__ void resident_barrier()
{
    if constexpr (NT > 64)
        lds_barrier();
    else
        asm volatile("" ::: "memory");
}

// The exchange buffer.  With two halves used in turn (B2 > 0: the offset of the other one) a
// transpose writes the half that the one before the last wrote: the barrier between has seen
// every wave past its reads, so one barrier per transpose is enough and its writes can start
// while the layer before still computes.
template <typename V, int B2>
struct ResidentLds {
    V *buf;
    bool odd;
    __device__ __forceinline__ V *next()
    {
        if constexpr (B2 == 0) return buf;
        odd = !odd;
        return buf + (odd ? B2 : 0);
    }
};

template <int NT, int RB, int FROM, int TO, typename V, int B2>
__device__ __forceinline__ void resident_transpose(V (&x)[1 << RB], ResidentLds<V, B2> &l)
{
    const uint32_t tid = threadIdx.x;
    V *lds = l.next();
    V *pf = lds + lds_pos(thread_part<RB>(tid, FROM)), *pt = lds + lds_pos(thread_part<RB>(tid, TO));
    if constexpr (B2 == 0) resident_barrier<NT>();
#pragma unroll
    for (int r = 0; r < (1 << RB); ++r) pf[lds_pos((uint32_t)r << FROM)] = x[r];
    resident_barrier<NT>();
#pragma unroll
    for (int r = 0; r < (1 << RB); ++r) x[r] = pt[lds_pos((uint32_t)r << TO)];
}

// Butterflies on the bits of window K that no lower window holds, then the windows below
// (DOWN) or above it.
template <int N, int RB, int K, bool DOWN, typename V, int B2>
__device__ __forceinline__ void resident_layer(V (&x)[1 << RB], ResidentLds<V, B2> &lds)
{
    constexpr int NW = (N + RB - 1) / RB, NT = 1 << (N - RB);
    constexpr int W = K * RB < N - RB ? K * RB : N - RB;
    reg_bfly<RB>(x, ((1u << RB) - 1u) & ~((1u << (K * RB - W)) - 1u));
    constexpr int K2 = DOWN ? K - 1 : K + 1;
    if constexpr (K2 >= 0 && K2 < NW) {
        constexpr int W2 = K2 * RB < N - RB ? K2 * RB : N - RB;
        resident_transpose<NT, RB, W, W2>(x, lds);
        resident_layer<N, RB, K2, DOWN>(x, lds);
    }
}

// Factor of register j: th[0], the factors of its set bits (the highest bit first: few
// products are alive at a time), the window table.  use(j, factor) takes them.
template <int RB, int V, typename F>
__device__ __forceinline__ void resident_phase(double2 p, int j, const double2 (&th)[1 + RB], ctab q, F use)
{
    if constexpr (V == 0) {
        use(j, cmul(p, ld2(q, j)));
    } else {
        resident_phase<RB, V - 1>(p, j, th, q, use);
        resident_phase<RB, V - 1>(cmul(p, th[V]), j | (1 << (V - 1)), th, q, use);
    }
}

// complex64: the factors of every amplitude, formed by the operations of the LDS sweep's phase
// step.  A factor that differs in its last bit now and then rounds an amplitude to the other
// FP32 neighbour, and later roundings spread that over the state; with one way to form
// them complex64 states do not depend on the kernel.  Block (phase, chain), 256 threads.
template <int T>
__global__ __launch_bounds__(kThreads) void resident_diag_kernel(ResidentPhaseArgs a)
{
    __shared__ double2 qtab[1 << (T - kFixedBits)];
    const ResidentPhase ph = a.phases[blockIdx.x];
    const int ax = ph.d.axis >= 0 && ph.d.axis < 3 ? ph.d.axis : 0;
    const double *wg = a.chains ? a.chains[blockIdx.y].wg[ax] : a.wg[ax];
    const double *jt = a.chains ? a.chains[blockIdx.y].jt[ax] : a.jt[ax];
    double2 *out = reinterpret_cast<double2 *>(a.tab) + (((size_t)blockIdx.y * a.n_phases + blockIdx.x) << a.n);
    build_qtab<T>(qtab, ph.d, jt);
    __syncthreads();
    diag_factors<T>(1 << a.n, ph.d, wg, jt, qtab, (uint64_t)threadIdx.x, [&](int t, double2 z) { out[t] = z; });
}

// The factors of the phase tables, register-major: block = phase.
template <int N>
__global__ __launch_bounds__(resident_threads(N)) void resident_factor_kernel(const double *tab, double *fac)
{
    constexpr int RB = resident_reg_bits(N), NT = 1 << (N - RB);
    const double2 *t = reinterpret_cast<const double2 *>(tab) + (size_t)blockIdx.x * resident_phase_entries(N);
    double2 *out = reinterpret_cast<double2 *>(fac) + ((size_t)blockIdx.x << N);
    double2 th[1 + RB];
#pragma unroll
    for (int v = 0; v <= RB; ++v) th[v] = t[v * NT + threadIdx.x];
    const ctab q = as_const(reinterpret_cast<const double *>(t + NT * (1 + RB)));
    resident_phase<RB, RB>(th[0], 0, th, q, [&](int j, double2 z) { out[j * NT + threadIdx.x] = z; });
}

// FP64 observables of the state in registers (window w; real kinds: norm, S^x, S^y, S^z of a
// spin, S^z S^z, M^z), written to out[slot].  S^x and S^y read the flipped partner from LDS.
template <int N, int RB, typename V>
__device__ void resident_record(const V (&x)[1 << RB], int w, V *lds, const ObsDev *obs, int n_obs, double *out)
{
    constexpr int NT = 1 << (N - RB), WAVES = NT > 64 ? NT / 64 : 1;
    __shared__ double red[WAVES][kMaxObs];
    const uint32_t t0 = thread_part<RB>(threadIdx.x, w);
    bool flips = false;
    for (int o = 0; o < n_obs; ++o) flips = flips || obs[o].kind == 1 || obs[o].kind == 2;
    resident_barrier<NT>();
    if (flips) {
#pragma unroll
        for (int r = 0; r < (1 << RB); ++r) lds[lds_pos(t0 | ((uint32_t)r << w))] = x[r];
        resident_barrier<NT>();
    }
    for (int o = 0; o < n_obs; ++o) {
        const ObsDev ob = obs[o];
        double acc = 0.0;
        if (ob.kind == 1 || ob.kind == 2) {
#pragma unroll
            for (int r = 0; r < (1 << RB); ++r) {
                const uint32_t t = t0 | ((uint32_t)r << w);
                if ((t >> ob.i) & 1) continue;
                const V u = lds[lds_pos(t | (1u << ob.i))];
                const double cr = x[r].x, ci = x[r].y;
                const double zr = cr * u.x + ci * u.y, zi = cr * u.y - ci * u.x;
                acc += (ob.kind == 1) ? zr : -zi;
            }
        } else {
#pragma unroll
            for (int r = 0; r < (1 << RB); ++r) {
                const uint32_t t = t0 | ((uint32_t)r << w);
                const double cr = x[r].x, ci = x[r].y, p = cr * cr + ci * ci;
                double f = 1.0;
                if (ob.kind == 3) f = ((t >> ob.i) & 1) ? 0.5 : -0.5;
                if (ob.kind == 4) f = (((t >> ob.i) ^ (t >> ob.j)) & 1) ? -0.25 : 0.25;
                if (ob.kind == 5) f = (double)__popc(t) - 0.5 * N;
                acc += f * p;
            }
        }
#pragma unroll
        for (int off = (NT > 64 ? 64 : NT) / 2; off > 0; off >>= 1) acc += __shfl_down(acc, off, 64);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6][o] = acc;
    }
    resident_barrier<NT>();
    for (int o = threadIdx.x; o < n_obs; o += NT) {
        double s = 0.0;
        for (int k = 0; k < WAVES; ++k) s += red[k][o];
        out[obs[o].slot] = s;
    }
    resident_barrier<NT>();
}

// SOLO: one system, alone on its CU: the phase steps multiply by factors formed once per plan,
// loaded one op ahead, and the exchange buffer is double.  Otherwise (many chains) several
// workgroups share a CU and complex128 forms the factors from the small tables (a chain's
// factors take 64 KB per phase step at N = 12, more than the caches hold for 256 chains).
// complex64 always multiplies by stored factors (resident_diag_kernel).
template <typename R, int N, bool SOLO>
__global__ __launch_bounds__(resident_threads(N)) void resident_kernel(ResidentArgs a)
{
    constexpr bool ASC = resident_ascending(std::is_same<R, float>::value);
    constexpr bool FAC = ASC || (SOLO && N <= kResidentFactorSpins), FACL = SOLO && FAC && N <= kResidentFactorLdsSpins;
    constexpr bool AHEAD = N <= kResidentFactorSpins || !FAC;   // the next step's row fits the registers
    using V = typename Vec<R>::T;
    constexpr int RB = resident_reg_bits(N), NT = 1 << (N - RB), E = 1 << RB;
    constexpr int NW = (N + RB - 1) / RB, WT = N - RB;   // windows; start of the highest one
    constexpr int HALF = (1 << N) + ((1 << N) >> 4) + 1;
    constexpr int B2 = SOLO && 2 * HALF * sizeof(V) <= 140 * 1024 ? HALF : 0;
    __shared__ V buf[HALF + B2];
    ResidentLds<V, B2> lds{buf, false};
    const uint32_t tid = threadIdx.x;
    V *psi;
    const double *tab = a.tab;
    double *rec = nullptr;
    if (a.chains) {  // batched: one chain per workgroup
        psi = static_cast<V *>(a.chains[blockIdx.x].psi);
        rec = a.chains[blockIdx.x].rec;
        tab += 2 * (size_t)blockIdx.x * a.n_phases * (ASC ? 1 << N : resident_phase_entries(N));
    } else {
        psi = reinterpret_cast<V *>(a.psi[blockIdx.x]);
    }
    V x[E];
#pragma unroll
    for (int r = 0; r < E; ++r) x[r] = psi[tid + r * NT];
    const int reps = a.n_rep > 0 ? a.n_rep : 1;
    bool top = true;   // the register window: the highest or the lowest
    // the next phase step's factors, or the thread's row of its table, loaded one op ahead
    extern __shared__ double2 resident_dyn[];
    const double2 *fac = reinterpret_cast<const double2 *>(ASC ? tab : a.fac);
    if constexpr (FACL) {
        const double2 *f = fac;
        for (int i = tid; i < a.n_phases << N; i += NT) resident_dyn[i] = f[i];   // each thread reads what it wrote
    }
    double2 th[FAC ? E : 1 + RB];
    auto load_row = [&](int phase) {
        const double2 *t = FACL  ? resident_dyn + ((size_t)phase << N)
                           : FAC ? fac + ((size_t)phase << N)
                                 : reinterpret_cast<const double2 *>(tab) + (size_t)phase * resident_phase_entries(N);
#pragma unroll
        for (int v = 0; v < (FAC ? E : 1 + RB); ++v) th[v] = t[v * NT + tid];
    };
    // the ops are read with scalar loads, two ahead
    typedef const __attribute__((address_space(4))) ResidentOp *cop;
    const cop ops = (cop)(const __attribute__((address_space(4))) void *)a.ops;
    auto op_at = [&](int s) {
        while (s >= a.n_ops) s -= a.n_ops;
        const cop o = ops + s;
        return ResidentOp{o->phase, o->post, o->rec, o->start};
    };
    ResidentOp op1{-1, 0, -1, 0}, op2 = op1;
    if (a.n_ops > 0) {
        op1 = op_at(0);
        op2 = op_at(1);
    }
    if constexpr (AHEAD) load_row(op1.phase >= 0 ? op1.phase : 0);
    if (a.rec_first) resident_record<N, RB>(x, WT, buf, a.obs, a.n_obs, a.rec_rows - a.slots);
    for (int r = 0; r < reps; ++r) {
        for (int s = 0; s < a.n_ops; ++s) {
            const ResidentOp op = op1;
            op1 = op2;
            op2 = op_at(s + 2);
            if constexpr (NW > 1 && !ASC) {
                if (op.start && !top) {  // every segment starts alike: the same arithmetic
                    resident_transpose<NT, RB, 0, WT>(x, lds);
                    top = true;
                }
            }
            if (op.phase >= 0) {
                if constexpr (!AHEAD) {
#pragma unroll
                    for (int j = 0; j < E; ++j) apply_phase(x[j], fac[((size_t)op.phase << N) + j * NT + tid]);
                } else if constexpr (FAC) {
#pragma unroll
                    for (int j = 0; j < E; ++j) apply_phase(x[j], th[j]);
                } else {
                    const ctab q = as_const(tab) +
                                   2 * ((size_t)op.phase * resident_phase_entries(N) + NT * (1 + RB));
                    resident_phase<RB, RB>(th[0], 0, th, q, [&](int j, double2 z) { apply_phase(x[j], z); });
                }
            }
            if constexpr (AHEAD) {
                if (op1.phase >= 0) load_row(op1.phase);
            }
            if (op.post) {
                if constexpr (NW == 1) {
                    resident_layer<N, RB, 0, false>(x, lds);
                } else if constexpr (ASC) {
                    resident_transpose<NT, RB, WT, 0>(x, lds);
                    resident_layer<N, RB, 0, false>(x, lds);
                } else {
                    if (top)
                        resident_layer<N, RB, NW - 1, true>(x, lds);
                    else
                        resident_layer<N, RB, 0, false>(x, lds);
                    top = !top;
                }
            }
            if (op.rec >= 0 && rec)
                resident_record<N, RB>(x, top ? WT : 0, buf, a.obs, a.n_obs, rec + (size_t)op.rec * a.slots);
        }
        if (a.rec_rows)
            resident_record<N, RB>(x, top ? WT : 0, buf, a.obs, a.n_obs, a.rec_rows + (size_t)r * a.slots);
    }
    if constexpr (NW > 1 && !ASC) {
        if (!top) resident_transpose<NT, RB, 0, WT>(x, lds);
    }
#pragma unroll
    for (int r = 0; r < E; ++r) psi[tid + r * NT] = x[r];
}

// ----------------------------------------------------------------------- reductions

__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    return v;
}

// Sums of up to NO observables.  Bound by the read of each state involved (2^27 complex128
// amplitudes and their overlap: 1.49 -> 0.70 ms, 6.1 TB/s): a thread holds kRedElems amplitudes at a
// time, loaded together, and reads a state again only where the next observable names another.
constexpr int kRedElems = 4;
template <typename R, int NO>
__global__ __launch_bounds__(kThreads) void reduce_kernel(ReduceArgs a, double *partials)
{
    using V = typename Vec<R>::T;
    constexpr int U = kRedElems;
    double acc[NO][2];
#pragma unroll
    for (int o = 0; o < NO; ++o) acc[o][0] = acc[o][1] = 0.0;
    // the observables are read from LDS where they are used: all of them held across the loop
    // do not fit the scalar registers
    __shared__ ObsDev obs[NO];
    if (threadIdx.x < NO) obs[threadIdx.x] = a.obs[threadIdx.x];
    __syncthreads();
    const uint64_t dim = 1ull << a.n;
    for (uint64_t b0 = (uint64_t)blockIdx.x * (U * kThreads); b0 < dim; b0 += (uint64_t)gridDim.x * (U * kThreads)) {
        const uint64_t b1 = b0 + threadIdx.x;
        V c[U];
        double pr[U];   // |c|^2
        int cur = -1;
        auto load = [&](V(&x)[U], int v) {
            const V *p = reinterpret_cast<const V *>(a.psi[v]);
#pragma unroll
            for (int u = 0; u < U; ++u) x[u] = b1 + u * kThreads < dim ? p[b1 + u * kThreads] : V{0, 0};
        };
#pragma unroll
        for (int o = 0; o < NO; ++o) {
            if (o >= a.n_obs) continue;
            asm volatile("" ::: "memory");
            const ObsDev ob{__builtin_amdgcn_readfirstlane(obs[o].kind), __builtin_amdgcn_readfirstlane(obs[o].i),
                            __builtin_amdgcn_readfirstlane(obs[o].j), __builtin_amdgcn_readfirstlane(obs[o].ket),
                            __builtin_amdgcn_readfirstlane(obs[o].bra), 0};
            if (ob.kind == 6) continue;
            const V *ket = reinterpret_cast<const V *>(a.psi[ob.ket]);
            if (ob.ket != cur) {
                load(c, ob.ket);
                cur = ob.ket;
#pragma unroll
                for (int u = 0; u < U; ++u) pr[u] = (double)c[u].x * c[u].x + (double)c[u].y * c[u].y;
            }
            if (obs_complex(ob.kind)) {
                V w[U];
                load(w, ob.bra);
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const double cr = c[u].x, ci = c[u].y;
                    const double f = ob.kind == kObsOverlap ? 1.0 : ((b1 + u * kThreads) >> ob.i) & 1 ? 0.5 : -0.5;
                    acc[o][0] += f * ((double)w[u].x * cr + (double)w[u].y * ci);
                    acc[o][1] += f * ((double)w[u].x * ci - (double)w[u].y * cr);
                }
                continue;
            }
            const uint64_t mi = 1ull << ob.i, mj = 1ull << ob.j;
            if (ob.kind == 1 || ob.kind == 2) {
                // every partner is loaded before one is used (a masked load each waits for its own)
                V w[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const uint64_t b = b1 + u * kThreads;
                    w[u] = ket[b < dim ? b | mi : 0];
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const double cr = c[u].x, ci = c[u].y;
                    const double z = ob.kind == 1 ? cr * w[u].x + ci * w[u].y : ci * w[u].x - cr * w[u].y;
                    acc[o][0] += ((b1 + u * kThreads) & mi) || b1 + u * kThreads >= dim ? 0.0 : z;
                }
                continue;
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint64_t b = b1 + u * kThreads;
                const double cr = c[u].x, ci = c[u].y, p = pr[u];
                switch (ob.kind) {
                case 0: acc[o][0] += p; break;
                case 3: acc[o][0] += ((b & mi) ? 0.5 : -0.5) * p; break;
                case 4: acc[o][0] += ((((b >> ob.i) ^ (b >> ob.j)) & 1) ? -0.25 : 0.25) * p; break;
                case 5: acc[o][0] += ((double)__popcll(b) - 0.5 * a.n) * p; break;
                case kObsSxSx:
                case kObsSySy:
                    // pairs (b, b + 2^i + 2^j) and (b + 2^i, b + 2^j) at the member with both bits clear
                    if (b < dim && !(b & (mi | mj))) {
                        const V c11 = ket[b | mi | mj], c01 = ket[b | mi], c10 = ket[b | mj];
                        const double A = cr * c11.x + ci * c11.y;
                        const double B = (double)c01.x * c10.x + (double)c01.y * c10.y;
                        acc[o][0] += 0.5 * (ob.kind == kObsSxSx ? A + B : B - A);
                    }
                    break;
                default: break;
                }
            }
        }
    }
    __shared__ double red[kThreads / 64][NO * 2];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
    for (int o = 0; o < NO; ++o) {
        if (o >= a.n_obs) continue;
        const double s0 = wave_sum(acc[o][0]), s1 = wave_sum(acc[o][1]);
        if (lane == 0) {
            red[wv][2 * o] = s0;
            red[wv][2 * o + 1] = s1;
        }
    }
    __syncthreads();
    if (threadIdx.x < 2 * a.n_obs && a.obs[threadIdx.x >> 1].kind != 6) {
        double s = 0.0;
        for (int w = 0; w < kThreads / 64; ++w) s += red[w][threadIdx.x];
        partials[(size_t)blockIdx.x * (2 * kMaxObs) + threadIdx.x] = s;
    }
}

// One pass of the energy (EnergyPass).  Each op reads its tile from LDS once, so a pass costs
// the read of the state or, with about ten ops, that of the tile from LDS; gathering the
// flipped partners of every basis index from memory instead read the state 0.75 times per
// bond, by lanes of which three quarters waited.  N = 24 chain, complex128: 2.3 -> 0.22 ms in three passes.  The
// next tile's amplitudes are under way while the ops run.
template <typename R, int TM>
__global__ __launch_bounds__(kThreads) void energy_kernel(const typename Vec<R>::T *__restrict__ psi, EnergyPass a,
                                                          int first, double *__restrict__ partials)
{
    using V = typename Vec<R>::T;
    constexpr int EPT = 1 << (TM - kFixedBits);
    __shared__ V tile[(1 << TM) + (1 << (TM - 4)) + 1];
    __shared__ double red[kThreads / 64];
    const uint32_t tid = threadIdx.x, ne = 1u << a.T;
    const uint64_t lpart = dep(tid, a.tile_runs, a.n_tile_runs);
    typedef const __attribute__((address_space(4))) EnergyOp *cops;
    const cops ops = (cops)(const __attribute__((address_space(4))) void *)a.ops;
    auto at = [&](uint32_t t) { return tile[lds_pos(t)]; };
    V x[EPT];
    auto fetch = [&](uint64_t t) {
        const V *p = psi + dep(t, a.out_runs, a.n_out_runs);
#pragma unroll
        for (int k = 0; k < EPT; ++k)
            x[k] = tid + k * kThreads < ne ? (p + dep(k * kThreads, a.tile_runs, a.n_tile_runs))[lpart] : V{0, 0};
    };
    double acc = 0.0;
    uint64_t t = blockIdx.x;
    if (t < a.n_tiles) fetch(t);
    for (; t < a.n_tiles; t += gridDim.x) {
        __syncthreads();
#pragma unroll
        for (int k = 0; k < EPT; ++k)
            if (tid + k * kThreads < ne) tile[lds_pos(tid + k * kThreads)] = x[k];
        __syncthreads();
        if (t + gridDim.x < a.n_tiles) fetch(t + gridDim.x);
        for (int k = 0; k < a.n_ops; ++k) {
            const cops op = ops + k;
            const int qa = op->a, qb = op->b;
            const double w0 = op->w[0], w1 = op->w[1], w2 = op->w[2], w3 = op->w[3], cA = op->cA, cB = op->cB;
            auto dot = [](V c, V u) { return (double)c.x * u.x + (double)c.y * u.y; };
            auto crs = [](V c, V u) { return (double)c.x * u.y - (double)c.y * u.x; };
            if (qb < 0) {
                if (tid < ne / 2) {
                    const V c = at(tid << 1), u = at((tid << 1) | 1);
                    acc += w0 * dot(c, c) + w1 * dot(u, u) + op->hx[0] * dot(c, u) - op->hy[0] * crs(c, u);
                }
                continue;
            }
            const uint32_t ma = 1u << qa, mb = 1u << qb;
            const int lo = qa < qb ? qa : qb, hi = qa < qb ? qb : qa;
            auto quad = [&](uint32_t q) {
                const uint32_t e = ins0(ins0(q, lo), hi);
                const V c00 = at(e), c10 = at(e | ma), c01 = at(e | mb), c11 = at(e | ma | mb);
                double v = w0 * dot(c00, c00) + w1 * dot(c10, c10) + w2 * dot(c01, c01) + w3 * dot(c11, c11);
                v += cA * dot(c00, c11) + cB * dot(c10, c01);
                if (op->flips) {
                    v += op->hx[0] * (dot(c00, c10) + dot(c01, c11)) - op->hy[0] * (crs(c00, c10) + crs(c01, c11));
                    v += op->hx[1] * (dot(c00, c01) + dot(c10, c11)) - op->hy[1] * (crs(c00, c01) + crs(c10, c11));
                }
                acc += v;
            };
            if (ne == 1u << TM) {
#pragma unroll
                for (int k2 = 0; k2 < EPT / 4; ++k2) quad(tid + k2 * kThreads);
            } else {
                for (uint32_t q = tid; q < ne / 4; q += kThreads) quad(q);
            }
        }
    }
    acc = wave_sum(acc);
    if ((tid & 63) == 0) red[tid >> 6] = acc;
    __syncthreads();
    if (tid == 0) {
        double s = 0.0;
        for (int w = 0; w < kThreads / 64; ++w) s += red[w];
        double *o = partials + (size_t)blockIdx.x * (2 * kMaxObs);
        *o = first ? s : *o + s;
    }
}

// Sum the per-block partials in a fixed order and write the requested slots: one wavefront
// per slot (a workgroup of its own: 14 slots of 1024 rows by four waves in turn took 20 us,
// at once 6), each lane a Neumaier-compensated strided sum, then a fixed shuffle tree.
__global__ __launch_bounds__(64) void finalize_kernel(const double *partials, int nblocks, ReduceArgs a,
                                                      double *out)
{
    const int lane = threadIdx.x, s = blockIdx.x, part = s & 1;
    const ObsDev ob = a.obs[s >> 1];
    if (part && !obs_complex(ob.kind)) return;
    double acc = 0.0, comp = 0.0;
#pragma unroll 4
    for (int b = lane; b < nblocks; b += 64) {
        const double x = partials[(size_t)b * (2 * kMaxObs) + s];
        const double t = acc + x;
        comp += (fabs(acc) >= fabs(x)) ? (acc - t) + x : (x - t) + acc;
        acc = t;
    }
    const double tot = wave_sum(acc + comp);
    if (lane == 0) out[ob.slot + part] = tot;
}

// Batched observables: blockIdx.y = chain, the chain's vector split over gridDim.x blocks;
// partials[(chain * gridDim.x + block) * kMaxObs + o].
template <typename R>
__global__ __launch_bounds__(kThreads) void batch_reduce_kernel(BatchReduceArgs a, double *partials)
{
    using V = typename Vec<R>::T;
    const ChainPtrs cp = a.chains[blockIdx.y];
    const V *psi = static_cast<const V *>(cp.psi);
    double acc[kMaxObs];
#pragma unroll
    for (int o = 0; o < kMaxObs; ++o) acc[o] = 0.0;
    const uint64_t dim = 1ull << a.n;
    for (uint64_t b = (uint64_t)blockIdx.x * kThreads + threadIdx.x; b < dim;
         b += (uint64_t)gridDim.x * kThreads) {
        const V c = psi[b];
        const double cr = c.x, ci = c.y, p = cr * cr + ci * ci;
#pragma unroll
        for (int o = 0; o < kMaxObs; ++o) {
            if (o >= a.n_obs) continue;
            const ObsDev ob = a.obs[o];
            switch (ob.kind) {
            case 0: acc[o] += p; break;
            case 3: acc[o] += (((b >> ob.i) & 1) ? 0.5 : -0.5) * p; break;
            case 4: acc[o] += ((((b >> ob.i) ^ (b >> ob.j)) & 1) ? -0.25 : 0.25) * p; break;
            case 5: acc[o] += ((double)__popcll(b) - 0.5 * a.n) * p; break;
            case 1:
            case 2:
                if (!((b >> ob.i) & 1)) {
                    const V u = psi[b | (1ull << ob.i)];
                    const double zr = cr * u.x + ci * u.y, zi = cr * u.y - ci * u.x;
                    acc[o] += (ob.kind == 1) ? zr : -zi;
                }
                break;
            default: break;
            }
        }
    }
    __shared__ double red[kThreads / 64][kMaxObs];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
    for (int o = 0; o < kMaxObs; ++o) {
        if (o >= a.n_obs) continue;
        const double s = wave_sum(acc[o]);
        if (lane == 0) red[wv][o] = s;
    }
    __syncthreads();
    if (threadIdx.x < a.n_obs) {
        double s = 0.0;
        for (int w = 0; w < kThreads / 64; ++w) s += red[w][threadIdx.x];
        partials[((size_t)blockIdx.y * gridDim.x + blockIdx.x) * kMaxObs + threadIdx.x] = s;
    }
}

// One workgroup per chain: sum its blocks' partials in order, write record a.rec.
__global__ __launch_bounds__(kThreads) void batch_finalize_kernel(BatchReduceArgs a, const double *partials,
                                                                  int nbpc)
{
    const ChainPtrs cp = a.chains[blockIdx.x];
    const int lane = threadIdx.x & 63;
    for (int o = threadIdx.x >> 6; o < a.n_obs; o += kThreads / 64) {
        double s = 0.0;
        for (int b = lane; b < nbpc; b += 64) s += partials[((size_t)blockIdx.x * nbpc + b) * kMaxObs + o];
        s = wave_sum(s);
        if (lane == 0) cp.rec[(size_t)a.rec * a.slots + a.obs[o].slot] = s;
    }
}

// --------------------------------------------------------------------------- adjoint

// out = O psi for the Hermitian observables (S^x, S^y, S^z of one spin, S^z S^z, M^z).
template <typename R>
__global__ __launch_bounds__(kThreads) void apply_obs_kernel(const typename Vec<R>::T *__restrict__ psi,
                                                             typename Vec<R>::T *__restrict__ out,
                                                             int kind, int i, int j, int n)
{
    using V = typename Vec<R>::T;
    const uint64_t dim = 1ull << n;
    const uint64_t m = 1ull << i;
    for (uint64_t b = (uint64_t)blockIdx.x * kThreads + threadIdx.x; b < dim;
         b += (uint64_t)gridDim.x * kThreads) {
        V o;
        if (kind == 1 || kind == 2) {
            const V c = psi[b ^ m];
            if (kind == 1) {  // (S^x psi)_b = c_{b^m} / 2
                o.x = (R)0.5 * c.x;
                o.y = (R)0.5 * c.y;
            } else {          // (S^y psi)_b = (i/2) sigma c_{b^m}, sigma = +1 for a clear bit
                const R sg = ((b >> i) & 1) ? (R)-0.5 : (R)0.5;
                o.x = -sg * c.y;
                o.y = sg * c.x;
            }
        } else {
            double f;
            if (kind == 3) f = ((b >> i) & 1) ? 0.5 : -0.5;
            else if (kind == 4) f = (((b >> i) ^ (b >> j)) & 1) ? -0.25 : 0.25;
            else f = (double)__popcll(b) - 0.5 * n;
            const V c = psi[b];
            o.x = (R)(f * c.x);
            o.y = (R)(f * c.y);
        }
        out[b] = o;
    }
}

// out = H psi, gathered per basis index b (H of Sec. 2, Eq. 1):
//   (H psi)_b = D_z(b) c_b + sum_q (h^x_q / 2 + s_q h^y_q / 2) c_{b ^ 2^q}
//             + sum_bonds (J^x / 4 + t_ij J^y / 4) c_{b ^ 2^i ^ 2^j},
// with s_q = +i if bit q of b is clear and -i if set (S^y takes up to down with +i/2), and
// t_ij = -1 if bits i and j of b are equal, +1 otherwise (the product of two such factors).
template <typename R>
__global__ __launch_bounds__(kThreads) void apply_ham_kernel(const typename Vec<R>::T *__restrict__ psi,
                                                             typename Vec<R>::T *__restrict__ out, int n,
                                                             const double *__restrict__ hf,
                                                             const HamBond *__restrict__ hb, int nb)
{
    using V = typename Vec<R>::T;
    const uint64_t dim = 1ull << n;
    for (uint64_t b = (uint64_t)blockIdx.x * kThreads + threadIdx.x; b < dim;
         b += (uint64_t)gridDim.x * kThreads) {
        const V c = psi[b];
        double dz = 0.0, orr = 0.0, oi = 0.0;
        for (int q = 0; q < n; ++q) {
            const bool up = (b >> q) & 1;
            dz += hf[3 * q + 2] * (up ? 0.5 : -0.5);
            const double hx = hf[3 * q], hy = hf[3 * q + 1];
            if (hx != 0.0 || hy != 0.0) {
                const V u = psi[b ^ (1ull << q)];
                const double sy = up ? -0.5 * hy : 0.5 * hy;   // (i sy) u
                orr += 0.5 * hx * u.x - sy * u.y;
                oi += 0.5 * hx * u.y + sy * u.x;
            }
        }
        for (int k = 0; k < nb; ++k) {
            const HamBond t = hb[k];
            const bool eq = !((((b >> t.i) ^ (b >> t.j)) & 1));
            dz += t.jz * (eq ? 0.25 : -0.25);
            if (t.jx != 0.0 || t.jy != 0.0) {
                const V u = psi[b ^ (1ull << t.i) ^ (1ull << t.j)];
                const double w = 0.25 * (t.jx + (eq ? -t.jy : t.jy));
                orr += w * u.x;
                oi += w * u.y;
            }
        }
        V o;
        o.x = (R)(dz * c.x + orr);
        o.y = (R)(dz * c.y + oi);
        out[b] = o;
    }
}

// Per-block partial sums of  sum_b f_p(b) Im(conj(lam_b) psi_b)  for a chunk of parameters
// (f = s_i for a field, s_i s_j for a coupling); both vectors are in the frame of the
// phase step that was applied last.
template <typename R>
__global__ __launch_bounds__(kThreads) void grad_reduce_kernel(const typename Vec<R>::T *__restrict__ psi,
                                                               const typename Vec<R>::T *__restrict__ lam,
                                                               GradArgs a)
{
    using V = typename Vec<R>::T;
    double acc[kGradChunk];
#pragma unroll
    for (int p = 0; p < kGradChunk; ++p) acc[p] = 0.0;
    const uint64_t dim = 1ull << a.n;
    for (uint64_t b = (uint64_t)blockIdx.x * kThreads + threadIdx.x; b < dim;
         b += (uint64_t)gridDim.x * kThreads) {
        const V u = psi[b], l = lam[b];
        const double w = (double)l.x * (double)u.y - (double)l.y * (double)u.x;
#pragma unroll
        for (int p = 0; p < kGradChunk; ++p) {
            if (p >= a.np) continue;
            const int i = a.pi[p], j = a.pj[p];
            double f;
            if (j < 0) f = ((b >> i) & 1) ? 0.5 : -0.5;
            else f = (((b >> i) ^ (b >> j)) & 1) ? -0.25 : 0.25;
            acc[p] += f * w;
        }
    }
    __shared__ double red[kThreads / 64][kGradChunk];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
    for (int p = 0; p < kGradChunk; ++p) {
        if (p >= a.np) continue;
        const double s = wave_sum(acc[p]);
        if (lane == 0) red[wv][p] = s;
    }
    __syncthreads();
    if (threadIdx.x < a.np) {
        double s = 0.0;
        for (int w = 0; w < kThreads / 64; ++w) s += red[w][threadIdx.x];
        a.slots[(size_t)blockIdx.x * a.stride + a.off + threadIdx.x] += a.coef * s;
    }
}

// The same sums for every parameter of an axis at once.  Lane t of workgroup w takes the
// amplitudes b = w * 1024 + e * 64 + t, e < 16 (coalesced loads; index bits 6-9 vary along
// e, the others are fixed for the lane) and forms the Walsh sums
// M[m] = sum_e w_e prod_{k in m} s_{6+k}(b_e) of w = Im(conj(lam) psi) over the subsets m of
// those four bits (four butterfly stages: the sum without bit k, and half the difference
// for the subsets with it, s = +-1/2).  A parameter whose spins among bits 6-9 form the set
// m then gets M[m] times s_q of each of its other spins (fixed for the lane); the host groups
// the parameters by m so that M is indexed at compile time.  One wave reduction per
// parameter; lane 0 adds the workgroup's sum to its row of the slots.
template <typename R>
__global__ __launch_bounds__(kGradWalshBlock) void grad_walsh_kernel(const typename Vec<R>::T *__restrict__ psi,
                                                                   const typename Vec<R>::T *__restrict__ lam,
                                                                   GradWalshArgs a)
{
    using V = typename Vec<R>::T;
    constexpr int L = kGradWalshLow;
    const uint64_t base = (uint64_t)blockIdx.x * (kGradWalshBlock * kGradWalshElems) + threadIdx.x;
    double M[kGradWalshElems];
#pragma unroll
    for (int e = 0; e < kGradWalshElems; ++e) {
        const V u = psi[base + ((uint64_t)e << L)], l = lam[base + ((uint64_t)e << L)];
        M[e] = (double)l.x * (double)u.y - (double)l.y * (double)u.x;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int e = 0; e < kGradWalshElems; ++e)
            if (!(e & (1 << k))) {
                const double w0 = M[e], w1 = M[e | (1 << k)];
                M[e] = w0 + w1;
                M[e | (1 << k)] = 0.5 * (w1 - w0);
            }
    // every lane's Walsh sums into LDS (row m padded to 65 entries: rows with different m
    // fall in different banks); then lane p, one parameter per lane, sums the 64 lanes'
    // entries of its row m times the signs of its spins among the lane bits 0-5, and times
    // the signs of its spins at bits 10 and above (fixed for the workgroup)
    __shared__ double gm[kGradWalshElems * 65];
#pragma unroll
    for (int m = 0; m < kGradWalshElems; ++m) gm[m * 65 + threadIdx.x] = M[m];
    __syncthreads();
    const uint64_t wbase = (uint64_t)blockIdx.x * (kGradWalshBlock * kGradWalshElems);
    double *row = a.slots + (size_t)blockIdx.x * a.stride + a.off;
    for (int p = threadIdx.x; p < a.np; p += kGradWalshBlock) {
        const int i = a.pi[p], j = a.pj[p];
        int m = 0, li = -1, lj = -1;
        double s = 1.0;
        if (i < L) li = i;
        else if (i < L + 4) m |= 1 << (i - L);
        else s = ((wbase >> i) & 1) ? 0.5 : -0.5;
        if (j >= 0) {
            if (j < L) lj = j;
            else if (j < L + 4) m |= 1 << (j - L);
            else s *= ((wbase >> j) & 1) ? 0.5 : -0.5;
        }
        double acc = 0.0;
        for (int t = 0; t < kGradWalshBlock; ++t) {
            double f = gm[m * 65 + t];
            if (li >= 0) f *= ((t >> li) & 1) ? 0.5 : -0.5;
            if (lj >= 0) f *= ((t >> lj) & 1) ? 0.5 : -0.5;
            acc += f;
        }
        row[a.col[p]] += a.coef * s * acc;
    }
}

hipError_t launch_grad_walsh(int dtype, const void *psi, const void *lam, const GradWalshArgs &a,
                             hipStream_t s)
{
    if (a.n < 10 || a.np < 1) return hipErrorInvalidValue;
    const uint32_t nblocks = (uint32_t)(1ull << (a.n - 10));
    if (dtype == 0)
        hipLaunchKernelGGL((grad_walsh_kernel<double>), dim3(nblocks), dim3(kGradWalshBlock), 0, s,
                           static_cast<const double2 *>(psi), static_cast<const double2 *>(lam), a);
    else
        hipLaunchKernelGGL((grad_walsh_kernel<float>), dim3(nblocks), dim3(kGradWalshBlock), 0, s,
                           static_cast<const float2 *>(psi), static_cast<const float2 *>(lam), a);
    return hipGetLastError();
}

// out[c] = sum over workgroups (fixed order) of the accumulated slots.
__global__ __launch_bounds__(kThreads) void grad_finalize_kernel(const double *slots, int nblocks,
                                                                 int ncols, double *out)
{
    const int lane = threadIdx.x & 63;
    for (int c = (int)(blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6)); c < ncols;
         c += (int)(gridDim.x * (kThreads / 64))) {
        double s = 0.0;
        for (int b = lane; b < nblocks; b += 64) s += slots[(size_t)b * ncols + c];
        s = wave_sum(s);
        if (lane == 0) out[c] = s;
    }
}

// ------------------------------------------------------------------------ launchers

hipError_t launch_batch_reduce(int dtype, const BatchReduceArgs &a, int nchains, double *partials,
                               int nbpc, hipStream_t s)
{
    if (dtype == 0)
        hipLaunchKernelGGL((batch_reduce_kernel<double>), dim3(nbpc, nchains), dim3(kThreads), 0, s, a,
                           partials);
    else
        hipLaunchKernelGGL((batch_reduce_kernel<float>), dim3(nbpc, nchains), dim3(kThreads), 0, s, a,
                           partials);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(batch_finalize_kernel, dim3(nchains), dim3(kThreads), 0, s, a, partials, nbpc);
    return hipGetLastError();
}

hipError_t launch_apply_obs(int dtype, const void *psi, void *out, int kind, int i, int j, int n,
                            hipStream_t s)
{
    const uint64_t dim = 1ull << n;
    uint64_t nb = (dim + kThreads - 1) / kThreads;
    if (nb > 4096) nb = 4096;
    if (dtype == 0)
        hipLaunchKernelGGL((apply_obs_kernel<double>), dim3((uint32_t)nb), dim3(kThreads), 0, s,
                           static_cast<const double2 *>(psi), static_cast<double2 *>(out), kind, i, j, n);
    else
        hipLaunchKernelGGL((apply_obs_kernel<float>), dim3((uint32_t)nb), dim3(kThreads), 0, s,
                           static_cast<const float2 *>(psi), static_cast<float2 *>(out), kind, i, j, n);
    return hipGetLastError();
}

hipError_t launch_apply_ham(int dtype, const void *psi, void *out, int n, const double *ham_h,
                            const HamBond *ham_b, int nb, hipStream_t s)
{
    const uint64_t dim = 1ull << n;
    uint64_t nblk = (dim + kThreads - 1) / kThreads;
    if (nblk > 4096) nblk = 4096;
    if (dtype == 0)
        hipLaunchKernelGGL((apply_ham_kernel<double>), dim3((uint32_t)nblk), dim3(kThreads), 0, s,
                           static_cast<const double2 *>(psi), static_cast<double2 *>(out), n, ham_h,
                           ham_b, nb);
    else
        hipLaunchKernelGGL((apply_ham_kernel<float>), dim3((uint32_t)nblk), dim3(kThreads), 0, s,
                           static_cast<const float2 *>(psi), static_cast<float2 *>(out), n, ham_h,
                           ham_b, nb);
    return hipGetLastError();
}

hipError_t launch_grad_reduce(int dtype, const void *psi, const void *lam, const GradArgs &a,
                              int nblocks, hipStream_t s)
{
    if (dtype == 0)
        hipLaunchKernelGGL((grad_reduce_kernel<double>), dim3(nblocks), dim3(kThreads), 0, s,
                           static_cast<const double2 *>(psi), static_cast<const double2 *>(lam), a);
    else
        hipLaunchKernelGGL((grad_reduce_kernel<float>), dim3(nblocks), dim3(kThreads), 0, s,
                           static_cast<const float2 *>(psi), static_cast<const float2 *>(lam), a);
    return hipGetLastError();
}

hipError_t launch_grad_finalize(const double *slots, int nblocks, int ncols, double *out, hipStream_t s)
{
    const int per = kThreads / 64;
    const int grid = (ncols + per - 1) / per;
    hipLaunchKernelGGL(grad_finalize_kernel, dim3(grid), dim3(kThreads), 0, s, slots, nblocks, ncols, out);
    return hipGetLastError();
}

template <typename R, int T>
static hipError_t launch_sweep_t(void *psi, const SweepArgs &a, uint32_t nblocks, hipStream_t s)
{
    hipLaunchKernelGGL((sweep_kernel<R, T>), dim3(nblocks), dim3(kThreads), 0, s,
                       reinterpret_cast<typename Vec<R>::T *>(psi), a);
    return hipGetLastError();
}

hipError_t launch_sweep(int dtype, int T, void *psi, const SweepArgs &a, uint32_t nblocks,
                        hipStream_t s)
{
#define TS_SW_CASE(TT) \
    case TT: return dtype == 0 ? launch_sweep_t<double, TT>(psi, a, nblocks, s) \
                               : launch_sweep_t<float, TT>(psi, a, nblocks, s);
    switch (T) {
        TS_SW_CASE(8)
        TS_SW_CASE(9)
        TS_SW_CASE(10)
        TS_SW_CASE(11)
        TS_SW_CASE(12)
        TS_SW_CASE(13)
    case 14:
        if (dtype == 1) return launch_sweep_t<float, 14>(psi, a, nblocks, s);
        break;
    default: break;
    }
#undef TS_SW_CASE
    return hipErrorInvalidValue;
}

// One workgroup per tile.
template <typename R, int T, int RB>
static hipError_t launch_reg_t(void *psi, const RegSweepArgs &a, uint64_t grid, hipStream_t s)
{
    hipLaunchKernelGGL((sweep_reg_kernel<R, T, RB>), dim3((uint32_t)grid), dim3(1 << (T - RB)),
                       0, s, reinterpret_cast<typename Vec<R>::T *>(psi), a);
    return hipGetLastError();
}

static hipError_t launch_reg_any(int dtype, int T, int RB, void *psi, const RegSweepArgs &a,
                                 uint64_t grid, hipStream_t s)
{
    if (grid == 0 || grid > 0x7fffffffull) return hipErrorInvalidValue;
#define TS_RG_CASE(TT, RR)                                                                        \
    if (T == TT && RB == RR)                                                                      \
        return dtype == 0 ? launch_reg_t<double, TT, RR>(psi, a, grid, s)                         \
                          : launch_reg_t<float, TT, RR>(psi, a, grid, s);
    TS_RG_CASE(8, 4)
    TS_RG_CASE(9, 4)
    TS_RG_CASE(10, 4)
    TS_RG_CASE(11, 4)
    TS_RG_CASE(12, 4)
    TS_RG_CASE(13, 4)
    TS_RG_CASE(8, 3)
    TS_RG_CASE(9, 3)
    TS_RG_CASE(10, 3)
    TS_RG_CASE(11, 3)
    TS_RG_CASE(12, 3)
    TS_RG_CASE(13, 3)
    if (T == 14 && RB == 4 && dtype == 1) return launch_reg_t<float, 14, 4>(psi, a, grid, s);
#undef TS_RG_CASE
    return hipErrorInvalidValue;
}

hipError_t launch_sweep_reg(int dtype, int T, int RB, void *psi, const RegSweepArgs &a, hipStream_t s)
{
    if (a.chains) return hipErrorInvalidValue;
    return launch_reg_any(dtype, T, RB, psi, a, a.psi2 ? 2 * a.n_tiles : a.n_tiles, s);
}

hipError_t launch_sweep_half(int T, int RB, void *psi, const RegSweepArgs &a, hipStream_t s)
{
    if (a.chains) return hipErrorInvalidValue;
    const uint64_t grid = a.psi2 ? 2 * a.n_tiles : a.n_tiles;
    if (grid == 0 || grid > 0x7fffffffull) return hipErrorInvalidValue;
#define TS_HALF_CASE(TT, RR)                                                                        \
    if (T == TT && RB == RR) {                                                                      \
        hipLaunchKernelGGL((sweep_half_kernel<TT, RR>), dim3((uint32_t)grid), dim3(1 << (TT - RR)), \
                           0, s, static_cast<double2 *>(psi), a);                                   \
        return hipGetLastError();                                                                   \
    }
    TS_HALF_CASE(11, 4)
    TS_HALF_CASE(12, 4)
#undef TS_HALF_CASE
    return hipErrorInvalidValue;
}

// Resident workgroups of one pipelined sweep instance: CUs x blocks per CU, cached.
template <typename R, int T, int RB>
static hipError_t launch_pipe_t(void *psi, const RegSweepArgs &a, hipStream_t s)
{
    static int resident = 0;
    if (resident == 0) {
        int dev = 0, cus = 0, per_cu = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
        if (e == hipSuccess)
            e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, sweep_pipe_kernel<R, T, RB>,
                                                             1 << (T - RB), 0);
        if (e != hipSuccess) return e;
        if (cus <= 0 || per_cu <= 0) return hipErrorInvalidConfiguration;
        resident = cus * per_cu;
    }
    const uint64_t grid = a.n_tiles < (uint64_t)resident ? a.n_tiles : (uint64_t)resident;
    if (grid == 0) return hipErrorInvalidValue;
    hipLaunchKernelGGL((sweep_pipe_kernel<R, T, RB>), dim3((uint32_t)grid), dim3(1 << (T - RB)), 0,
                       s, reinterpret_cast<typename Vec<R>::T *>(psi), a);
    return hipGetLastError();
}

hipError_t launch_sweep_pipe(int dtype, int T, int RB, void *psi, const RegSweepArgs &a, hipStream_t s)
{
    if (a.chains) return hipErrorInvalidValue;
#define TS_PIPE_CASE(TT, RR)                                                                      \
    if (T == TT && RB == RR)                                                                      \
        return dtype == 0 ? launch_pipe_t<double, TT, RR>(psi, a, s) : launch_pipe_t<float, TT, RR>(psi, a, s);
    // two register sets must fit without spills: tiles up to 2^12 (2^13 for complex64 with
    // eight amplitudes per thread)
    TS_PIPE_CASE(10, 4)
    TS_PIPE_CASE(10, 3)
    TS_PIPE_CASE(11, 4)
    TS_PIPE_CASE(11, 3)
    TS_PIPE_CASE(12, 4)
    TS_PIPE_CASE(12, 3)
    if (T == 13 && RB == 3 && dtype == 1) return launch_pipe_t<float, 13, 3>(psi, a, s);
#undef TS_PIPE_CASE
    return hipErrorInvalidValue;
}

hipError_t launch_sweep_reg_batch(int dtype, int T, int RB, const RegSweepArgs &a, uint32_t nchains,
                                  hipStream_t s)
{
    if (!a.chains || a.tiles_per_chain == 0) return hipErrorInvalidValue;
    return launch_reg_any(dtype, T, RB, nullptr, a, (uint64_t)nchains * a.tiles_per_chain, s);
}

template <typename R, int N>
static hipError_t launch_res_n(const ResidentArgs &a, int nvec, hipStream_t s)
{
    const size_t dyn = N <= kResidentFactorLdsSpins ? ((size_t)a.n_phases << N) * sizeof(double2) : 0;
    if (!a.chains && (a.fac || sizeof(R) == 4 || N > kResidentFactorSpins) && dyn <= 48 * 1024) {
        hipLaunchKernelGGL((resident_kernel<R, N, true>), dim3(nvec), dim3(resident_threads(N)), dyn, s, a);
        return hipGetLastError();
    }
    hipLaunchKernelGGL((resident_kernel<R, N, false>), dim3(nvec), dim3(resident_threads(N)), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_resident(int dtype, const ResidentArgs &a, int nvec, hipStream_t s)
{
    if (!a.tab || a.n_ops < 0 || nvec <= 0 || (a.chains && a.fac)) return hipErrorInvalidValue;
#define TS_RES_CASE(NN) \
    case NN: return dtype == 0 ? launch_res_n<double, NN>(a, nvec, s) : launch_res_n<float, NN>(a, nvec, s);
    switch (a.n) {
        TS_RES_CASE(1)
        TS_RES_CASE(2)
        TS_RES_CASE(3)
        TS_RES_CASE(4)
        TS_RES_CASE(5)
        TS_RES_CASE(6)
        TS_RES_CASE(7)
        TS_RES_CASE(8)
        TS_RES_CASE(9)
        TS_RES_CASE(10)
        TS_RES_CASE(11)
        TS_RES_CASE(12)
        TS_RES_CASE(13)
    case 14:
        if (dtype == 1) return launch_res_n<float, 14>(a, nvec, s);
        break;
    default: break;
    }
#undef TS_RES_CASE
    return hipErrorInvalidValue;
}

hipError_t launch_resident_phases(int dtype, const ResidentPhaseArgs &a, int nchains, hipStream_t s)
{
    if (a.n < 1 || a.n > 14 || a.n_phases <= 0 || !a.phases || !a.tab || (nchains > 0) != (a.chains != nullptr))
        return hipErrorInvalidValue;
    const dim3 grid(a.n_phases, nchains > 0 ? nchains : 1);
    if (!resident_ascending(dtype)) {
        const int nt = resident_threads(a.n) > 16 ? resident_threads(a.n) : 16;
        hipLaunchKernelGGL(resident_phase_kernel, grid, dim3(nt), 0, s, a);
        return hipGetLastError();
    }
#define TS_RESD_CASE(TT)                                                                       \
    case TT:                                                                                   \
        hipLaunchKernelGGL((resident_diag_kernel<TT>), grid, dim3(kThreads), 0, s, a);         \
        return hipGetLastError();
    switch (a.n < 8 ? 8 : a.n) {
        TS_RESD_CASE(8)
        TS_RESD_CASE(9)
        TS_RESD_CASE(10)
        TS_RESD_CASE(11)
        TS_RESD_CASE(12)
        TS_RESD_CASE(13)
        TS_RESD_CASE(14)
    default: break;
    }
#undef TS_RESD_CASE
    return hipErrorInvalidValue;
}

hipError_t launch_resident_factors(int n, int n_phases, const double *tab, double *fac, hipStream_t s)
{
    if (n_phases <= 0 || !tab || !fac) return hipErrorInvalidValue;
#define TS_RESF_CASE(NN)                                                                              \
    case NN:                                                                                          \
        hipLaunchKernelGGL((resident_factor_kernel<NN>), dim3(n_phases), dim3(resident_threads(NN)), 0, s, tab, fac); \
        return hipGetLastError();
    switch (n) {
        TS_RESF_CASE(1)
        TS_RESF_CASE(2)
        TS_RESF_CASE(3)
        TS_RESF_CASE(4)
        TS_RESF_CASE(5)
        TS_RESF_CASE(6)
        TS_RESF_CASE(7)
        TS_RESF_CASE(8)
        TS_RESF_CASE(9)
        TS_RESF_CASE(10)
        TS_RESF_CASE(11)
        TS_RESF_CASE(12)
    default: break;
    }
#undef TS_RESF_CASE
    return hipErrorInvalidValue;
}

template <typename R>
static hipError_t launch_reduce_r(const ReduceArgs &a, double *partials, int nblocks, hipStream_t s)
{
    // accumulators live in registers: as few as the request needs
    if (a.n_obs <= 2)
        hipLaunchKernelGGL((reduce_kernel<R, 2>), dim3(nblocks), dim3(kThreads), 0, s, a, partials);
    else if (a.n_obs <= 8)
        hipLaunchKernelGGL((reduce_kernel<R, 8>), dim3(nblocks), dim3(kThreads), 0, s, a, partials);
    else
        hipLaunchKernelGGL((reduce_kernel<R, kMaxObs>), dim3(nblocks), dim3(kThreads), 0, s, a, partials);
    return hipGetLastError();
}

hipError_t launch_reduce(int dtype, const ReduceArgs &a, double *partials, int nblocks, hipStream_t s)
{
    if (a.n_obs < 1 || a.n_obs > kMaxObs) return hipErrorInvalidValue;
    return dtype == 0 ? launch_reduce_r<double>(a, partials, nblocks, s)
                      : launch_reduce_r<float>(a, partials, nblocks, s);
}

hipError_t launch_energy(int dtype, const void *psi, const EnergyPass &p, bool first, double *partials, int nblocks,
                         hipStream_t s)
{
    if (p.T < 1 || p.T > energy_tile_bits(dtype) || p.n_ops < 0 || !p.ops || nblocks < 1) return hipErrorInvalidValue;
    if (dtype == 0)
        hipLaunchKernelGGL((energy_kernel<double, energy_tile_bits(0)>), dim3(nblocks), dim3(kThreads), 0, s,
                           static_cast<const double2 *>(psi), p, (int)first, partials);
    else
        hipLaunchKernelGGL((energy_kernel<float, energy_tile_bits(1)>), dim3(nblocks), dim3(kThreads), 0, s,
                           static_cast<const float2 *>(psi), p, (int)first, partials);
    return hipGetLastError();
}

// The fixed scratch: one copy per GPU.  In host code `scratch` names a host-side stand-in,
// not device memory, so every host use goes through the address hipGetSymbolAddress returns.
static __device__ __align__(256) double scratch[kScratchDoubles];

hipError_t scratch_address(double **out)
{
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static double *addr[kMaxDevices] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        addr[dev] = static_cast<double *>(p);
    }
    *out = addr[dev];
    return hipSuccess;
}

hipError_t launch_sweep_etab(int dtype, int T, int RB, void *psi, const RegSweepArgs &a, hipStream_t s)
{
    if ((RB != 3 && RB != 4) || a.n_tiles == 0 || a.n_tiles > 0x7fffffffull || a.chains) return hipErrorInvalidValue;
#define TS_ETAB_CASE(TT, RR)                                                                      \
    if (T == TT && RB == RR) {                                                                    \
        if (dtype == 0)                                                                           \
            hipLaunchKernelGGL((sweep_etab_kernel<double, TT, RR>), dim3((uint32_t)a.n_tiles),     \
                               dim3(1 << (TT - RR)), 0, s, static_cast<double2 *>(psi), a);       \
        else                                                                                      \
            hipLaunchKernelGGL((sweep_etab_kernel<float, TT, RR>), dim3((uint32_t)a.n_tiles),      \
                               dim3(1 << (TT - RR)), 0, s, static_cast<float2 *>(psi), a);        \
        return hipGetLastError();                                                                 \
    }
    TS_ETAB_CASE(8, 4)
    TS_ETAB_CASE(9, 4)
    TS_ETAB_CASE(10, 4)
    TS_ETAB_CASE(11, 4)
    TS_ETAB_CASE(12, 4)
    TS_ETAB_CASE(13, 4)
    TS_ETAB_CASE(8, 3)
    TS_ETAB_CASE(9, 3)
    TS_ETAB_CASE(10, 3)
    TS_ETAB_CASE(11, 3)
    TS_ETAB_CASE(12, 3)
    TS_ETAB_CASE(13, 3)
#undef TS_ETAB_CASE
    return hipErrorInvalidValue;
}

hipError_t launch_energy_table(int dtype, void *out, int n, const double *h, const HamBond *bonds, int n_bonds,
                               int axis, hipStream_t s)
{
    if (!out || !h || (n_bonds > 0 && !bonds) || n < 1 || n > 40 || axis < 0 || axis > 2)
        return hipErrorInvalidValue;
    const uint64_t count = 1ull << n;
    const uint64_t blocks = std::min<uint64_t>((count + kThreads - 1) / kThreads, 1u << 16);
    if (dtype == 0)
        hipLaunchKernelGGL(energy_table_kernel<double>, dim3((uint32_t)blocks), dim3(kThreads), 0, s,
                           static_cast<double *>(out), n, h, bonds, n_bonds, axis, count);
    else
        hipLaunchKernelGGL(energy_table_kernel<float>, dim3((uint32_t)blocks), dim3(kThreads), 0, s,
                           static_cast<float *>(out), n, h, bonds, n_bonds, axis, count);
    return hipGetLastError();
}

hipError_t launch_sweep_pair(int dtype, int T, int RB, void *psi, void *lam, const RegSweepArgs &a,
                             const PairGradArgs &g, hipStream_t s)
{
    if (RB != 4 || a.n_tiles == 0 || a.n_tiles > 0x7fffffffull) return hipErrorInvalidValue;
#define TS_PAIR_CASE(TT)                                                                          \
    if (T == TT) {                                                                                \
        if (dtype == 0)                                                                           \
            hipLaunchKernelGGL((sweep_pair_kernel<double, TT, 4>), dim3((uint32_t)a.n_tiles),      \
                               dim3(1 << (TT - 4)), 0, s, static_cast<double2 *>(psi),             \
                               static_cast<double2 *>(lam), a, g);                                \
        else                                                                                      \
            hipLaunchKernelGGL((sweep_pair_kernel<float, TT, 4>), dim3((uint32_t)a.n_tiles),       \
                               dim3(1 << (TT - 4)), 0, s, static_cast<float2 *>(psi),              \
                               static_cast<float2 *>(lam), a, g);                                 \
        return hipGetLastError();                                                                 \
    }
    TS_PAIR_CASE(8)
    TS_PAIR_CASE(9)
    TS_PAIR_CASE(10)
    TS_PAIR_CASE(11)
    TS_PAIR_CASE(12)
#undef TS_PAIR_CASE
    return hipErrorInvalidValue;
}

template <typename R, int T, int KIND>
static hipError_t launch_cone_k(typename Vec<R>::T *psi, const ConeArgs *a, uint64_t n_tiles, int reverse,
                                const ConeRec *rec, hipStream_t s)
{
    const dim3 grid((uint32_t)n_tiles), block(1 << (T - 4));
    if (rec)
        hipLaunchKernelGGL((cone_rec_kernel<R, T, 4, KIND>), grid, block, 0, s, psi, a, n_tiles, reverse, *rec);
    else
        hipLaunchKernelGGL((cone_kernel<R, T, 4, KIND>), grid, block, 0, s, psi, a, n_tiles, reverse);
    return hipGetLastError();
}

template <typename R, int T>
static hipError_t launch_cone_t(typename Vec<R>::T *psi, const ConeArgs *a, uint64_t n_tiles, int reverse,
                                const ConeRec *rec, hipStream_t s, uint64_t few_tiles)
{
    if (n_tiles <= few_tiles) return launch_cone_k<R, T, kConeFew>(psi, a, n_tiles, reverse, rec, s);
    if constexpr (sizeof(R) == 8)
        if (n_tiles <= kConeMidTiles) return launch_cone_k<R, T, kConeMid>(psi, a, n_tiles, reverse, rec, s);
    return launch_cone_k<R, T, kConeMany>(psi, a, n_tiles, reverse, rec, s);
}

static hipError_t launch_cone_any(int dtype, int T, int RB, void *psi, const ConeArgs *a, int n_phases,
                                  uint64_t n_tiles, int reverse, const ConeRec *rec, hipStream_t s,
                                  uint64_t few_tiles = kConeFewTiles)
{
    if (!a || RB != 4 || n_phases < 0 || n_phases > kConePhases || n_tiles == 0 || n_tiles > 0x7fffffffull)
        return hipErrorInvalidValue;
#define TS_CONE_CASE(TT)                                                                              \
    if (T == TT)                                                                                      \
        return dtype == 0 ? launch_cone_t<double, TT>(static_cast<double2 *>(psi), a, n_tiles, reverse, rec, s, few_tiles) \
                          : launch_cone_t<float, TT>(static_cast<float2 *>(psi), a, n_tiles, reverse, rec, s, few_tiles);
    TS_CONE_CASE(11)
    TS_CONE_CASE(12)
#undef TS_CONE_CASE
    return hipErrorInvalidValue;
}

hipError_t launch_cone(int dtype, int T, int RB, void *psi, const ConeArgs *a, int n_phases,
                       uint64_t n_tiles, int reverse, hipStream_t s, uint64_t few_tiles)
{
    return launch_cone_any(dtype, T, RB, psi, a, n_phases, n_tiles, reverse, nullptr, s, few_tiles);
}

hipError_t launch_cone_rec(int dtype, int T, int RB, void *psi, const ConeArgs *a, int n_phases,
                           uint64_t n_tiles, int reverse, const ConeRec &rec, hipStream_t s)
{
    if (!rec.partials || rec.n_obs < 0 || rec.n_obs > kConeRecMax) return hipErrorInvalidValue;
    return launch_cone_any(dtype, T, RB, psi, a, n_phases, n_tiles, reverse, &rec, s);
}

hipError_t launch_cone_pair(int dtype, int T, int RB, void *psi, void *lam, const ConeArgs *a, int n_phases,
                            const ConeGradArgs *g, int n_slots, double *slots, int stride, uint64_t n_tiles,
                            int reverse, hipStream_t s)
{
    if (!a || !g || !slots || RB != 4 || n_phases < 0 || n_phases > kConePhases || n_slots < 0 ||
        n_slots > kConeGradSlots || n_tiles == 0 || n_tiles > 0x7fffffffull)
        return hipErrorInvalidValue;
#define TS_CONEP_CASE(TT)                                                                         \
    if (T == TT) {                                                                                \
        const size_t dyn = cone_tab_bytes<TT, 4>(n_phases) + (size_t)n_slots * 64 * sizeof(double); \
        if (dtype == 0)                                                                           \
            hipLaunchKernelGGL((cone_pair_c128_kernel<TT, 4>), dim3((uint32_t)n_tiles),            \
                               dim3(1 << (TT - 4)), dyn, s, static_cast<double2 *>(psi),           \
                               static_cast<double2 *>(lam), a, g, slots, stride, n_tiles, reverse); \
        else                                                                                      \
            hipLaunchKernelGGL((cone_pair_c64_kernel<TT, 4>), dim3((uint32_t)n_tiles),             \
                               dim3(1 << (TT - 4)), dyn, s, static_cast<float2 *>(psi),            \
                               static_cast<float2 *>(lam), a, g, slots, stride, n_tiles, reverse); \
        return hipGetLastError();                                                                 \
    }
    TS_CONEP_CASE(11)
    TS_CONEP_CASE(12)
#undef TS_CONEP_CASE
    return hipErrorInvalidValue;
}

// First pass of a long finalize: workgroup g sums rows [g * 1024, (g + 1) * 1024) of every
// used column into row g of tmp (a fixed order: per thread, then a wave and an LDS tree).
__global__ __launch_bounds__(kThreads) void partial_rows_kernel(const double *partials, int nrows,
                                                                int ncols, double *tmp)
{
    __shared__ double red[kThreads / 64];
    const int r0 = blockIdx.x * 1024, r1 = min(nrows, r0 + 1024);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    for (int c = 0; c < ncols; ++c) {
        double acc = 0.0;
        for (int r = r0 + (int)threadIdx.x; r < r1; r += kThreads) acc += partials[(size_t)r * (2 * kMaxObs) + c];
        acc = wave_sum(acc);
        if (lane == 0) red[wv] = acc;
        __syncthreads();
        if (threadIdx.x == 0) {
            double sum = 0.0;
            for (int w = 0; w < kThreads / 64; ++w) sum += red[w];
            tmp[(size_t)blockIdx.x * (2 * kMaxObs) + c] = sum;
        }
        __syncthreads();
    }
}

hipError_t launch_finalize(const double *partials, int nblocks, const ReduceArgs &a, double *out,
                           double *tmp, hipStream_t s)
{
    if (nblocks > 1024) {
        const int groups = (nblocks + 1023) / 1024;
        if (groups > 1024 || !tmp) return hipErrorInvalidValue;
        hipLaunchKernelGGL(partial_rows_kernel, dim3(groups), dim3(kThreads), 0, s, partials, nblocks,
                           2 * a.n_obs, tmp);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        partials = tmp;
        nblocks = groups;
    }
    hipLaunchKernelGGL(finalize_kernel, dim3(2 * a.n_obs), dim3(64), 0, s, partials, nblocks, a, out);
    return hipGetLastError();
}

hipError_t launch_cone_batch(int dtype, int T, int RB, void *packed, const int64_t *off,
                             const ConeArgs *args, uint32_t nchains, uint64_t tiles_per_chain, int reverse,
                             hipStream_t s)
{
    const uint64_t grid = (uint64_t)nchains * tiles_per_chain;
    if (!packed || !off || !args || RB != 4 || grid == 0 || grid > 0x7fffffffull) return hipErrorInvalidValue;
#define TS_CONEB_CASE(TT)                                                                         \
    if (T == TT) {                                                                                \
        if (dtype == 0)                                                                           \
            hipLaunchKernelGGL((cone_batch_kernel<double, TT, 4>), dim3((uint32_t)grid),           \
                               dim3(1 << (TT - 4)), 0, s,                                         \
                               static_cast<double2 *>(packed), off, args, tiles_per_chain, reverse); \
        else                                                                                      \
            hipLaunchKernelGGL((cone_batch_kernel<float, TT, 4>), dim3((uint32_t)grid),            \
                               dim3(1 << (TT - 4)), 0, s,                                         \
                               static_cast<float2 *>(packed), off, args, tiles_per_chain, reverse); \
        return hipGetLastError();                                                                 \
    }
    TS_CONEB_CASE(11)
    TS_CONEB_CASE(12)
#undef TS_CONEB_CASE
    return hipErrorInvalidValue;
}

}  // namespace tsk
