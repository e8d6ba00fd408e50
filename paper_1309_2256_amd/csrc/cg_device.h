// Device parts of the CG scalar updates and the search-direction update,
// shared by the stand-alone kernels (blas.hip) and the persistent batch
// kernel (dslash.hip) so that both perform the same operations in the same
// order: a right-hand side solved in a batch follows its single solve bit
// for bit.  Every function here is called by all threads of a 256-thread
// block (the sums use the block's LDS and barriers).
//
// The block partial sums and the CG scalars are small arrays that blocks on
// different XCDs write within one launch of the persistent kernel (several
// writers share a cache line).  They are read and written with device-scope
// atomic loads and stores, which do not depend on the state of a
// non-coherent L2 copy of the line; the data fields themselves are never
// shared between writers at line granularity.
#pragma once

#include "tm_internal.h"

namespace cgdev {

constexpr int kThreads = 256;

template <typename V>
__device__ __forceinline__ V ld_coh(const V *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename V>
__device__ __forceinline__ void st_coh(V *p, V v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// v + (v of the lane that DPP control CTRL names), in the rows of 16 lanes of
// the mask ROWS; + 0 where that lane is outside the row
template <int CTRL, int ROWS>
__device__ __forceinline__ double add_dpp(double v)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROWS, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROWS, 0xf, false);
    return v + __hiloint2double(hi, lo);
}

// sum over the wave (all 64 lanes active), in every lane.  On the VALU: prefix
// sums in rows of 16, then across the rows.  Twelve exchanges through the LDS
// crossbar (__shfl_down) are a chain of about 1000 cycles; with the scalars of
// finish_alpha / finish_beta loaded ahead of their sums, a mixed solve of one
// right-hand side on 16^3 x 32 takes 4% less time.
__device__ __forceinline__ double wave_sum(double v)
{
    v = add_dpp<0x111, 0xf>(v);  // row_shr:1
    v = add_dpp<0x112, 0xf>(v);  // row_shr:2
    v = add_dpp<0x114, 0xf>(v);  // row_shr:4
    v = add_dpp<0x118, 0xf>(v);  // row_shr:8
    v = add_dpp<0x142, 0xa>(v);  // row_bcast:15
    v = add_dpp<0x143, 0xc>(v);  // row_bcast:31
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), 63),
                            __builtin_amdgcn_readlane(__double2loint(v), 63));
}

// sum over the block; result valid in thread 0
__device__ __forceinline__ double block_sum(double v)
{
    __shared__ double red[kThreads / 64];
    v = wave_sum(v);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (lane == 0) red[w] = v;
    __syncthreads();
    double s = 0;
    if (threadIdx.x == 0) {
#pragma unroll
        for (int k = 0; k < kThreads / 64; k++) s += red[k];
    }
    __syncthreads();
    return s;
}

// sum_b part[idx * nblk + b]: thread-strided partial sums, then the block
// tree; result valid in thread 0
__device__ __forceinline__ double sum_partials(const double *part, int nblk, int idx)
{
    const double *p = part + (size_t)idx * nblk;
    double acc = 0;
    int b = threadIdx.x;
    // eight loads in flight: one at a time, 64 of them (32^3 x 64) would each
    // wait for the memory latency
    for (; b + 7 * kThreads < nblk; b += 8 * kThreads) {
        double v[8];
#pragma unroll
        for (int k = 0; k < 8; k++) v[k] = ld_coh(p + b + k * kThreads);
#pragma unroll
        for (int k = 0; k < 8; k++) acc += v[k];
    }
    for (; b < nblk; b += kThreads) acc += ld_coh(p + b);
    return block_sum(acc);
}

__device__ __forceinline__ bool finite(double v) { return v == v && v - v == 0; }

// alpha = |r|^2 / |q|^2 of right-hand side r, also kept for ring position pos;
// part layout [rhs][nblk]
__device__ __forceinline__ void finish_alpha(CGScalars *sc, const double *part, int nblk, int pos, int r)
{
    // the scalars' loads overlap those of the sum
    CGScalars &s = sc[r];
    const double rr = ld_coh(&s.rr);
    const int active = ld_coh(&s.active);
    const double qq = sum_partials(part, nblk, r);
    if (threadIdx.x == 0) {
        st_coh(&s.qq, qq);
        if (!finite(qq) || !finite(rr)) st_coh(&s.bad, 1);
        const double alpha = (active && qq > 0 && finite(qq)) ? rr / qq : 0.0;
        st_coh(&s.alpha, alpha);
        st_coh(&s.hist[pos], alpha);
    }
}

// beta, the new |r|^2 and |rho|^2 and the convergence / reliable-update
// flags of right-hand side r.  part layout: [slot 0: |r|^2 for all rhs]
// [slot 1: |rho|^2 for all rhs].  With reliable updates (delta > 0) slot 1
// is not used: the Schur residual rho -= alpha q has
// |rho'|^2 = |rho|^2 - 2 alpha <r, p> + alpha^2 |q|^2 = |rho|^2 - alpha |r|^2
// (CG: <r, p> = |r|^2, alpha = |r|^2 / |q|^2), a recurrence whose rounding
// stays far below the delta^2 |rho_ref|^2 it is compared with between two
// updates (each update resets it to the FP64 true residual).
__device__ __forceinline__ void finish_beta(CGScalars *sc, const double *part, int nblk, int nrhs, double delta,
                                            int r)
{
    CGScalars &s = sc[r];
    const int active = ld_coh(&s.active), iters = ld_coh(&s.iters);
    const double rr_old = ld_coh(&s.rr), rho2_old = ld_coh(&s.rho2), target2 = ld_coh(&s.target2);
    const double alpha = ld_coh(&s.alpha), rho2_ref = ld_coh(&s.rho2_ref);
    const double rr = sum_partials(part, nblk, r);
    double rho2 = delta > 0 ? 0.0 : sum_partials(part, nblk, nrhs + r);
    if (threadIdx.x == 0) {
        if (delta > 0) rho2 = active ? fmax(rho2_old - alpha * rr_old, 0.0) : rho2_old;
        if (!finite(rr) || !finite(rho2)) st_coh(&s.bad, 1);
        if (active) {
            st_coh(&s.beta, (rr_old > 0) ? rr / rr_old : 0.0);
            st_coh(&s.rr, rr);
            st_coh(&s.rho2, rho2);
            st_coh(&s.iters, iters + 1);
            if (delta > 0) {
                // reliable-update solver: converged estimate or residual fallen
                // by delta since the last update -> request an update
                if (rho2 <= target2 || rho2 < delta * delta * rho2_ref) st_coh(&s.want_update, 1);
            } else if (rho2 <= target2) {
                st_coh(&s.active, 0);
            }
        } else {
            st_coh(&s.beta, 0.0);
        }
    }
}

// what finish_beta will leave: whether right-hand side r iterates on, and beta;
// in every thread
struct NextBeta {
    bool active;
    double beta;
};
__device__ __forceinline__ NextBeta next_beta(const CGScalars *sc, const double *part, int nblk, int nrhs, double delta,
                                              int r)
{
    __shared__ NextBeta next;
    const CGScalars &s = sc[r];
    const int active = ld_coh(&s.active);
    const double rr_old = ld_coh(&s.rr), target2 = ld_coh(&s.target2);
    const double rr = sum_partials(part, nblk, r);
    const double rho2 = delta > 0 ? 0.0 : sum_partials(part, nblk, nrhs + r);
    if (threadIdx.x == 0) {
        next.active = active && (delta > 0 || !(rho2 <= target2));
        next.beta = active && rr_old > 0 ? rr / rr_old : 0.0;
    }
    __syncthreads();
    return next;
}
__device__ __forceinline__ NextBeta stored_beta(const CGScalars *sc, int r)
{
    return {ld_coh(&sc[r].active) != 0, ld_coh(&sc[r].beta)};
}

// The vector updates of one iteration for elements e0, e0 + step, ... < e1 of
// right-hand side r (n complex per right-hand side).  Elementwise: any split of
// the range gives the same result.

// pout = rv + beta pin (the solution follows at the end of the ring)
template <typename S>
__device__ __forceinline__ void update_p(S *pout, const S *pin, const S *rv, size_t n, NextBeta nb, int r, size_t e0,
                                         size_t e1, size_t step)
{
    using T = typename StoreTraits<S>::real;
    if (!nb.active) return;
    const T b = (T)nb.beta;
    const size_t base = (size_t)r * n;
    for (size_t e = e0; e < e1; e += step) {
        const cx<T> pv = ldT<T>(pin, base + e);
        stT<T>(pout, base + e, ldT<T>(rv, base + e) + b * pv);
    }
}

// x += hist[0] p[0] + ... + hist[M - 1] p[M - 1], one after the other; then
// p[0] = rv + beta p[M - 1], or the last direction that moved x if the
// right-hand side is no longer active.  ring: its M buffers (S *const *).
template <int M, typename S, typename XS, typename R>
__device__ __forceinline__ void update_px(const R &ring, const S *rv, XS *x, size_t n, const CGScalars *sc, NextBeta nb,
                                          int r, size_t e0, size_t e1, size_t step)
{
    using T = typename StoreTraits<S>::real;
    using TX = typename StoreTraits<XS>::real;
    const bool active = nb.active;
    double h[M];
    bool any = active;
    int last = 0;
#pragma unroll
    for (int q = 0; q < M; q++) {
        h[q] = ld_coh(&sc[r].hist[q]);
        if (h[q] != 0.0) any = true, last = q;
    }
    if (!any) return;
    const T b = active ? (T)nb.beta : (T)0;
    const size_t base = (size_t)r * n;
    for (size_t e = e0; e < e1; e += step) {
        const size_t k = base + e;
        cx<T> pv[M];
#pragma unroll
        for (int q = 0; q < M; q++) pv[q] = ldT<T>((const S *)ring[q], k);
        cx<TX> xv = ldT<TX>(x, k);
        cx<T> pn = active ? ldT<T>(rv, k) + b * pv[M - 1] : pv[0];
#pragma unroll
        for (int q = 0; q < M; q++) {
            if (active || h[q] != 0.0) xv = xv + (TX)h[q] * cx<TX>{(TX)pv[q].r, (TX)pv[q].i};
            if (!active && q == last) pn = pv[q];
        }
        stT<TX>(x, k, xv);
        if (active || last > 0) stT<T>((S *)ring[0], k, pn);
    }
}

// an incomplete round of cnt directions: x as above, p[cnt] the current
// direction of a right-hand side that is no longer active
template <typename S, typename XS, typename R>
__device__ __forceinline__ void flush_x(const R &ring, int cnt, XS *x, size_t n, const CGScalars *sc, int r,
                                        size_t e0, size_t e1, size_t step)
{
    using T = typename StoreTraits<S>::real;
    using TX = typename StoreTraits<XS>::real;
    const bool active = ld_coh(&sc[r].active) != 0;
    int last = 0;
    for (int q = 0; q < cnt; q++)
        if (ld_coh(&sc[r].hist[q]) != 0.0) last = q;
    const size_t base = (size_t)r * n;
    for (size_t e = e0; e < e1; e += step) {
        const size_t k = base + e;
        cx<TX> xv = ldT<TX>(x, k);
        for (int q = 0; q < cnt; q++) {
            const double h = ld_coh(&sc[r].hist[q]);
            const cx<T> pv = ldT<T>((const S *)ring[q], k);
            if (active || h != 0.0) xv = xv + (TX)h * cx<TX>{(TX)pv.r, (TX)pv.i};
            if (!active && q == last) stT<T>((S *)ring[cnt], k, pv);
        }
        stT<TX>(x, k, xv);
    }
}

}  // namespace cgdev
