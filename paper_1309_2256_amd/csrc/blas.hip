// Vector kernels of the solvers: spin-diagonal scaling, precision conversion,
// axpy forms and per-right-hand-side norms.  Reductions are deterministic:
// each block writes one FP64 partial per right-hand side (fixed grid, fixed
// wave-then-LDS tree) and a single block per right-hand side sums the
// partials in a fixed order.  Products are formed in the arithmetic precision
// and accumulated in FP64.
#include "cg_device.h"

namespace {

constexpr int kBlock = 256;
constexpr int kMaxPart = 1024;

using cgdev::block_sum;
using cgdev::sum_partials;
static_assert(kBlock == cgdev::kThreads, "block sums assume 256 threads");

template <typename S>
__global__ __launch_bounds__(kBlock) void k_spin_diag(S *out, const S *in, int hs, cx<float> fu,
                                                      cx<float> fl, cx<double> du, cx<double> dl)
{
    using T = typename StoreTraits<S>::real;
    const size_t n = (size_t)12 * hs;
    const size_t base = (size_t)blockIdx.y * n;
    for (size_t e = (size_t)blockIdx.x * kBlock + threadIdx.x; e < n; e += (size_t)gridDim.x * kBlock) {
        const int k = (int)(e / hs);
        cx<T> f;
        if (sizeof(T) == 8) {
            cx<double> d = k < 6 ? du : dl;
            f = {(T)d.r, (T)d.i};
        } else {
            cx<float> d = k < 6 ? fu : fl;
            f = {(T)d.r, (T)d.i};
        }
        stT<T>(out, base + e, f * ldT<T>(in, base + e));
    }
}

template <typename SO, typename SI>
__global__ __launch_bounds__(kBlock) void k_convert(SO *out, const SI *in, size_t n, const double *scale)
{
    const size_t base = (size_t)blockIdx.y * n;
    const double sc = scale ? scale[blockIdx.y] : 1.0;
    for (size_t e = (size_t)blockIdx.x * kBlock + threadIdx.x; e < n; e += (size_t)gridDim.x * kBlock) {
        cx<double> v = ldT<double>(in, base + e);
        stT<double>(out, base + e, sc * v);
    }
}

template <typename S>
__global__ __launch_bounds__(kBlock) void k_axpby(S *y, const S *x, size_t n, double a, double b)
{
    using T = typename StoreTraits<S>::real;
    for (size_t e = (size_t)blockIdx.x * kBlock + threadIdx.x; e < n; e += (size_t)gridDim.x * kBlock) {
        cx<T> xv = ldT<T>(x, e), yv = ldT<T>(y, e);
        stT<T>(y, e, (T)a * xv + (T)b * yv);
    }
}

template <typename S>
__global__ __launch_bounds__(kBlock) void k_zero(S *y, size_t n)
{
    for (size_t e = (size_t)blockIdx.x * kBlock + threadIdx.x; e < n; e += (size_t)gridDim.x * kBlock)
        stT<double>(y, e, cx<double>{0.0, 0.0});
}

// y[r] += a[r] * x[r] with per-rhs device scalars (x may be a lower precision)
template <typename SY, typename SX>
__global__ __launch_bounds__(kBlock) void k_axpy_dev(SY *y, const SX *x, size_t n, const double *a)
{
    using T = typename StoreTraits<SY>::real;
    const size_t base = (size_t)blockIdx.y * n;
    const T av = (T)a[blockIdx.y];
    for (size_t e = (size_t)blockIdx.x * kBlock + threadIdx.x; e < n; e += (size_t)gridDim.x * kBlock) {
        const size_t k = base + e;
        stT<T>(y, k, ldT<T>(y, k) + av * ldT<T>(x, k));
    }
}

// partial |v|^2 of right-hand side blockIdx.y over the vh valid sites of
// each of its 12 planes (the pad sites of a plane are skipped)
template <typename S>
__global__ __launch_bounds__(kBlock) void k_partial_norm2(const S *v, int vh, int hs, double *part, int nblk)
{
    using T = typename StoreTraits<S>::real;
    const size_t base = (size_t)blockIdx.y * 12 * hs;
    double acc = 0;
    for (int k = 0; k < 12; k++)
        for (int i = blockIdx.x * kBlock + threadIdx.x; i < vh; i += gridDim.x * kBlock) {
            cx<T> a = ldT<T>(v, base + (size_t)k * hs + i);
            acc += (double)(a.r * a.r + a.i * a.i);
        }
    double s = block_sum(acc);
    if (threadIdx.x == 0) part[(size_t)blockIdx.y * nblk + blockIdx.x] = s;
}

// out = scale in (converted; pads too) and the partial |out|^2 of the values as
// stored, in one pass; out = null: the norm only.  Bound: memory.  A reliable
// update made ten passes over the FP64 and FP16 fields beside its hops; with
// these and the residual form of the hop kernel six are left: 32^3 x 64, 12
// right-hand sides, 11.1 -> 8.9 ms an update.
template <typename SO, typename SI>
__global__ __launch_bounds__(kBlock) void k_convert_norm(SO *out, const SI *in, int vh, int hs, const double *scale,
                                                         double *part)
{
    using T = typename StoreTraits<SO>::real;
    const size_t base = (size_t)blockIdx.y * 12 * hs;
    const double sc = scale[blockIdx.y];
    double acc = 0;
#pragma unroll 4
    for (int k = 0; k < 12; k++)
        for (int i = blockIdx.x * kBlock + threadIdx.x; i < hs; i += gridDim.x * kBlock) {
            const size_t e = base + (size_t)k * hs + i;
            const cx<double> v = sc * ldT<double>(in, e);
            SO st;
            stT<double>(&st, 0, v);
            if (out) out[e] = st;
            const cx<T> a = ldT<T>(&st, 0);
            if (i < vh) acc += (double)(a.r * a.r + a.i * a.i);
        }
    const double s = block_sum(acc);
    if (threadIdx.x == 0) part[(size_t)blockIdx.y * gridDim.x + blockIdx.x] = s;
}

__global__ __launch_bounds__(kBlock) void k_finish_sum(const double *part, int nblk, double *out)
{
    double s = sum_partials(part, nblk, blockIdx.x);
    if (threadIdx.x == 0) out[blockIdx.x] = s;
}

// part layout: [slot 0: |r|^2 for all rhs][slot 1: |rho|^2 for all rhs]
__global__ __launch_bounds__(kBlock) void k_finish_beta(CGScalars *sc, const double *part, int nblk,
                                                        int nrhs, double delta)
{
    cgdev::finish_beta(sc, part, nblk, nrhs, delta, blockIdx.x);
}

struct RingArg {
    void *p[kCgRing];
    __device__ void *operator[](int q) const { return p[q]; }
};

// M = 0: position pos before the last of the ring; else its end, M directions.
// BETA: beta from the partial sums in every block instead of from a launch of
// its own (see cg_beta_late).
template <int M, bool BETA, typename S, typename XS>
__global__ __launch_bounds__(kBlock) void k_update(const RingArg ring, int pos, const S *rv, XS *x, size_t n,
                                                   const CGScalars *sc, const double *part, int nblk, int nrhs,
                                                   double delta)
{
    const int r = blockIdx.y;
    const cgdev::NextBeta nb = BETA ? cgdev::next_beta(sc, part, nblk, nrhs, delta, r) : cgdev::stored_beta(sc, r);
    const size_t e0 = (size_t)blockIdx.x * kBlock + threadIdx.x, step = (size_t)gridDim.x * kBlock;
    if constexpr (M == 0)
        cgdev::update_p((S *)ring[pos + 1], (const S *)ring[pos], rv, n, nb, r, e0, n, step);
    else
        cgdev::update_px<M, S>(ring, rv, x, n, sc, nb, r, e0, n, step);
}

template <typename S, typename XS>
__global__ __launch_bounds__(kBlock) void k_flush_x(const RingArg ring, int cnt, XS *x, size_t n, const CGScalars *sc)
{
    cgdev::flush_x<S>(ring, cnt, x, n, sc, blockIdx.y, (size_t)blockIdx.x * kBlock + threadIdx.x, n,
                      (size_t)gridDim.x * kBlock);
}

// Several lattices per launch (a batch iteration).  Scalar kernel: block b
// is right-hand side b - rstart[i] of lattice i.  Update: lattice i owns
// blocks [ustart[i], ustart[i+1]) laid out as its single launch's
// (gx[i] x nrhs) grid, so every element sees the same thread-stride loop.
constexpr int kTailInst = 8;
template <typename S, typename XS>
struct TailArgs {
    CGScalars *sc[kTailInst];
    const double *part[kTailInst];
    RingArg ring[kTailInst];
    const S *r[kTailInst];
    XS *x[kTailInst];
    size_t n[kTailInst];
    double delta[kTailInst];
    int nblk[kTailInst], nrhs[kTailInst], gx[kTailInst];
    int rstart[kTailInst + 1], ustart[kTailInst + 1];
    int ninst, pos;
};
static_assert(sizeof(TailArgs<double2, double2>) <= 4096, "kernel arguments exceed 4 KiB");

__device__ __forceinline__ int tail_inst(const int *start, int n, int b)
{
    int i = 0;
    while (i + 1 < n && b >= start[i + 1]) i++;
    return i;
}

template <typename S, typename XS>
__global__ __launch_bounds__(kBlock) void k_finish_beta_multi(const TailArgs<S, XS> a)
{
    const int i = tail_inst(a.rstart, a.ninst, blockIdx.x);
    cgdev::finish_beta(a.sc[i], a.part[i], a.nblk[i], a.nrhs[i], a.delta[i], blockIdx.x - a.rstart[i]);
}

// M = 0: a position before the last of the ring
template <int M, typename S, typename XS>
__global__ __launch_bounds__(kBlock) void k_update_multi(const TailArgs<S, XS> a)
{
    const int i = tail_inst(a.ustart, a.ninst, blockIdx.x);
    const int local = blockIdx.x - a.ustart[i], gx = a.gx[i];
    const int r = local / gx, bx = local - r * gx;
    const size_t e0 = (size_t)bx * kBlock + threadIdx.x, step = (size_t)gx * kBlock;
    if constexpr (M == 0)
        cgdev::update_p((S *)a.ring[i][a.pos + 1], (const S *)a.ring[i][a.pos], a.r[i], a.n[i],
                        cgdev::stored_beta(a.sc[i], r), r, e0, a.n[i], step);
    else
        cgdev::update_px<M, S>(a.ring[i], a.r[i], a.x[i], a.n[i], a.sc[i], cgdev::stored_beta(a.sc[i], r), r, e0, a.n[i],
                               step);
}

// complex elements of one right-hand side of a half field, pads included
size_t half_elems(tm_ctx *c) { return (size_t)12 * c->geo.hs; }

int grid_for(size_t n)
{
    size_t g = (n + kBlock * 4 - 1) / (kBlock * 4);
    if (g < 1) g = 1;
    if (g > 4096) g = 4096;
    return (int)g;
}

template <typename F>
void dispatch_prec(int prec, F &&f)
{
    switch (prec) {
    case TM_F64: f((double2 *)nullptr); break;
    case TM_F32: f((float2 *)nullptr); break;
    case TM_F16: f((h2 *)nullptr); break;
    case TM_BF16: f((b2 *)nullptr); break;
    default: throw TmError{TM_ERR_ARG, "bad precision"};
    }
}

}  // namespace

void launch_spin_diag(tm_ctx *c, void *out, const void *in, int prec, int nrhs, SpinDiag d, hipStream_t s)
{
    size_t n = half_elems(c);
    dim3 grid(grid_for(n), nrhs);
    cx<float> fu{(float)d.u.r, (float)d.u.i}, fl{(float)d.l.r, (float)d.l.i};
    account(c, 2.0 * n * nrhs * prec_bytes(prec), 6.0 * n * nrhs);
    dispatch_prec(prec, [&](auto *tag) {
        using S = std::remove_pointer_t<decltype(tag)>;
        hipLaunchKernelGGL(k_spin_diag<S>, grid, dim3(kBlock), 0, s, (S *)out, (const S *)in, c->geo.hs, fu,
                           fl, d.u, d.l);
    });
    TM_HIP(hipGetLastError());
}

void launch_copy_convert(tm_ctx *c, void *out, int out_prec, const void *in, int in_prec, int nrhs,
                         const double *dscale, hipStream_t s)
{
    size_t n = half_elems(c);
    dim3 grid(grid_for(n), nrhs);
    account(c, (double)n * nrhs * (prec_bytes(in_prec) + prec_bytes(out_prec)), dscale ? 2.0 * n * nrhs : 0.0);
    dispatch_prec(out_prec, [&](auto *to) {
        using SO = std::remove_pointer_t<decltype(to)>;
        dispatch_prec(in_prec, [&](auto *ti) {
            using SI = std::remove_pointer_t<decltype(ti)>;
            hipLaunchKernelGGL((k_convert<SO, SI>), grid, dim3(kBlock), 0, s, (SO *)out, (const SI *)in, n,
                               dscale);
        });
    });
    TM_HIP(hipGetLastError());
}

void launch_axpby_host(tm_ctx *c, void *y, const void *x, int prec, int nrhs, double a, double b,
                       hipStream_t s)
{
    size_t n = half_elems(c) * nrhs;
    account(c, 3.0 * n * prec_bytes(prec), 6.0 * n);
    dispatch_prec(prec, [&](auto *tag) {
        using S = std::remove_pointer_t<decltype(tag)>;
        hipLaunchKernelGGL(k_axpby<S>, dim3(grid_for(n)), dim3(kBlock), 0, s, (S *)y, (const S *)x, n, a, b);
    });
    TM_HIP(hipGetLastError());
}

template <typename S, typename XS>
static TailArgs<S, XS> tail_args(const std::vector<CgTail> &t, size_t i0, size_t i1, int pos)
{
    TailArgs<S, XS> a{};
    a.pos = pos;
    a.ninst = (int)(i1 - i0);
    a.rstart[0] = a.ustart[0] = 0;
    for (size_t k = i0; k < i1; k++) {
        const int j = (int)(k - i0);
        const CgTail &q = t[k];
        a.sc[j] = q.sc;
        a.part[j] = q.partb;
        std::copy(q.ring.p, q.ring.p + kCgRing, a.ring[j].p);
        a.r[j] = (const S *)q.r;
        a.x[j] = (XS *)q.x;
        a.n[j] = half_elems(q.c);
        a.delta[j] = q.delta;
        a.nblk[j] = q.nblk;
        a.nrhs[j] = q.nrhs;
        a.gx[j] = grid_for(a.n[j]);
        a.rstart[j + 1] = a.rstart[j] + q.nrhs;
        a.ustart[j + 1] = a.ustart[j] + a.gx[j] * q.nrhs;
    }
    return a;
}

template <typename F>
static void dispatch_tail(int prec, int xprec, F &&f)
{
    if (prec == TM_F64) {
        TM_REQUIRE(xprec == TM_F64, "FP64 CG needs an FP64 solution vector");
        f((double2 *)nullptr, (double2 *)nullptr);
        return;
    }
    TM_REQUIRE(xprec == TM_F32, "low-precision CG accumulates in FP32");
    dispatch_prec(prec, [&](auto *tag) { f(tag, (float2 *)nullptr); });
}

// the kernel form of a ring position: 0 before the last one, else the ring's
// length (FP64 solves update x in every iteration)
template <typename S, typename F>
static void ring_form(int m, int pos, F &&f)
{
    if constexpr (!std::is_same<S, double2>::value) {
        if (pos < m - 1) return f(std::integral_constant<int, 0>{});
        if (m == 8) return f(std::integral_constant<int, 8>{});
        if (m == 4) return f(std::integral_constant<int, 4>{});
        if (m == 2) return f(std::integral_constant<int, 2>{});
    }
    TM_REQUIRE(m == 1, "bad ring of search directions");
    f(std::integral_constant<int, 1>{});
}

void cg_tail_multi(const std::vector<CgTail> &t, int pos, int prec, int xprec, hipStream_t s)
{
    for (size_t i0 = 0; i0 < t.size(); i0 += kTailInst) {
        const size_t i1 = std::min(t.size(), i0 + kTailInst);
        dispatch_tail(prec, xprec, [&](auto *ts, auto *tx) {
            using S = std::remove_pointer_t<decltype(ts)>;
            using XS = std::remove_pointer_t<decltype(tx)>;
            const TailArgs<S, XS> a = tail_args<S, XS>(t, i0, i1, pos);
            hipLaunchKernelGGL((k_finish_beta_multi<S, XS>), dim3(a.rstart[a.ninst]), dim3(kBlock), 0, s, a);
            TM_HIP(hipGetLastError());
            auto go = [&](auto m) {
                hipLaunchKernelGGL((k_update_multi<m(), S, XS>), dim3(a.ustart[a.ninst]), dim3(kBlock), 0, s, a);
            };
            ring_form<S>(t[i0].ring.m, pos, go);
            TM_HIP(hipGetLastError());
        });
        for (size_t k = i0; k < i1; k++) {
            double b, f;
            cg_update_cost(t[k].ring, pos, prec, xprec, b, f);
            const double n = (double)half_elems(t[k].c) * t[k].nrhs;
            account(t[k].c, n * b, n * f);
        }
    }
}

// partial-sum blocks of the vector norms (a few per CU, at most kMaxPart)
int norm_blocks(tm_ctx *c)
{
    // one site per thread: its 12 planes, 12 elements
    size_t n = c->geo.vh;
    size_t g = (n + kBlock - 1) / kBlock;
    if (g < 1) g = 1;
    if (g > kMaxPart) g = kMaxPart;
    return (int)g;
}

void launch_partial_norm2(tm_ctx *c, const void *v, int prec, int nrhs, double *part, hipStream_t s)
{
    const int nblk = norm_blocks(c);
    account(c, (double)half_elems(c) * nrhs * prec_bytes(prec), 4.0 * half_elems(c) * nrhs);
    dispatch_prec(prec, [&](auto *tag) {
        using S = std::remove_pointer_t<decltype(tag)>;
        hipLaunchKernelGGL(k_partial_norm2<S>, dim3(nblk, nrhs), dim3(kBlock), 0, s, (const S *)v, c->geo.vh,
                           c->geo.hs, part, nblk);
    });
    TM_HIP(hipGetLastError());
}

void launch_sum_partials(const double *part, int nblk, int n, double *dev_out, hipStream_t s)
{
    hipLaunchKernelGGL(k_finish_sum, dim3(n), dim3(kBlock), 0, s, part, nblk, dev_out);
    TM_HIP(hipGetLastError());
}

void launch_norm2(tm_ctx *c, const void *v, int prec, int nrhs, double *dev_out, hipStream_t s)
{
    const int nblk = norm_blocks(c);
    double *part = (double *)ws_get(c, "norm_part", sizeof(double) * nblk * nrhs);
    launch_partial_norm2(c, v, prec, nrhs, part, s);
    launch_sum_partials(part, nblk, nrhs, dev_out, s);
}

void launch_convert_norm(tm_ctx *c, void *out, int out_prec, const void *in, int in_prec, int nrhs,
                         const double *dscale, double *part, hipStream_t s)
{
    TM_REQUIRE(in_prec == out_prec || in_prec == TM_F64, "convert with norm: from FP64 or in one precision");
    const size_t n = half_elems(c) * nrhs;
    account(c, (double)n * (prec_bytes(in_prec) + (out ? prec_bytes(out_prec) : 0)), 6.0 * n);
    dim3 grid(norm_blocks(c), nrhs);
    dispatch_prec(out_prec, [&](auto *to) {
        using SO = std::remove_pointer_t<decltype(to)>;
        if (in_prec == out_prec)
            hipLaunchKernelGGL((k_convert_norm<SO, SO>), grid, dim3(kBlock), 0, s, (SO *)out, (const SO *)in,
                               c->geo.vh, c->geo.hs, dscale, part);
        else
            hipLaunchKernelGGL((k_convert_norm<SO, double2>), grid, dim3(kBlock), 0, s, (SO *)out,
                               (const double2 *)in, c->geo.vh, c->geo.hs, dscale, part);
    });
    TM_HIP(hipGetLastError());
}

void cg_finish_beta(tm_ctx *c, CGScalars *sc, const double *part, int nblk, int nrhs, double delta,
                    hipStream_t s)
{
    hipLaunchKernelGGL(k_finish_beta, dim3(nrhs), dim3(kBlock), 0, s, sc, part, nblk, nrhs, delta);
    TM_HIP(hipGetLastError());
}

void launch_zero(tm_ctx *c, void *y, int prec, int nrhs, hipStream_t s)
{
    size_t n = half_elems(c) * nrhs;
    account(c, (double)n * prec_bytes(prec), 0.0);
    dispatch_prec(prec, [&](auto *tag) {
        using S = std::remove_pointer_t<decltype(tag)>;
        hipLaunchKernelGGL(k_zero<S>, dim3(grid_for(n)), dim3(kBlock), 0, s, (S *)y, n);
    });
    TM_HIP(hipGetLastError());
}

void launch_axpy_dev(tm_ctx *c, void *y, int yprec, const void *x, int xprec, int nrhs, const double *a_dev,
                     hipStream_t s)
{
    size_t n = half_elems(c);
    dim3 grid(grid_for(n), nrhs);
    account(c, (double)n * nrhs * (2 * prec_bytes(yprec) + prec_bytes(xprec)), 4.0 * n * nrhs);
    dispatch_prec(yprec, [&](auto *ty) {
        using SY = std::remove_pointer_t<decltype(ty)>;
        dispatch_prec(xprec, [&](auto *tx) {
            using SX = std::remove_pointer_t<decltype(tx)>;
            hipLaunchKernelGGL((k_axpy_dev<SY, SX>), grid, dim3(kBlock), 0, s, (SY *)y, (const SX *)x, n, a_dev);
        });
    });
    TM_HIP(hipGetLastError());
}

void cg_update_cost(const CgRing &ring, int pos, int prec, int xprec, double &bytes, double &flops)
{
    const bool end = pos == ring.m - 1;
    bytes = (end ? ring.m + 2 : 3) * prec_bytes(prec) + (end ? 2 * prec_bytes(xprec) : 0);
    flops = end ? 4.0 * ring.m + 4 : 4.0;
}

// A launch of the beta step costs 1.5 us in the chain of an iteration; without it
// every block of the update reads the partial sums of its right-hand side, with
// reliable updates one quantity, else two.  The two break even at about 18 MB of
// such reads (12 TB/s, from the L2): FP16 with reliable updates on 16^3 x 32 (1024
// partial sums), an iteration of one right-hand side 37.3 us with the launch and
// 36.0 without, of three (19 MB) 93.0 and 92.8, of 24 466 and 476; truncated, 24^4
// (2592), 24 right-hand sides, 974 and 1086.
bool cg_beta_late(tm_ctx *c, int nrhs, int nblk, double delta)
{
    const double blocks = (double)grid_for(half_elems(c)) * nrhs;
    return blocks * nblk * sizeof(double) * (delta > 0 ? 1 : 2) <= 18e6;
}

void cg_update(tm_ctx *c, const CgRing &ring, int pos, const void *r, void *x, int prec, int xprec, int nrhs,
               const CGScalars *sc, hipStream_t s, const double *part, int nblk, double delta)
{
    const size_t n = half_elems(c);
    dim3 grid(grid_for(n), nrhs);
    double b, f;
    cg_update_cost(ring, pos, prec, xprec, b, f);
    account(c, b * n * nrhs, f * n * nrhs);
    RingArg a;
    std::copy(ring.p, ring.p + kCgRing, a.p);
    dispatch_tail(prec, xprec, [&](auto *ts, auto *tx) {
        using S = std::remove_pointer_t<decltype(ts)>;
        using XS = std::remove_pointer_t<decltype(tx)>;
        ring_form<S>(ring.m, pos, [&](auto m) {
            if (part)
                hipLaunchKernelGGL((k_update<m(), true, S, XS>), grid, dim3(kBlock), 0, s, a, pos, (const S *)r,
                                   (XS *)x, n, sc, part, nblk, nrhs, delta);
            else
                hipLaunchKernelGGL((k_update<m(), false, S, XS>), grid, dim3(kBlock), 0, s, a, pos, (const S *)r,
                                   (XS *)x, n, sc, part, nblk, nrhs, delta);
        });
    });
    TM_HIP(hipGetLastError());
}

void cg_flush(tm_ctx *c, const CgRing &ring, int cnt, void *x, int prec, int xprec, int nrhs, const CGScalars *sc,
              hipStream_t s)
{
    const size_t n = half_elems(c);
    account(c, (double)n * nrhs * (cnt * prec_bytes(prec) + 2 * prec_bytes(xprec)), 4.0 * cnt * n * nrhs);
    RingArg a;
    std::copy(ring.p, ring.p + kCgRing, a.p);
    dispatch_tail(prec, xprec, [&](auto *ts, auto *tx) {
        using S = std::remove_pointer_t<decltype(ts)>;
        using XS = std::remove_pointer_t<decltype(tx)>;
        hipLaunchKernelGGL((k_flush_x<S, XS>), dim3(grid_for(n), nrhs), dim3(kBlock), 0, s, a, cnt, (XS *)x, n, sc);
    });
    TM_HIP(hipGetLastError());
}
