// Restarted flexible GMRES (Saad 1993) on the full system M(mu) x = b in FP64,
// right-preconditioned by the parallel-transport network (ptc.hip) or by the
// identity (plain GMRES(m)).  Arnoldi with classical Gram-Schmidt, complex
// Givens rotations and the small least-squares problem on the device (one
// thread per right-hand side); the host reads one flag per right-hand side
// per Arnoldi step to stop.  After each cycle the true residual b - M x is
// recomputed in FP64 and the cycle restarts from it.
//
// Vectors are full fields as two half-lattice FP64 blocks, the even block
// [nrhs][12][hs] followed by the odd one; the preconditioned directions z_j
// are kept in FP32 (the precision the network returns them in), so
// x = x0 + sum_j y_j z_j uses exactly the vectors that M was applied to.
#include <algorithm>
#include <cmath>
#include <cstring>

#include "cg_device.h"
#include "runtime.h"

namespace {

constexpr int kBlock = 256;
constexpr int kChunk = 8;   // basis vectors per multi-dot / multi-axpy launch
constexpr int kDotBlk = 256;
constexpr int kMaxpyBlk = 2048;
static_assert(kMaxpyBlk <= kChunk * kDotBlk, "partials of the norm");
constexpr int kMaxM = 32;

using cgdev::wave_sum;

template <typename SV>
__device__ __forceinline__ cx<double> ldv(const SV *p, size_t k)
{
    return ldT<double>(p, k);
}

// part[((r*kChunk + i)*2 + h)*nblk + blk] (re, im) = block sums of conj(v_i) w
// over half h of right-hand side r (the vh valid sites of its 12 planes of
// stride ps; pad sites skipped), i < NB; grid (nblk, nrhs, 2).  Bound: memory.
// NB at compile time lets all loads of a site go out together, and the sums of
// a wave are DPP adds: sixteen of them through the LDS crossbar were 7 us a block.
template <int NB, typename SV>
__global__ __launch_bounds__(kBlock) void k_mdot(const SV *V, size_t vstride, const double2 *w, size_t n, size_t half,
                                                 int vh, int ps, double2 *part)
{
    const int r = blockIdx.y, h = blockIdx.z, nblk = gridDim.x;
    const size_t base = h * half + (size_t)r * n;
    double acc[2 * NB];
#pragma unroll
    for (int q = 0; q < 2 * NB; q++) acc[q] = 0;
    for (int k = 0; k < 12; k++) {
        for (int si = blockIdx.x * kBlock + threadIdx.x; si < vh; si += nblk * kBlock) {
            const size_t e = (size_t)k * ps + si;
            const double2 wv = w[base + e];
#pragma unroll
            for (int i = 0; i < NB; i++) {
                const cx<double> v = ldv(V, i * vstride + base + e);
                acc[2 * i] = fma(v.r, wv.x, fma(v.i, wv.y, acc[2 * i]));
                acc[2 * i + 1] = fma(v.r, wv.y, fma(-v.i, wv.x, acc[2 * i + 1]));
            }
        }
    }
    __shared__ double red[kBlock / 64][2 * NB];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
    for (int q = 0; q < 2 * NB; q++) {
        const double s = wave_sum(acc[q]);
        if (lane == 0) red[wv][q] = s;
    }
    __syncthreads();
    if (threadIdx.x < NB) {
        const int i = threadIdx.x;
        double re = 0, im = 0;
        for (int k = 0; k < kBlock / 64; k++) {
            re += red[k][2 * i];
            im += red[k][2 * i + 1];
        }
        part[(((size_t)r * kChunk + i) * 2 + h) * nblk + blockIdx.x] = make_double2(re, im);
    }
}

// out[r*ld + i0 + i] = sum over halves and blocks (fixed order) of the partials
// of vector i of `per` per right-hand side; one wave per (r, i), block r * nb + i
// (a thread each walked the 512 partials in series, 46 us a launch; now 3)
__global__ __launch_bounds__(64) void k_mdot_finish(const double2 *part, int per, int nb, int nblk, double2 *out,
                                                    int ld, int i0)
{
    const int r = blockIdx.x / nb, i = blockIdx.x % nb;
    const double2 *p = part + ((size_t)r * per + i) * 2 * nblk;
    double re = 0, im = 0;
    for (int b = threadIdx.x; b < 2 * nblk; b += 64) {
        re += p[b].x;
        im += p[b].y;
    }
    re = wave_sum(re);
    im = wave_sum(im);
    if (threadIdx.x == 0) out[(size_t)r * ld + i0 + i] = make_double2(re, im);
}

// w += sign * sum_i coef[r*ld + i0 + i] v_i, i < NB; grid (blocks, nrhs, 2).
// NORM: also the partial |w|^2 of each half (vh valid sites per plane of stride
// ps) as part[(r * 2 + h) * blocks + block], which saves reading w again
template <int NB, bool NORM, typename SV>
__global__ __launch_bounds__(kBlock) void k_maxpy(double2 *w, const SV *V, size_t vstride,
                                                  const double2 *__restrict__ coef, int ld, int i0, double sign,
                                                  size_t n, size_t half, int vh, int ps, double2 *part)
{
    const int r = blockIdx.y, h = blockIdx.z;
    const size_t base = h * half + (size_t)r * n;
    cx<double> cf[NB];
#pragma unroll
    for (int i = 0; i < NB; i++) {
        const double2 v = coef[(size_t)r * ld + i0 + i];
        cf[i] = {sign * v.x, sign * v.y};
    }
    double s = 0;
    for (size_t e = (size_t)blockIdx.x * kBlock + threadIdx.x; e < n; e += (size_t)gridDim.x * kBlock) {
        double2 a = w[base + e];
        cx<double> acc = {a.x, a.y};
#pragma unroll
        for (int i = 0; i < NB; i++) cmac(acc, cf[i], ldv(V, i * vstride + base + e));
        w[base + e] = make_double2(acc.r, acc.i);
        if constexpr (NORM)
            if ((int)((unsigned)e % (unsigned)ps) < vh) s = fma(acc.r, acc.r, fma(acc.i, acc.i, s));
    }
    if constexpr (NORM) {
        s = cgdev::block_sum(s);
        if (threadIdx.x == 0) part[((size_t)r * 2 + h) * gridDim.x + blockIdx.x] = make_double2(s, 0.0);
    }
}

// v = scale[r] w, and z = v in FP32 (z may be null); n elements per (half,
// right-hand side), grid (blocks, 2 nrhs)
__global__ __launch_bounds__(kBlock) void k_next(double2 *v, float2 *z, const double2 *w, size_t n, const double *scale)
{
    const size_t base = (size_t)blockIdx.y * n;
    const double sc = scale[blockIdx.y];
    for (size_t e = (size_t)blockIdx.x * kBlock + threadIdx.x; e < n; e += (size_t)gridDim.x * kBlock) {
        const double2 a = w[base + e];
        const double2 o = make_double2(sc * a.x, sc * a.y);
        v[base + e] = o;
        if (z) z[base + e] = make_float2((float)o.x, (float)o.y);
    }
}

struct GState {
    double2 *H;      // [nrhs][m+1][m], column j of the rotated Hessenberg matrix
    double *cs;      // [nrhs][m]
    double2 *sn;     // [nrhs][m]
    double2 *g;      // [nrhs][m+1]
    double2 *dots;   // [nrhs][m+1]: h_0..h_j of the current column, |w|^2 at j+1
    int *active;     // [nrhs]
    int *ncol;       // [nrhs] columns of the current cycle in the solution
    double *res2;    // [nrhs] |g_{ncol}|^2, the residual estimate squared
    const double *target2;  // [nrhs]
    double *vscale;  // [2 nrhs] scale of the next basis vector (both halves)
};

// Arnoldi column j for every right-hand side: rotate, new Givens rotation,
// residual estimate, convergence flag.  One thread per right-hand side.
__global__ void k_arnoldi(GState st, int j, int m, int nrhs)
{
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= nrhs) return;
    const double2 *d = st.dots + (size_t)r * (m + 1);
    const double hn = sqrt(fmax(d[j + 1].x, 0.0));
    const bool act = st.active[r] != 0;
    const double sc = act && hn > 0 ? 1.0 / hn : 0.0;
    st.vscale[r] = sc;
    st.vscale[r + nrhs] = sc;
    if (!act) return;
    cx<double> h[kMaxM + 1];
    for (int i = 0; i <= j; i++) h[i] = {d[i].x, d[i].y};
    h[j + 1] = {hn, 0};
    double *cs = st.cs + (size_t)r * m;
    double2 *sn = st.sn + (size_t)r * m;
    for (int i = 0; i < j; i++) {
        const cx<double> s = {sn[i].x, sn[i].y};
        const cx<double> t = cs[i] * h[i] + s * h[i + 1];
        h[i + 1] = cs[i] * h[i + 1] - conjg(s) * h[i];
        h[i] = t;
    }
    // G [a; b] = [rho; 0] with G = [[c, s], [-conj(s), c]], c real
    const cx<double> a = h[j], b = h[j + 1];
    const double na = sqrt(a.r * a.r + a.i * a.i), nb = sqrt(b.r * b.r + b.i * b.i);
    const double nn = sqrt(na * na + nb * nb);
    double c;
    cx<double> s;
    if (nn == 0) {
        c = 1;
        s = {0, 0};
    } else if (na == 0) {
        c = 0;
        s = {1, 0};
    } else {
        c = na / nn;
        const cx<double> ph = {a.r / na, a.i / na};
        s = (1.0 / nn) * (ph * conjg(b));
    }
    h[j] = c * a + s * b;
    h[j + 1] = {0, 0};
    cs[j] = c;
    sn[j] = make_double2(s.r, s.i);
    double2 *H = st.H + (size_t)r * (m + 1) * m;
    for (int i = 0; i <= j + 1; i++) H[(size_t)i * m + j] = make_double2(h[i].r, h[i].i);
    double2 *g = st.g + (size_t)r * (m + 1);
    const cx<double> gj = {g[j].x, g[j].y};
    const cx<double> g1 = {0, 0};
    const cx<double> nj = c * gj + s * g1, nj1 = c * g1 - conjg(s) * gj;
    g[j] = make_double2(nj.r, nj.i);
    g[j + 1] = make_double2(nj1.r, nj1.i);
    st.ncol[r] = j + 1;
    st.res2[r] = nj1.r * nj1.r + nj1.i * nj1.i;
    if (st.res2[r] <= st.target2[r]) st.active[r] = 0;
}

// y = R^-1 g over the ncol columns of the cycle (zeros beyond); one thread
// per right-hand side
__global__ void k_backsolve(GState st, double2 *y, int m, int nrhs)
{
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= nrhs) return;
    const int n = st.ncol[r];
    const double2 *H = st.H + (size_t)r * (m + 1) * m;
    const double2 *g = st.g + (size_t)r * (m + 1);
    double2 *yr = y + (size_t)r * m;
    for (int i = n; i < m; i++) yr[i] = make_double2(0, 0);
    for (int i = n - 1; i >= 0; i--) {
        cx<double> acc = {g[i].x, g[i].y};
        for (int k = i + 1; k < n; k++) {
            const cx<double> hk = {H[(size_t)i * m + k].x, H[(size_t)i * m + k].y};
            const cx<double> yk = {yr[k].x, yr[k].y};
            acc = acc - hk * yk;
        }
        const cx<double> d = {H[(size_t)i * m + i].x, H[(size_t)i * m + i].y};
        const double dd = d.r * d.r + d.i * d.i;
        const cx<double> q = dd > 0 ? cx<double>{(acc.r * d.r + acc.i * d.i) / dd, (acc.i * d.r - acc.r * d.i) / dd}
                                    : cx<double>{0, 0};
        yr[i] = make_double2(q.r, q.i);
    }
}

struct Fg {
    tm_ctx *c;
    int nrhs, m;
    size_t n, hs;  // elements per right-hand side per half (pads included), per half
    hipStream_t s;
    double2 *part;
};

// f(integral constant nb), 1 <= nb <= kChunk
template <typename F>
void with_count(int nb, F &&f)
{
    static_assert(kChunk == 8);
    switch (nb) {
    case 1: return f(std::integral_constant<int, 1>{});
    case 2: return f(std::integral_constant<int, 2>{});
    case 3: return f(std::integral_constant<int, 3>{});
    case 4: return f(std::integral_constant<int, 4>{});
    case 5: return f(std::integral_constant<int, 5>{});
    case 6: return f(std::integral_constant<int, 6>{});
    case 7: return f(std::integral_constant<int, 7>{});
    default: return f(std::integral_constant<int, 8>{});
    }
}

// out[r*ld + i0 .. i0 + nb) = <v_i, w> for nb basis vectors in chunks
template <typename SV>
void mdot(Fg &f, const SV *V, size_t vstride, int nb, const double2 *w, double2 *out, int ld, int i0)
{
    // both halves: nb basis vectors and w read once, 8 flops per complex product-add
    account(f.c, 2.0 * f.n * f.nrhs * (nb * sizeof(SV) + sizeof(double2)), 16.0 * f.n * f.nrhs * nb);
    for (int c0 = 0; c0 < nb; c0 += kChunk) {
        const int k = std::min(kChunk, nb - c0);
        with_count(k, [&](auto m) {
            hipLaunchKernelGGL((k_mdot<m(), SV>), dim3(kDotBlk, f.nrhs, 2), dim3(kBlock), 0, f.s, V + c0 * vstride,
                               vstride, w, f.n, f.hs, f.c->geo.vh, f.c->geo.hs, f.part);
        });
        TM_HIP(hipGetLastError());
        hipLaunchKernelGGL(k_mdot_finish, dim3(f.nrhs * k), dim3(64), 0, f.s, (const double2 *)f.part, kChunk, k,
                           kDotBlk, out, ld, i0 + c0);
        TM_HIP(hipGetLastError());
    }
}

// norm: also |w|^2 of the result into norm[r*ld] (re)
template <typename SV>
void maxpy(Fg &f, double2 *w, const SV *V, size_t vstride, int nb, const double2 *coef, int ld, double sign,
           double2 *norm = nullptr)
{
    const int blocks = (int)std::min<size_t>((f.n + kBlock - 1) / kBlock, kMaxpyBlk);
    account(f.c, 2.0 * f.n * f.nrhs * (nb * sizeof(SV) + 2 * sizeof(double2)), 16.0 * f.n * f.nrhs * nb);
    for (int c0 = 0; c0 < nb; c0 += kChunk) {
        const int k = std::min(kChunk, nb - c0);
        with_count(k, [&](auto m) {
            const dim3 grid(blocks, f.nrhs, 2);
            if (norm && c0 + k == nb)
                hipLaunchKernelGGL((k_maxpy<m(), true, SV>), grid, dim3(kBlock), 0, f.s, w, V + c0 * vstride, vstride,
                                   coef, ld, c0, sign, f.n, f.hs, f.c->geo.vh, f.c->geo.hs, f.part);
            else
                hipLaunchKernelGGL((k_maxpy<m(), false, SV>), grid, dim3(kBlock), 0, f.s, w, V + c0 * vstride, vstride,
                                   coef, ld, c0, sign, f.n, f.hs, f.c->geo.vh, f.c->geo.hs, f.part);
        });
        TM_HIP(hipGetLastError());
    }
    if (norm) {
        hipLaunchKernelGGL(k_mdot_finish, dim3(f.nrhs), dim3(64), 0, f.s, (const double2 *)f.part, 1, 1, blocks, norm,
                           ld, 0);
        TM_HIP(hipGetLastError());
    }
}

// v = scale w per half and right-hand side, z = v in FP32 (may be null)
void next_vector(Fg &f, double2 *v, float2 *z, const double2 *w, const double *scale)
{
    const size_t all = 2 * f.n * f.nrhs;
    account(f.c, (double)all * (2 * sizeof(double2) + (z ? sizeof(float2) : 0)), 2.0 * all);
    const int blocks = (int)std::min<size_t>((f.n + 4 * kBlock - 1) / (4 * kBlock), 4096);
    hipLaunchKernelGGL(k_next, dim3(blocks, 2 * f.nrhs), dim3(kBlock), 0, f.s, v, z, w, f.n, scale);
    TM_HIP(hipGetLastError());
}

// out = M in on full FP64 fields (halves consecutive)
void apply_M(Fg &f, double2 *out, const double2 *in, double epsp)
{
    tm_ctx *c = f.c;
    const SpinDiag dh = sd_scalar(-c->kappa), dw = sd_twist(epsp);
    op_dslash(c, out, in + f.hs, in, f.nrhs, TM_F64, 0, 0, dh, dw, f.s);
    op_dslash(c, out + f.hs, in, in + f.hs, f.nrhs, TM_F64, 1, 0, dh, dw, f.s);
}

}  // namespace

SolveOut fgmres_halves(tm_ctx *c, void *xe, void *xo, const void *be, const void *bo, int nrhs,
                       const tm_solve_params &p, hipStream_t s)
{
    const double t0 = now_s();
    const bool ptc = p.solver == TM_FGMRES_PTC;
    TM_REQUIRE(p.tol > 0 && std::isfinite(p.tol), "tol must be > 0");
    TM_REQUIRE(p.maxiter > 0, "maxiter must be > 0");
    TM_REQUIRE(p.mu_sign == 1 || p.mu_sign == -1, "mu_sign must be +1 or -1");
    TM_REQUIRE(!ptc || c->ptc_nc > 0, "FGMRES with the network needs weights (tm_ptc_set_weights / train)");
    const int m = p.check_every > 0 ? p.check_every : 16;
    TM_REQUIRE(m >= 1 && m <= kMaxM, "restart length must be in [1, 32]");
    const double epsp = eps_of(c, p.mu_sign);
    Fg f{c, nrhs, m, (size_t)12 * c->geo.hs, (size_t)12 * c->geo.hs * nrhs, s, nullptr};
    const size_t vs = 2 * f.hs;  // complex elements per full vector (all rhs)
    f.part = (double2 *)ws_get(c, "fg_part", sizeof(double2) * nrhs * kChunk * 2 * kDotBlk);
    double2 *V = (double2 *)ws_get(c, "fg_V", sizeof(double2) * vs * (m + 1));
    float2 *Z = ptc ? (float2 *)ws_get(c, "fg_Z", sizeof(float2) * vs * m) : nullptr;
    float2 *zin = ptc ? (float2 *)ws_get(c, "fg_zin", sizeof(float2) * vs) : nullptr;
    double2 *x = (double2 *)ws_get(c, "fg_x", sizeof(double2) * vs);
    double2 *b = (double2 *)ws_get(c, "fg_b", sizeof(double2) * vs);
    double2 *w = (double2 *)ws_get(c, "fg_w", sizeof(double2) * vs);
    double2 *zt = ptc ? (double2 *)ws_get(c, "fg_zt", sizeof(double2) * vs) : nullptr;
    GState st;
    st.H = (double2 *)ws_get(c, "fg_H", sizeof(double2) * nrhs * (m + 1) * m);
    st.cs = (double *)ws_get(c, "fg_cs", sizeof(double) * nrhs * m);
    st.sn = (double2 *)ws_get(c, "fg_sn", sizeof(double2) * nrhs * m);
    st.g = (double2 *)ws_get(c, "fg_g", sizeof(double2) * nrhs * (m + 1));
    st.dots = (double2 *)ws_get(c, "fg_dots", sizeof(double2) * nrhs * (m + 1));
    st.active = (int *)ws_get(c, "fg_active", sizeof(int) * nrhs);
    st.ncol = (int *)ws_get(c, "fg_ncol", sizeof(int) * nrhs);
    st.res2 = (double *)ws_get(c, "fg_res2", sizeof(double) * nrhs);
    double *target2 = (double *)ws_get(c, "fg_target2", sizeof(double) * nrhs);
    st.target2 = target2;
    st.vscale = (double *)ws_get(c, "fg_vscale", sizeof(double) * 2 * nrhs);
    double2 *y = (double2 *)ws_get(c, "fg_y", sizeof(double2) * nrhs * m);
    const size_t hb = field_bytes(c, TM_F64, nrhs);
    copy_field(b, be, hb, s);
    copy_field(b + f.hs, bo, hb, s);
    launch_zero(c, x, TM_F64, 2 * nrhs, s);

    std::vector<double> bn2(nrhs), t2(nrhs), beta2(nrhs), res2(nrhs), hscale(2 * nrhs);
    std::vector<int> iters(nrhs, 0), act(nrhs);
    std::vector<double2> h_d(nrhs * (m + 1));
    {
        mdot(f, b, vs, 1, b, st.dots, m + 1, 0);
        download(c, h_d.data(), st.dots, sizeof(double2) * nrhs * (m + 1), s);
        for (int r = 0; r < nrhs; r++) {
            bn2[r] = h_d[(size_t)r * (m + 1)].x;
            TM_REQUIRE(std::isfinite(bn2[r]), "NaN/Inf in the source");
            t2[r] = p.tol * p.tol * bn2[r];
        }
        upload(target2, t2.data(), sizeof(double) * nrhs, s);
    }
    int restarts = 0, total = 0;
    bool nan = false, fallback = false;
    std::vector<double> prev2(nrhs, 0.0);
    while (true) {
        // V_0 = b - M x, beta = |V_0|
        apply_M(f, w, x, epsp);
        copy_field(V, b, 2 * hb, s);
        launch_axpby_host(c, V, w, TM_F64, 2 * nrhs, -1.0, 1.0, s);
        mdot(f, V, vs, 1, V, st.dots, m + 1, 0);
        download(c, h_d.data(), st.dots, sizeof(double2) * nrhs * (m + 1), s);
        bool any = false, stalled = false;
        for (int r = 0; r < nrhs; r++) {
            beta2[r] = h_d[(size_t)r * (m + 1)].x;
            if (!std::isfinite(beta2[r])) nan = true;
            act[r] = beta2[r] > t2[r] ? 1 : 0;
            any |= act[r] != 0;
            res2[r] = beta2[r];
            // a full restart cycle that did not halve the residual
            if (ptc && restarts > 0 && act[r] && beta2[r] > 0.25 * prev2[r]) stalled = true;
            prev2[r] = beta2[r];
        }
        if (nan || !any || total >= p.maxiter) break;
        if (stalled) {
            fallback = true;
            break;
        }
        std::vector<double2> g0((size_t)nrhs * (m + 1), make_double2(0, 0));
        for (int r = 0; r < nrhs; r++) {
            const double be_ = std::sqrt(beta2[r]);
            hscale[r] = hscale[r + nrhs] = act[r] ? 1.0 / be_ : 0.0;
            g0[(size_t)r * (m + 1)] = make_double2(act[r] ? be_ : 0.0, 0.0);
        }
        upload(st.g, g0.data(), sizeof(double2) * g0.size(), s);
        upload(st.active, act.data(), sizeof(int) * nrhs, s);
        std::vector<int> zero(nrhs, 0);
        upload(st.ncol, zero.data(), sizeof(int) * nrhs, s);
        upload(st.vscale, hscale.data(), sizeof(double) * 2 * nrhs, s);
        next_vector(f, V, zin, V, st.vscale);
        int j = 0;
        for (; j < m && total < p.maxiter; j++) {
            double2 *vj = V + (size_t)j * vs;
            // w = M z_j, z_j = N(v_j) (zin: v_j in FP32) or v_j
            if (ptc) {
                float2 *zj = Z + (size_t)j * vs;
                ptc_apply_halves(c, zin, zin + f.hs, zj, zj + f.hs, nrhs, s);
                launch_copy_convert(c, zt, TM_F64, zj, TM_F32, 2 * nrhs, nullptr, s);
                apply_M(f, w, zt, epsp);
            } else {
                apply_M(f, w, vj, epsp);
            }
            // classical Gram-Schmidt against v_0..v_j, then |w|^2
            mdot(f, V, vs, j + 1, w, st.dots, m + 1, 0);
            maxpy(f, w, V, vs, j + 1, st.dots, m + 1, -1.0, st.dots + j + 1);
            hipLaunchKernelGGL(k_arnoldi, dim3((nrhs + 63) / 64), dim3(64), 0, s, st, j, m, nrhs);
            TM_HIP(hipGetLastError());
            next_vector(f, V + (size_t)(j + 1) * vs, zin, w, st.vscale);
            total++;
            for (int r = 0; r < nrhs; r++) iters[r] += act[r];
            download(c, act.data(), st.active, sizeof(int) * nrhs, s);
            bool still = false;
            for (int r = 0; r < nrhs; r++) still |= act[r] != 0;
            if (!still) {
                j++;
                break;
            }
        }
        // x += sum_j y_j z_j
        hipLaunchKernelGGL(k_backsolve, dim3((nrhs + 63) / 64), dim3(64), 0, s, st, y, m, nrhs);
        TM_HIP(hipGetLastError());
        if (ptc)
            maxpy(f, x, Z, vs, j, y, m, 1.0);
        else
            maxpy(f, x, V, vs, j, y, m, 1.0);
        restarts++;
    }
    // Fallback when the preconditioned iteration stalls: the remaining
    // correction M d = b - M x (in V_0, unscaled) by the plain mixed-precision
    // CG (FP16 storage, FP64 reliable updates) to the tolerance that brings
    // every right-hand side to tol, then x += d and the true residual again.
    std::vector<tm_solve_stats> cg_st;
    if (fallback && !nan) {
        double tol_d = 1.0;
        for (int r = 0; r < nrhs; r++)
            if (beta2[r] > t2[r]) tol_d = std::min(tol_d, p.tol * std::sqrt(bn2[r] / beta2[r]));
        tm_solve_params pc = p;
        pc.solver = TM_CG_MIXED;
        pc.inner_prec = TM_F16;
        pc.tol = tol_d;
        pc.maxiter = std::max(1, p.maxiter - total) * 8;
        pc.check_every = 0;
        pc.delta = 0;
        double2 *d = (double2 *)ws_get(c, "fg_d", sizeof(double2) * vs);
        double2 *rr = (double2 *)ws_get(c, "fg_r", sizeof(double2) * vs);
        copy_field(rr, V, 2 * hb, s);
        SolveOut cg = solve_halves(c, d, d + f.hs, rr, rr + f.hs, nrhs, pc, s);
        if (cg.status == TM_ERR_NAN) nan = true;
        cg_st = cg.st;
        launch_axpby_host(c, x, d, TM_F64, 2 * nrhs, 1.0, 1.0, s);
        apply_M(f, w, x, epsp);
        copy_field(V, b, 2 * hb, s);
        launch_axpby_host(c, V, w, TM_F64, 2 * nrhs, -1.0, 1.0, s);
        mdot(f, V, vs, 1, V, st.dots, m + 1, 0);
        download(c, h_d.data(), st.dots, sizeof(double2) * nrhs * (m + 1), s);
        for (int r = 0; r < nrhs; r++) {
            beta2[r] = h_d[(size_t)r * (m + 1)].x;
            if (!std::isfinite(beta2[r])) nan = true;
        }
    }
    // solution out; true residual already in beta2 (b - M x of the last x)
    copy_field(xe, x, hb, s);
    copy_field(xo, x + f.hs, hb, s);
    TM_HIP(hipStreamSynchronize(s));
    SolveOut out;
    out.st.resize(nrhs);
    for (int r = 0; r < nrhs; r++) {
        tm_solve_stats &q = out.st[r];
        q = tm_solve_stats{};
        q.iters = iters[r] + (cg_st.empty() ? 0 : cg_st[r].iters);
        q.n_reliable = restarts;
        q.fallback = fallback ? 1 : 0;
        q.true_rel_res = std::sqrt(beta2[r] / bn2[r]);
        q.iter_rel_res = q.true_rel_res;
        q.converged = q.true_rel_res <= p.tol ? 1 : 0;
        q.seconds = now_s() - t0;
        if (!q.converged && out.status == TM_OK) out.status = TM_ERR_NOCONV;
    }
    if (nan) out.status = TM_ERR_NAN;
    return out;
}
