// Momentum projection of the loops (appendix A.2, contraction kernels, and
// the Fourier step of appendix A.3): the colour-traced Dirac outer products are formed per site,
// C(x)[b][a] = sum_r sum_c v_{r,bc}(x) w*_{r,ac}(x) for ultra-local
// insertions, and for the one-derivative insertions (the covariant-derivative
// kernel of appendix A.2) in each direction mu
//   D_mu(x)[b][a] = 1/4 sum_r sum_c [(nabla_mu v)_{bc} w*_{ac} - v_{bc} (nabla_mu w)*_{ac}],
//   nabla_mu f(x) = U_mu(x) f(x + mu) - U_mu(x - mu)^dag f(x - mu)
// (the symmetric left-right derivative of the bilinear w^dag Gamma D_mu v
// attributed to x, time-boundary phase included).  The two backward terms at
// x are the forward terms at x - mu:
//   D_mu(x) = (E_mu(x) + E_mu(x - mu)) / 4,
//   E_mu(x)[b][a] = sum_r sum_c [(U_mu(x) v(x + mu))_{bc} w*_{ac}(x) - v_{bc}(x) (U_mu(x) w(x + mu))*_{ac}],
// so only E is formed per site, and the shift by mu is a factor e^{i p_mu}
// (spatial mu) or the neighbouring slice (time) of its Fourier sum.  For
// v = w the second term of E is the adjoint of the first.  Then they are
// transformed over the spatial coordinates of each time slice,
//   C_p(t) = sum_{x in t} e^{i p.x} C(x),  p = 2 pi (nx/Lx, ny/Ly, nz/Lz),
// for every integer n with |n|^2 <= p2max.  The transform is separable, so it
// runs as three direct one-dimensional transforms (x, then y, then z) over
// the 2N+1 needed components per direction (N = floor(sqrt(p2max))), each a
// fixed-order sum, the first inside the kernel that forms the products.  The
// last kernel selects the momenta inside the sphere and inserts the Gamma
// matrices.  Phases come from FP64 tables of e^{2 pi i k / L}, k = n x mod L.
#include <cmath>

#include "runtime.h"

namespace {

constexpr int kBlock = 256;

// What a site kernel forms (16 products per site and block of products): v w*
// at the site, or F_mu for the four mu
enum { SITE_LOCAL = 0, SITE_HOP = 1 };

// C[b][a] = sum_r v_b w*_a at half-site i (SITE_HOP: (U v(x + mu))_b, link U at
// lk, neighbour jf).  SAME (local only): v and w are one field, read once.
// One thread keeps all 16 products (two waves per SIMD with a link): two
// threads per site at three waves, each the products of two spins, took 5.95
// against 4.77 ms at 32^3 x 64 and 12 right-hand sides, half-empty loads
// costing more than the waves gave.
template <int KIND, bool SAME>
__device__ __forceinline__ void site_products(cx<double> C[16], const double2 *v, const double2 *w, const double2 *lk,
                                              size_t vh, size_t hs, size_t i, size_t jf, int nrhs)
{
    cx<double> U[9];
    if constexpr (KIND == SITE_HOP) {
#pragma unroll
        for (int e = 0; e < 9; e++) {
            const double2 a = lk[e * vh + i];
            U[e] = {a.x, a.y};
        }
    }
    for (int r = 0; r < nrhs; r++) {
        const double2 *vr = v + (size_t)r * 12 * hs + (KIND == SITE_HOP ? jf : i), *wr = w + (size_t)r * 12 * hs + i;
        cx<double> wx[12];
#pragma unroll
        for (int k = 0; k < 12; k++) {
            const double2 a = wr[k * hs];
            wx[k] = {a.x, a.y};
        }
#pragma unroll
        for (int b = 0; b < 4; b++) {
            cx<double> h[3];
            if constexpr (SAME) {
#pragma unroll
                for (int c = 0; c < 3; c++) h[c] = wx[3 * b + c];
            } else {
                cx<double> f[3];
#pragma unroll
                for (int c = 0; c < 3; c++) {
                    const double2 x = vr[(3 * b + c) * hs];
                    f[c] = {x.x, x.y};
                }
#pragma unroll
                for (int q = 0; q < 3; q++) {
                    if constexpr (KIND == SITE_HOP) {
                        h[q] = {0, 0};
#pragma unroll
                        for (int c = 0; c < 3; c++) cmac(h[q], U[3 * q + c], f[c]);
                    } else {
                        h[q] = f[q];
                    }
                }
            }
#pragma unroll
            for (int a = 0; a < 4; a++)
#pragma unroll
                for (int c = 0; c < 3; c++) cmac_conj(C[4 * b + a], wx[3 * a + c], h[c]);
        }
    }
}

// sum_k f[k] g[k stride], k < n.  SITE_LOCAL: one chain of FMAs.  SITE_HOP: four (terms
// k mod 4), added in pairs.  The forward products of the derivative are summed apart
// from their counterparts, with larger partial sums than those of the derivative
// itself: with one chain its insertions were up to 10% further from sums in 80 bits
// than site-by-site derivatives, with four they are as close (12 x 12 x 14 x 8, one
// right-hand side: 3.7e-16, 4.1e-16 with one chain, 3.7e-16 site by site).
template <int KIND>
__device__ __forceinline__ cx<double> chain_sum(const double2 *f, const double2 *g, int n, long stride)
{
    constexpr int NC = KIND == SITE_HOP ? 4 : 1;
    cx<double> acc[4] = {{0, 0}, {0, 0}, {0, 0}, {0, 0}};
    int k = 0;
    for (; k + NC <= n; k += NC)
#pragma unroll
        for (int q = 0; q < NC; q++) {
            const double2 a = f[k + q], b = g[(k + q) * stride];
            cmac(acc[q], cx<double>{a.x, a.y}, cx<double>{b.x, b.y});
        }
    if constexpr (NC == 1) return acc[0];
#pragma unroll
    for (int q = 0; q < NC - 1; q++)
        if (k + q < n) {
            const double2 a = f[k + q], b = g[(k + q) * stride];
            cmac(acc[q], cx<double>{a.x, a.y}, cx<double>{b.x, b.y});
        }
    return (acc[0] + acc[1]) + (acc[2] + acc[3]);
}

// The products of every site (thread) and their transform along x: a block
// takes `rows` whole x rows (rows Lx <= 256 sites); T1[(blk 16 + e)][row][j] =
// sum_x ph[j][x] C(x, row)[e], each a fixed-order sum over x, four of the 16
// products at a time through LDS (rows padded by one against bank conflicts).
// Writing the products to memory first cost a pass of 16 V complex out and
// back (64 V with derivatives) and a transform kernel of its own.
// Measured at 32^3 x 64, 12 right-hand sides, |n|^2 <= 9: the 64 derivative
// products and their x transform 12.4 ms before E and this fusion, now 4.8 ms
// for v = w and twice that else (two fields of 4.8 GB, read once per
// direction where the neighbour is no longer in the L2; the rest is the wait
// of two waves per SIMD); the local ones 1.9 -> 1.1 ms (4.5 TB/s) for v = w.
// Block order (nblk = 4, one per mu): block b runs on XCD b % 8 (round-robin
// dispatch).  XCD k owns the contiguous range of row groups [k per, (k + 1)
// per) and takes them in order, the directions of one group as consecutive
// blocks, so that they read the sites' fields (2.3 KB per site and field at 12
// right-hand sides) while they are in that XCD's L2.
constexpr int kPass = 4;

template <int KIND, bool SAME>
__global__ __launch_bounds__(kBlock, 2) void k_site_rows(const double2 *ve, const double2 *vo, const double2 *we,
                                                         const double2 *wo, const double2 *l0, const double2 *l1, Geo g,
                                                         int nrhs, int rows, long nrow, long per, const double2 *ph,
                                                         int W, double2 *T1)
{
    extern __shared__ double2 tile[];  // [kPass][rows][Lx + 1]
    const int Lx = g.L[0];
    const int nblk = KIND == SITE_HOP ? 4 : 1;
    const long m = (long)(blockIdx.x >> 3);
    const int mu = (int)(m % nblk);
    const long row0 = ((long)(blockIdx.x & 7) * per + m / nblk) * rows;
    if (row0 >= nrow) return;
    const int lr = (int)threadIdx.x / Lx, x = (int)threadIdx.x - lr * Lx;
    const bool on = lr < rows && row0 + lr < nrow;
    cx<double> C[16];
#pragma unroll
    for (int e = 0; e < 16; e++) C[e] = {0, 0};
    if (on) {
        const int q = (int)(row0 + lr);
        const int y = q % g.L[1], q2 = q / g.L[1], z = q2 % g.L[2], t = q2 / g.L[2];
        const int p = (x + y + z + t) & 1;
        const size_t i = (size_t)(x >> 1) + (size_t)g.lxh * q;
        size_t jf = 0;
        if constexpr (KIND == SITE_HOP) {
            int c[4] = {x, y, z, t};
            c[mu] = c[mu] + 1 == g.L[mu] ? 0 : c[mu] + 1;
            jf = (size_t)eo_index(g, c[0], c[1], c[2], c[3]);
        }
        // links[p][d][9][vh]: d = mu is U_mu(x), time-boundary phase included;
        // a hop reads v on the other parity
        const double2 *lk = KIND == SITE_HOP ? (p ? l1 : l0) + (size_t)mu * 9 * g.vh : nullptr;
        site_products<KIND, SAME>(C, (p == (KIND == SITE_HOP)) ? ve : vo, p ? wo : we, lk, (size_t)g.vh, (size_t)g.hs,
                                  i, jf, nrhs);
    }
    const int rs = Lx + 1, plane = rows * rs;
    const int nout = kPass * rows * W;
#pragma unroll
    for (int e0 = 0; e0 < 16; e0 += kPass) {
        if (e0) __syncthreads();
        if (on) {
#pragma unroll
            for (int e = 0; e < kPass; e++) tile[e * plane + lr * rs + x] = make_double2(C[e0 + e].r, C[e0 + e].i);
        }
        __syncthreads();
        for (int o = threadIdx.x; o < nout; o += kBlock) {
            const int j = o % W, er = o / W, row = er % rows, e = er / rows;
            if (row0 + row >= nrow) continue;
            const double2 *f = ph + (long)j * Lx, *src = tile + e * plane + row * rs;
            const cx<double> acc = chain_sum<KIND>(f, src, Lx, 1);
            T1[((long)(16 * mu + e0 + e) * nrow + row0 + row) * W + j] = make_double2(acc.r, acc.i);
        }
    }
}

// The products alone, Cf[blk 16 + e][s], s = x + Lx (y + Ly (z + Lz t)): x
// rows longer than a block, transformed by k_dft_dim afterwards.
template <int KIND, bool SAME>
__global__ __launch_bounds__(kBlock, 2) void k_sites(const double2 *ve, const double2 *vo, const double2 *we,
                                                     const double2 *wo, const double2 *l0, const double2 *l1, Geo g,
                                                     long V, int nrhs, double2 *Cf)
{
    const long s = (long)blockIdx.x * kBlock + threadIdx.x;
    if (s >= V) return;
    const int mu = blockIdx.y;
    int c[4];
    c[0] = (int)(s % g.L[0]);
    const long q = s / g.L[0];
    c[1] = (int)(q % g.L[1]);
    const long q2 = q / g.L[1];
    c[2] = (int)(q2 % g.L[2]);
    c[3] = (int)(q2 / g.L[2]);
    const int p = (c[0] + c[1] + c[2] + c[3]) & 1;
    if constexpr (KIND == SITE_HOP) c[mu] = c[mu] + 1 == g.L[mu] ? 0 : c[mu] + 1;
    const size_t jf = (size_t)eo_index(g, c[0], c[1], c[2], c[3]);
    const double2 *lk = KIND == SITE_HOP ? (p ? l1 : l0) + (size_t)mu * 9 * g.vh : nullptr;
    cx<double> C[16];
#pragma unroll
    for (int e = 0; e < 16; e++) C[e] = {0, 0};
    site_products<KIND, SAME>(C, (p == (KIND == SITE_HOP)) ? ve : vo, p ? wo : we, lk, (size_t)g.vh, (size_t)g.hs,
                              (size_t)(s >> 1), jf, nrhs);
#pragma unroll
    for (int e = 0; e < 16; e++) Cf[((size_t)mu * 16 + e) * V + s] = make_double2(C[e].r, C[e].i);
}

// One direction of the transform: in [outer][n][inner] -> out[outer][W][inner]
// with out[o][j][k] = sum_m ph[j][m] in[o][m][k] (fixed order in m).
template <int KIND>
__global__ __launch_bounds__(kBlock) void k_dft_dim(const double2 *in, double2 *out, const double2 *ph, long outer,
                                                    int n, int W, long inner)
{
    const long idx = (long)blockIdx.x * kBlock + threadIdx.x;
    const long total = outer * W * inner;
    if (idx >= total) return;
    const long k = idx % inner;
    const long rest = idx / inner;
    const int j = (int)(rest % W);
    const long o = rest / W;
    const double2 *src = in + (o * n) * inner + k;
    const double2 *f = ph + (long)j * n;
    const cx<double> acc = chain_sum<KIND>(f, src, n, inner);
    out[idx] = make_double2(acc.r, acc.i);
}

// Gamma_n of the chiral basis and the matrices inserted for the three
// estimator forms (GammaForm): Gamma, gamma5 Gamma, gamma5 Gamma gamma5
struct Insertions {
    double2 X[3][16][16];  // [form][n][4 a + b]
};
constexpr Insertions make_insertions()
{
    // products with gamma_mu have one entry of +-1 or +-i per row, so integer
    // arithmetic is exact
    struct Z {
        int r, i;
    };
    Z gm[4][4][4] = {};
    gm[0][0][3] = gm[0][1][2] = Z{0, -1};
    gm[0][2][1] = gm[0][3][0] = Z{0, 1};
    gm[1][0][3] = gm[1][3][0] = Z{-1, 0};
    gm[1][1][2] = gm[1][2][1] = Z{1, 0};
    gm[2][0][2] = gm[2][3][1] = Z{0, -1};
    gm[2][1][3] = gm[2][2][0] = Z{0, 1};
    gm[3][0][2] = gm[3][1][3] = gm[3][2][0] = gm[3][3][1] = Z{1, 0};
    Insertions out{};
    for (int n = 0; n < 16; n++) {
        Z G[4][4] = {};
        for (int a = 0; a < 4; a++) G[a][a] = Z{1, 0};
        for (int mu = 0; mu < 4; mu++) {
            if (!((n >> mu) & 1)) continue;
            Z T[4][4] = {};
            for (int a = 0; a < 4; a++)
                for (int b = 0; b < 4; b++)
                    for (int k = 0; k < 4; k++) {
                        const Z p = G[a][k], q = gm[mu][k][b];
                        T[a][b].r += p.r * q.r - p.i * q.i;
                        T[a][b].i += p.r * q.i + p.i * q.r;
                    }
            for (int a = 0; a < 4; a++)
                for (int b = 0; b < 4; b++) G[a][b] = T[a][b];
        }
        for (int a = 0; a < 4; a++)
            for (int b = 0; b < 4; b++) {
                const int l = a < 2 ? 1 : -1, r = b < 2 ? 1 : -1;  // gamma5 = diag(1, 1, -1, -1)
                const double re = G[a][b].r, im = G[a][b].i;
                out.X[G_PLAIN][n][4 * a + b].x = re;
                out.X[G_PLAIN][n][4 * a + b].y = im;
                out.X[G_G5_LEFT][n][4 * a + b].x = l * re;
                out.X[G_G5_LEFT][n][4 * a + b].y = l * im;
                out.X[G_G5_BOTH][n][4 * a + b].x = l * r * re;
                out.X[G_G5_BOTH][n][4 * a + b].y = l * r * im;
            }
    }
    return out;
}
__constant__ const Insertions c_ins = make_insertions();

// out[m][ins0 + 16 blk + n][t] = coef sum_ab X_n[a][b] C[b][a], the loops of
// the listed momenta, from the Fourier sums T[16 blk + e][t][nz + N][ny + N][nx + N]:
// C is T itself (G null), or with derivatives (nblk = 4, blk = mu; T and G the
// sums of F(v, w) and F(w, v)) C = (E(p, t) (1 + e^{i p_mu}))/4 for spatial mu
// and (E(p, t) + E(p, t - 1))/4 for time, E[b][a](p) = T[b][a](p) - conj(G[a][b](-p)).
// shift: [3][W] of 1 + e^{i p_mu}.
__global__ __launch_bounds__(kBlock) void k_insert(const double2 *T, const double2 *G, const int *mom, int n_mom,
                                                   int nblk, Geo g, int W, int N, const double2 *shift, int form,
                                                   cx<double> coef, int n_ins, int ins0, double2 *out)
{
    const long idx = (long)blockIdx.x * kBlock + threadIdx.x;
    const int Lt = g.L[3];
    if (idx >= (long)n_mom * nblk * 16 * Lt) return;
    const int t = (int)(idx % Lt);
    long rest = idx / Lt;
    const int n = (int)(rest % 16);
    rest /= 16;
    const int blk = (int)(rest % nblk), m = (int)(rest / nblk);
    const int jx = mom[3 * m] + N, jy = mom[3 * m + 1] + N, jz = mom[3 * m + 2] + N;
    const long w3 = (long)W * W * W, at = ((long)jz * W + jy) * W + jx;
    cx<double> sh = {0, 0};
    if (G && blk < 3) {
        const double2 v = shift[blk * W + (blk == 0 ? jx : blk == 1 ? jy : jz)];
        sh = {v.x, v.y};
    }
    auto E = [&](int b, int a, int tt) {
        const double2 u = T[((long)(16 * blk + 4 * b + a) * Lt + tt) * w3 + at];
        if (!G) return cx<double>{u.x, u.y};
        const double2 w = G[((long)(16 * blk + 4 * a + b) * Lt + tt) * w3 + (w3 - 1 - at)];
        return cx<double>{u.x - w.x, u.y + w.y};
    };
    cx<double> acc = {0, 0};
    for (int a = 0; a < 4; a++)
        for (int b = 0; b < 4; b++) {
            cx<double> C = E(b, a, t);
            if (G) {
                if (blk < 3) {
                    cx<double> q = {0, 0};
                    cmac(q, sh, C);
                    C = q;
                } else {
                    C = C + E(b, a, t == 0 ? Lt - 1 : t - 1);
                }
                C = 0.25 * C;
            }
            const double2 X = c_ins.X[form][n][4 * a + b];
            acc = acc + cx<double>{X.x, X.y} * C;
        }
    acc = coef * acc;
    out[((long)m * n_ins + ins0 + 16 * blk + n) * Lt + t] = make_double2(acc.r, acc.i);
}

// e^{2 pi i (j - N) x / L} for j < W, x < L, reduced mod L in integers
std::vector<double2> phase_table(int L, int N)
{
    const int W = 2 * N + 1;
    std::vector<double2> ph((size_t)W * L);
    for (int j = 0; j < W; j++)
        for (int x = 0; x < L; x++) {
            const long k = (((long)(j - N) * x) % L + L) % L;
            const double a = 2.0 * M_PI * (double)k / (double)L;
            ph[(size_t)j * L + x] = make_double2(std::cos(a), std::sin(a));
        }
    return ph;
}

}  // namespace

std::vector<Momentum> momenta_list(int p2max)
{
    std::vector<Momentum> out;
    if (p2max < 0) return out;
    int N = 0;
    while ((N + 1) * (N + 1) <= p2max) N++;
    for (int n2 = 0; n2 <= p2max; n2++)
        for (int nx = -N; nx <= N; nx++)
            for (int ny = -N; ny <= N; ny++)
                for (int nz = -N; nz <= N; nz++)
                    if (nx * nx + ny * ny + nz * nz == n2) out.push_back(Momentum{{nx, ny, nz}});
    return out;
}

void check_momenta(tm_ctx *c, int p2max)
{
    TM_REQUIRE(p2max >= 0, "p2max must be >= 0");
    int N = 0;
    while ((N + 1) * (N + 1) <= p2max) N++;
    for (int mu = 0; mu < 3; mu++)
        TM_REQUIRE(2 * N < c->geo.L[mu], "momentum components must stay below L/2 in every spatial direction");
}

namespace {

// Tables of one projection on the device, uploaded together: phases of x, y,
// z, the shifts of k_insert and the momentum list
struct Tables {
    const double2 *px, *py, *pz, *shift;
    const int *mom;
    int N, W;
};
Tables upload_tables(tm_ctx *c, const std::vector<Momentum> &mom, hipStream_t s)
{
    const int *L = c->geo.L;
    Tables t{};
    for (const auto &m : mom)
        for (int d = 0; d < 3; d++) t.N = std::max(t.N, std::abs(m.n[d]));
    t.W = 2 * t.N + 1;
    std::vector<double2> all;
    for (int d = 0; d < 3; d++) {
        const std::vector<double2> ph = phase_table(L[d], t.N);
        all.insert(all.end(), ph.begin(), ph.end());
    }
    for (int d = 0; d < 3; d++)
        for (int j = -t.N; j <= t.N; j++) {
            const double h = M_PI * (double)j / (double)L[d], c = std::cos(h);
            all.push_back(make_double2(2.0 * c * c, std::sin(2.0 * h)));
        }
    const size_t nph = all.size(), nm = mom.size();
    all.resize(nph + (3 * nm * sizeof(int) + sizeof(double2) - 1) / sizeof(double2));
    int *ml = (int *)(all.data() + nph);
    for (size_t m = 0; m < nm; m++)
        for (int d = 0; d < 3; d++) ml[3 * m + d] = mom[m].n[d];
    double2 *dev = (double2 *)ws_get(c, "mom_tab", sizeof(double2) * all.size());
    upload(dev, all.data(), sizeof(double2) * all.size(), s);
    t.px = dev;
    t.py = t.px + (size_t)t.W * L[0];
    t.pz = t.py + (size_t)t.W * L[1];
    t.shift = t.pz + (size_t)t.W * L[2];
    t.mom = (const int *)(dev + nph);
    return t;
}

// Fourier sums [16 nblk][Lt][W][W][W] of the products of v and w
template <int KIND>
const double2 *fourier_sums(tm_ctx *c, const void *ve, const void *vo, const void *we, const void *wo, int nrhs,
                            const Tables &tb, const char *name, hipStream_t s)
{
    const Geo &g = c->geo;
    const int Lx = g.L[0], Ly = g.L[1], Lz = g.L[2], Lt = g.L[3], W = tb.W;
    constexpr int nblk = KIND == SITE_HOP ? 4 : 1;
    const long ncomp = 16L * nblk, nrow = (long)Ly * Lz * Lt;
    // x: [ncomp Lt Lz Ly][Lx] -> [ncomp Lt Lz Ly][W]
    double2 *T1 = (double2 *)ws_get(c, "mom_t1", sizeof(double2) * ncomp * nrow * W);
    const bool same = KIND == SITE_LOCAL && ve == we && vo == wo;
    auto launch = [&](auto kern, dim3 grid, size_t lds, auto... more) {
        hipLaunchKernelGGL(kern, grid, dim3(kBlock), lds, s, (const double2 *)ve, (const double2 *)vo,
                           (const double2 *)we, (const double2 *)wo, (const double2 *)c->links64[0],
                           (const double2 *)c->links64[1], g, more...);
        TM_HIP(hipGetLastError());
    };
    if (Lx <= kBlock) {
        const int rows = kBlock / Lx;
        const long per = ((nrow + rows - 1) / rows + 7) / 8;  // row groups per XCD
        TM_REQUIRE(8 * nblk * per <= 0x7fffffffL, "lattice too large for the contraction grid");
        launch(same ? k_site_rows<KIND, KIND == SITE_LOCAL> : k_site_rows<KIND, false>, dim3((unsigned)(8 * nblk * per)),
               sizeof(double2) * kPass * rows * (Lx + 1), nrhs, rows, nrow, per, tb.px, W, T1);
    } else {
        double2 *Cf = (double2 *)ws_get(c, "mom_cf", sizeof(double2) * ncomp * c->V);
        launch(same ? k_sites<KIND, KIND == SITE_LOCAL> : k_sites<KIND, false>,
               dim3((unsigned)((c->V + kBlock - 1) / kBlock), nblk), 0, c->V, nrhs, Cf);
        const long n1 = ncomp * nrow * W;
        hipLaunchKernelGGL(k_dft_dim<KIND>, dim3((unsigned)((n1 + kBlock - 1) / kBlock)), dim3(kBlock), 0, s,
                           (const double2 *)Cf, T1, tb.px, ncomp * nrow, Lx, W, 1L);
    }
    // y: [ncomp Lt Lz][Ly][W] -> [ncomp Lt Lz][W][W]
    const long o2 = ncomp * Lt * Lz;
    double2 *T2 = (double2 *)ws_get(c, "mom_t2", sizeof(double2) * o2 * W * W);
    const long n2 = o2 * W * W;
    hipLaunchKernelGGL(k_dft_dim<KIND>, dim3((unsigned)((n2 + kBlock - 1) / kBlock)), dim3(kBlock), 0, s,
                       (const double2 *)T1, T2, tb.py, o2, Ly, W, (long)W);
    // z: [ncomp Lt][Lz][W W] -> [ncomp Lt][W][W W]
    const long o3 = ncomp * Lt;
    double2 *T3 = (double2 *)ws_get(c, name, sizeof(double2) * o3 * W * W * W);
    const long n3 = o3 * W * W * W;
    hipLaunchKernelGGL(k_dft_dim<KIND>, dim3((unsigned)((n3 + kBlock - 1) / kBlock)), dim3(kBlock), 0, s,
                       (const double2 *)T2, T3, tb.pz, o3, Lz, W, (long)W * W);
    TM_HIP(hipGetLastError());
    return T3;
}

}  // namespace

void momentum_loops(tm_ctx *c, const void *ve, const void *vo, const void *we, const void *wo, int nrhs,
                    const std::vector<Momentum> &mom, GammaForm form, cx<double> coef, bool local, bool deriv,
                    cx<double> *out, hipStream_t s)
{
    TM_REQUIRE(!deriv || c->have_gauge, "no gauge field set");
    const int n_mom = (int)mom.size(), n_ins = (local ? 16 : 0) + (deriv ? 64 : 0);
    const size_t bytes = sizeof(double2) * n_mom * n_ins * c->geo.L[3];
    const Tables tb = upload_tables(c, mom, s);
    double2 *dev = (double2 *)ws_get(c, "mom_out", bytes);
    auto insert = [&](const double2 *T, const double2 *G, int nblk, int ins0) {
        const long n = 16L * n_mom * nblk * c->geo.L[3];
        hipLaunchKernelGGL(k_insert, dim3((unsigned)((n + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, T, G, tb.mom,
                           n_mom, nblk, c->geo, tb.W, tb.N, tb.shift, (int)form, coef, n_ins, ins0, dev);
        TM_HIP(hipGetLastError());
    };
    if (local) insert(fourier_sums<SITE_LOCAL>(c, ve, vo, we, wo, nrhs, tb, "mom_t3", s), nullptr, 1, 0);
    if (deriv) {
        const double2 *F = fourier_sums<SITE_HOP>(c, ve, vo, we, wo, nrhs, tb, "mom_t3", s), *G = F;
        if (ve != we || vo != wo) G = fourier_sums<SITE_HOP>(c, we, wo, ve, vo, nrhs, tb, "mom_t3g", s);
        insert(F, G, 4, local ? 16 : 0);
    }
    download(c, out, dev, bytes, s);
}
