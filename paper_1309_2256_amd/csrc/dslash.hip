// Even-odd twisted-mass hopping kernel for gfx950.
//
// A block of four waves takes 64 output half-sites and up to `rpb` right-hand
// sides, one after the other.  Wave mu holds the two links of direction mu
// (x + mu and x - mu) of its 64 sites in registers for all of them.  Per
// right-hand side it loads the two neighbour spinors, projects each to a
// 2-spinor with (1 -+ gamma_mu) (chiral basis, appendix A.1 operator),
// multiplies by the colour link and leaves the result in LDS.  Three of the
// waves then each sum one colour over the eight directions in fixed order,
// rebuild the four spins and apply the spin-diagonal local terms (twist R =
// 1 + i eps gamma5, its inverse, gamma5, -kappa), so that the fused forms
// R^-1 H and R x - H y of the Schur operator (eq. A.2) cost no extra memory
// pass.
//
// What bounds it, and why this split (32^3 x 64, 12 right-hand sides, R^-1 H,
// against one thread per site walking the eight directions with 1-4
// right-hand sides): the misses of the 4 MB L2 of each XCD.  A block is short
// lived and its four directions' loads are in flight together, so the blocks
// resident at a time cover a quarter of the sites and meet their neighbours'
// spinors in the L2, and the links are loaded and rebuilt once for all
// right-hand sides.  FP16: 533 -> 459 us, 2.26 -> 1.59 GB fetched past the L2;
// FP64: 2449 -> 1780 us, 15.6 -> 10.2 GB (7.1 TB/s with the writes, what the
// memory side cache gives); FP32 1285 -> 982, BF16 617 -> 509 us.  On small
// lattices the serial chain of a thread is two directions and an LDS exchange
// instead of eight directions: 16^3 x 32, one right-hand side, FP16 8.6 -> 7.1,
// FP64 15.0 -> 14.2 us.
//
// Memory layout (all coalesced over the half-site index i):
//   spinors  [rhs][spin*3 + colour][hs] (hs >= vh, the padded plane stride)
//   links    [direction 0..7][row*3 + col][vh] for the output parity; the
//            backward links are stored conjugated and the antiperiodic
//            boundary phase is folded in, so the kernel has no branch on it.
#include <cmath>
#include <cstdlib>
#include <cstring>

#include "cg_device.h"

namespace {

constexpr int kBlock = 256;  // four waves, one per direction mu
constexpr int kSites = 64;   // output half-sites of a block
// resident blocks per CU (and waves per SIMD) requested from the compiler:
// bounded by the LDS exchange (24 KB per block in FP32, 48 KB in FP64, of
// 160 KB) and by the registers (512 / waves per lane).  FP16 spinors, 32^3 x 64,
// 12 right-hand sides: normal operator 2026 us with five, 1974 with six.  FP32
// and BF16 spill with five; BF16 with one right-hand side per block, which does
// not hold the links, fits six.
template <typename SS, typename LS, typename T, bool ONE = false>
constexpr int waves_for()
{
    if (sizeof(T) == 8) return ONE && !std::is_same<LS, L8D>::value ? 4 : 3;
    if (std::is_same<SS, float2>::value || std::is_same<LS, float2>::value) return 4;
    return std::is_same<SS, h2>::value || ONE ? 6 : 4;
}

// 16-byte aligned so that an array of records keeps every complex field
// naturally aligned
template <typename T>
struct alignas(16) DParams {
    void *out;
    const void *in;
    const void *own;
    const void *links;
    Geo g;
    int p;          // output parity
    int nrhs;
    int rpb;        // right-hand sides per block
    int alpha;      // see DslashCall; -1: its beta
    int ngroups;    // right-hand-side groups, ceil(nrhs / rpb)
    cx<T> own_u, own_l, hop_u, hop_l;
    // +1, passed at run time so that the +-1 factors of the spin projection
    // stay FMAs (which take the FP16 inputs directly) instead of being folded
    // into adds that need separate conversions
    T one;
    // fused epilogues: partial sums [quantity][rhs][site block]
    void *r;        // EPI_CG: normal residual, updated in place; EPI_RES: b
    union {
        void *rho;     // EPI_CG: Schur residual, updated in place
        double delta;  // beta step: threshold of the reliable updates
    };
    const CGScalars *sc;
    double *part;
    int nblk;       // site blocks
    int nb_t;       // site blocks per time slice (tiled traversal) or 0
    int t_bc;       // time-boundary factor (rebuilds the third row of 12-parameter links)
};

// Block -> (site block, right-hand-side group).  Hardware dispatches
// workgroup b to XCD b % 8.  Tiled traversal (when each time slice is a
// whole number of site blocks and of 8-block spatial chunks): XCD k owns the
// k-th eighth of every time slice and walks t slowest, so a site's t +- 1
// neighbours were loaded about eight site blocks earlier / later on the same
// XCD (its L2), z +- 1 two blocks away; the right-hand-side groups sharing a
// site block (and its links) are adjacent.  Otherwise: contiguous chunks of
// the natural order per XCD.
__device__ __forceinline__ int map_block(int b, int nblk_hw, int ngroups, int nb_t, int &grp)
{
    if (nb_t) {
        const int k = b & 7, m = b >> 3;
        grp = m % ngroups;
        const int m2 = m / ngroups, w = nb_t >> 3;
        const int t = m2 / w;
        return t * nb_t + k * w + (m2 - t * w);
    }
    const int lb = xcd_block(b, nblk_hw);
    grp = lb % ngroups;
    return lb / ngroups;
}

// A stored complex value as loaded: components in the storage type (FP16
// stays FP16 so that the projection below folds the conversion into a
// mixed-precision FMA), converted to T where they are combined.
template <typename L>
struct rawc {
    L r, i;
};

// h = u + S*l, h = u + S*i*l and h = u - S*i*l in arithmetic type T, each real
// part one FMA on the raw stored components
template <typename T, typename L>
__device__ __forceinline__ cx<T> p_add(rawc<L> u, rawc<L> l, T s)
{
    return {fma(s, (T)l.r, (T)u.r), fma(s, (T)l.i, (T)u.i)};
}
template <typename T, typename L>
__device__ __forceinline__ cx<T> p_addi(rawc<L> u, rawc<L> l, T s)
{
    return {fma(-s, (T)l.i, (T)u.r), fma(s, (T)l.r, (T)u.i)};
}

// Hop of one direction, (1 - S gamma_MU) (W (x) 1) psi for S = +1 or -1, in
// the half-spinor form: h = P psi (two spins), w = W h, the lower spins
// rebuilt from w (see rebuild).
// gamma_k = [[0, -i s_k], [i s_k, 0]]:  h = u + S (i s_k) l,  lower = -S (i s_k) w
// gamma_4 = [[0, 1], [1, 0]]:           h = u - S l,          lower = -S w
// with i s_1 = [[0, i], [i, 0]], i s_2 = [[0, 1], [-1, 0]], i s_3 = [[i, 0], [0, -i]].
// psi[3*spin + colour]; u = spins 0, 1 and l = spins 2, 3.
// acc += a * b for a link entry kept as stored binary16 (the conversion folds
// into mixed-precision FMAs) or already converted
template <typename T>
__device__ __forceinline__ void lmac(cx<T> &acc, cx<T> a, cx<T> b) { cmac(acc, a, b); }
template <typename T>
__device__ __forceinline__ void lmac(cx<T> &acc, rawc<_Float16> a, cx<T> b)
{
    acc.r = fma((T)a.r, b.r, acc.r);
    acc.r = fma(-(T)a.i, b.i, acc.r);
    acc.i = fma((T)a.r, b.i, acc.i);
    acc.i = fma((T)a.i, b.r, acc.i);
}

// Component A (0 or 1) of the half-spinor takes u = spin A and l = spin
// kLower<MU, A>.
template <int MU, int A>
constexpr int kLower = MU < 2 ? 3 - A : 2 + A;
template <int MU, int S, int A, typename T, typename L, typename WT>
__device__ __forceinline__ void half_hop_comp(cx<T> w[3], const WT W[9], const rawc<L> u[3], const rawc<L> l[3], T one)
{
    const T s = (T)S * one;
    cx<T> h[3];
#pragma unroll
    for (int c = 0; c < 3; c++) {
        if (MU == 0)        // h0 = u0 + S i l1, h1 = u1 + S i l0
            h[c] = p_addi(u[c], l[c], s);
        else if (MU == 1)   // h0 = u0 + S l1,   h1 = u1 - S l0
            h[c] = p_add(u[c], l[c], A ? -s : s);
        else if (MU == 2)   // h0 = u0 + S i l0, h1 = u1 - S i l1
            h[c] = p_addi(u[c], l[c], A ? -s : s);
        else                // h0 = u0 - S l0,   h1 = u1 - S l1
            h[c] = p_add(u[c], l[c], -s);
    }
#pragma unroll
    for (int r = 0; r < 3; r++) {
        w[r] = {0, 0};
#pragma unroll
        for (int c = 0; c < 3; c++) lmac(w[r], W[3 * r + c], h[c]);
    }
}
template <int MU, int S, typename T, typename L, typename WT>
__device__ __forceinline__ void half_hop(cx<T> w0[3], cx<T> w1[3], const WT W[9], const rawc<L> psi[12], T one)
{
    half_hop_comp<MU, S, 0>(w0, W, psi, psi + 3 * kLower<MU, 0>, one);
    half_hop_comp<MU, S, 1>(w1, W, psi + 3, psi + 3 * kLower<MU, 1>, one);
}

// acc[spin] += the four spins of one colour of a hop, from its half-spinor
// (w0, w1).  The rounding is that of one add per component, whatever the
// instantiation.
template <int MU, int S, typename T>
__device__ __forceinline__ void rebuild(cx<T> acc[4], cx<T> w0, cx<T> w1)
{
    acc[0] = acc[0] + w0;
    acc[1] = acc[1] + w1;
    auto add = [](cx<T> &a, bool plus, cx<T> w) { a = plus ? a + w : a - w; };
    const cx<T> iw0 = times_i(w0), iw1 = times_i(w1);
    if (MU == 0) {          // lower = -S (i w1, i w0)
        add(acc[2], S < 0, iw1);
        add(acc[3], S < 0, iw0);
    } else if (MU == 1) {   // lower = -S (w1, -w0)
        add(acc[2], S < 0, w1);
        add(acc[3], S > 0, w0);
    } else if (MU == 2) {   // lower = -S (i w0, -i w1)
        add(acc[2], S < 0, iw0);
        add(acc[3], S > 0, iw1);
    } else {                // lower = -S (w0, w1)
        add(acc[2], S < 0, w0);
        add(acc[3], S < 0, w1);
    }
}

// ---------------------------------------------------------------- buffer I/O
// Raw buffer loads/stores: the 128-bit resource descriptor (base, byte range)
// lives in SGPRs, each lane supplies a 32-bit byte offset and the component
// stride is a scalar offset, so a neighbour costs one VGPR of address state.
using rsrc_t = __amdgpu_buffer_rsrc_t;
typedef _Float16 hv2 __attribute__((ext_vector_type(2)));
// the builtins' own (GCC-style) vector types; values are moved in and out by
// bit_cast to plain structs (element access on these vectors lowers to a
// single-dword load with this compiler)
typedef unsigned v2u __attribute__((__vector_size__(2 * sizeof(unsigned))));
typedef unsigned v4u __attribute__((__vector_size__(4 * sizeof(unsigned))));
// descriptor word 3 for raw (untyped) access on gfx9-class parts
constexpr int kRsrcFlags = 0x00020000;
// cache-policy operand of the output stores: non-temporal (streaming) hint,
// outputs are not re-read by this launch.  Links are loaded with the default
// policy: the right-hand-side groups of a site block (adjacent workgroups on
// one XCD) read them again, and a streaming hint on them raised the fetched
// bytes by a quarter.
constexpr int kNT = 2;

__device__ __forceinline__ rsrc_t make_rsrc(const void *base, size_t bytes)
{
    const unsigned n = bytes >= 0xffffffffull ? 0xffffffffu : (unsigned)bytes;
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), (short)0, (int)n, kRsrcFlags);
}

template <typename S>
struct BufIO;
// component type of a raw load
template <typename S>
struct RawT {
    using L = float;
};
template <>
struct RawT<double2> {
    using L = double;
};
template <>
struct RawT<h2> {
    using L = _Float16;
};
struct F2 {
    float x, y;
};
struct D2 {
    double x, y;
};
template <>
struct BufIO<double2> {
    template <typename T>
    __device__ __forceinline__ static cx<T> ld(rsrc_t r, int voff, int soff)
    {
        D2 v = __builtin_bit_cast(D2, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0));
        return {(T)v.x, (T)v.y};
    }
    template <typename T>
    __device__ __forceinline__ static cx<T> ldlink(rsrc_t r, int voff, int soff)
    {
        D2 v = __builtin_bit_cast(D2, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0));
        return {(T)v.x, (T)v.y};
    }
    __device__ __forceinline__ static rawc<double> ldraw(rsrc_t r, int voff, int soff)
    {
        D2 v = __builtin_bit_cast(D2, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0));
        return {v.x, v.y};
    }
    template <typename T>
    __device__ __forceinline__ static void st(rsrc_t r, int voff, int soff, cx<T> c)
    {
        // 16-byte stores take the whole offset in the VGPR: with an SGPR
        // offset the compiler lets the next instruction overwrite the data
        // registers, and the last lanes then stored the new value (seen on
        // this chip; with a constant offset it keeps the needed wait state)
        D2 v{(double)c.r, (double)c.i};
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, v), r, voff + soff, 0, kNT);
    }
};
template <>
struct BufIO<float2> {
    template <typename T>
    __device__ __forceinline__ static cx<T> ld(rsrc_t r, int voff, int soff)
    {
        F2 v = __builtin_bit_cast(F2, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
        return {(T)v.x, (T)v.y};
    }
    template <typename T>
    __device__ __forceinline__ static cx<T> ldlink(rsrc_t r, int voff, int soff)
    {
        F2 v = __builtin_bit_cast(F2, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
        return {(T)v.x, (T)v.y};
    }
    __device__ __forceinline__ static rawc<float> ldraw(rsrc_t r, int voff, int soff)
    {
        F2 v = __builtin_bit_cast(F2, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
        return {v.x, v.y};
    }
    template <typename T>
    __device__ __forceinline__ static void st(rsrc_t r, int voff, int soff, cx<T> c)
    {
        F2 v{(float)c.r, (float)c.i};
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(v2u, v), r, voff, soff, kNT);
    }
};
template <>
struct BufIO<h2> {
    template <typename T>
    __device__ __forceinline__ static cx<T> ld(rsrc_t r, int voff, int soff)
    {
        unsigned v = __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0);
        h2 h = __builtin_bit_cast(h2, v);
        return {(T)(float)h.x, (T)(float)h.y};
    }
    __device__ __forceinline__ static rawc<_Float16> ldraw(rsrc_t r, int voff, int soff)
    {
        h2 h = __builtin_bit_cast(h2, __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
        return {h.x, h.y};
    }
    template <typename T>
    __device__ __forceinline__ static void st(rsrc_t r, int voff, int soff, cx<T> c)
    {
        // one packed conversion (v_cvt_pk_f16_f32, round to nearest even)
        const hv2 h = {(_Float16)(float)c.r, (_Float16)(float)c.i};
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, h), r, voff, soff, kNT);
    }
};
template <>
struct BufIO<b2> {
    template <typename T>
    __device__ __forceinline__ static cx<T> ld(rsrc_t r, int voff, int soff)
    {
        unsigned v = __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0);
        return {(T)__builtin_bit_cast(float, v << 16), (T)__builtin_bit_cast(float, v & 0xffff0000u)};
    }
    __device__ __forceinline__ static rawc<float> ldraw(rsrc_t r, int voff, int soff)
    {
        unsigned v = __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0);
        return {__builtin_bit_cast(float, v << 16), __builtin_bit_cast(float, v & 0xffff0000u)};
    }
    template <typename T>
    __device__ __forceinline__ static void st(rsrc_t r, int voff, int soff, cx<T> c)
    {
        __builtin_amdgcn_raw_buffer_store_b32(bf16_pair((float)c.r, (float)c.i), r, voff, soff, kNT);
    }
};

// link entry as held in registers: binary16 links stay binary16 (converted
// inside the FMAs), FP32/FP64 links and rebuilt 12-parameter links in the
// arithmetic type
template <typename LS, typename T>
struct LinkEl {
    using type = cx<T>;
};
template <typename T>
struct LinkEl<h2, T> {
    using type = rawc<_Float16>;
};

template <typename LS, typename T>
__device__ __forceinline__ void load_link(typename LinkEl<LS, T>::type W[9], rsrc_t lr, int vbytes, int voff)
{
#pragma unroll
    for (int k = 0; k < 9; k++) {
        if constexpr (std::is_same<LS, h2>::value)
            W[k] = BufIO<h2>::ldraw(lr, voff, k * vbytes);
        else
            W[k] = BufIO<LS>::template ldlink<T>(lr, voff, k * vbytes);
    }
}

// 12-parameter link (appendix A.1, link reconstruction): the first two rows in
// binary16, [8 directions][6][vh]; the third row of a special unitary matrix
// is the complex conjugate of the cross product of the first two.  The stored
// rows carry the time-boundary factor f = +-1, which cancels in the cross
// product (f^2 = 1), so the rebuilt row is multiplied by f again on links
// that cross the boundary.
template <typename RS, typename T>
__device__ __forceinline__ void load_link12(cx<T> W[9], rsrc_t lr, int vbytes, int voff, bool cross, T tbc)
{
#pragma unroll
    for (int k = 0; k < 6; k++) {
        if constexpr (std::is_same<RS, h2>::value) {
            const rawc<_Float16> w = BufIO<h2>::ldraw(lr, voff, k * vbytes);
            W[k] = {(T)w.r, (T)w.i};
        } else {
            W[k] = BufIO<RS>::template ldlink<T>(lr, voff, k * vbytes);
        }
    }
    // conj(a b - c d) for each entry of row0 x row1
    auto cr = [](cx<T> a, cx<T> b, cx<T> c, cx<T> d) {
        T re = a.r * b.r;
        re = fma(-a.i, b.i, re);
        re = fma(-c.r, d.r, re);
        re = fma(c.i, d.i, re);
        T im = a.r * b.i;
        im = fma(a.i, b.r, im);
        im = fma(-c.r, d.i, im);
        im = fma(-c.i, d.r, im);
        return cx<T>{re, -im};
    };
    W[6] = cr(W[1], W[5], W[2], W[4]);
    W[7] = cr(W[2], W[3], W[0], W[5]);
    W[8] = cr(W[0], W[4], W[1], W[3]);
    if (cross) {
#pragma unroll
        for (int k = 6; k < 9; k++) W[k] = {tbc * W[k].r, tbc * W[k].i};
    }
}

// 8-parameter FP64 link (appendix A.1; stored form in misc.hip): |a1| and
// |c1| from the unit first row and column, their phases from the stored
// angles, the 2x2 block from the cofactor relations conj(U) = cof(U):
//   b2 = -(conj(a1) a2 b1 + conj(c1) conj(a3)) / n,  b3 = (conj(a2) conj(c1) - conj(a1) a3 b1) / n,
//   c2 = (conj(a3) conj(b1) - conj(a1) a2 c1) / n,   c3 = -(conj(a2) conj(b1) + conj(a1) a3 c1) / n,
// n = |a2|^2 + |a3|^2; rows swapped and negated back for links stored that
// way (phase flag), then the time-boundary factor on crossing links
template <typename T>
__device__ __forceinline__ void load_link8(cx<T> W[9], rsrc_t lr, int vbytes, int voff, bool cross, T tbc)
{
    const cx<T> a2 = BufIO<double2>::template ldlink<T>(lr, voff, 0);
    const cx<T> a3 = BufIO<double2>::template ldlink<T>(lr, voff, vbytes);
    const cx<T> b1 = BufIO<double2>::template ldlink<T>(lr, voff, 2 * vbytes);
    const cx<T> ph = BufIO<double2>::template ldlink<T>(lr, voff, 3 * vbytes);
    const bool swap = ph.i > (T)4;
    const T tc = swap ? ph.i - (T)8 : ph.i;
    const T n = a2.r * a2.r + a2.i * a2.i + a3.r * a3.r + a3.i * a3.i;
    const T ra = sqrt((T)1 - n), rc = sqrt(fmax(n - (b1.r * b1.r + b1.i * b1.i), (T)0));
    T sa, ca, sc, cc;
    sincos(ph.r, &sa, &ca);
    sincos(tc, &sc, &cc);
    const cx<T> a1 = {ra * ca, ra * sa}, c1 = {rc * cc, rc * sc};
    const T inv = (T)1 / n;
    const cx<T> ab = conjg(a1) * b1, ac = conjg(a1) * c1;
    const cx<T> a2c = conjg(a2), a3c = conjg(a3), b1c = conjg(b1), c1c = conjg(c1);
    const cx<T> b2 = (ab * a2 + c1c * a3c) * cx<T>{-inv, 0};
    const cx<T> b3 = (a2c * c1c - ab * a3) * cx<T>{inv, 0};
    const cx<T> c2 = (a3c * b1c - ac * a2) * cx<T>{inv, 0};
    const cx<T> c3 = (a2c * b1c + ac * a3) * cx<T>{-inv, 0};
    const cx<T> m[9] = {a1, a2, a3, b1, b2, b3, c1, c2, c3};
    const T g = (swap ? (T)-1 : (T)1) * (cross ? tbc : (T)1);
#pragma unroll
    for (int k = 0; k < 3; k++) {
        W[k] = {g * m[k].r, g * m[k].i};
        const cx<T> r1 = swap ? m[6 + k] : m[3 + k], r2 = swap ? m[3 + k] : m[6 + k];
        W[3 + k] = {g * r1.r, g * r1.i};
        W[6 + k] = {g * r2.r, g * r2.i};
    }
}

// ------------------------------------------------ FP16 spinors, binary16 links
// Packed form of the hop for IEEE binary16 spinors and links: the spin
// projection h = u + a l (a = +-1, +-i) is one packed binary16 add per
// complex value, producing h in the two arrangements the colour product
// needs, conj(h) = (h.r, -h.i) and swap(h) = (h.i, h.r); each complex
// multiply-add of the 3x3 link product is then two v_dot2_f32_f16
//   Re(w h) += w.r h.r - w.i h.i = dot2(w, conj h),
//   Im(w h) += w.r h.i + w.i h.r = dot2(w, swap h),
// whose binary16 products are exact and whose sums are FP32.  Relative to
// the FP32 projection this rounds h once to binary16 (the storage precision
// of its inputs); all accumulation stays FP32.

// h = u + SG l (I = false) or u + SG i l (I = true), as (conj h, swap h):
// each one v_pk_add_f16 whose operand selection (op_sel: which half of each
// source feeds the low result, op_sel_hi: the high result) and negation
// modifiers (neg_lo, neg_hi: negate that source's value in the low / high
// result) form the arrangement, written out so that no separate swap or
// sign instruction is generated.  With u = (ur, ui), l = (lr, li):
//   real, SG > 0:  conj = (ur + lr, -ui - li)   swap = (ui + li, ur + lr)
//   real, SG < 0:  conj = (ur - lr, -ui + li)   swap = (ui - li, ur - lr)
//   i,    SG > 0:  conj = (ur - li, -ui - lr)   swap = (ui + lr, ur - li)
//   i,    SG < 0:  conj = (ur + li, -ui + lr)   swap = (ui - lr, ur + li)
template <bool I, int SG>
__device__ __forceinline__ void proj2(hv2 u, hv2 l, hv2 &hc, hv2 &hs)
{
    if constexpr (!I && SG > 0) {
        asm("v_pk_add_f16 %0, %1, %2 neg_hi:[1,1]" : "=v"(hc) : "v"(u), "v"(l));
        asm("v_pk_add_f16 %0, %1, %2 op_sel:[1,1] op_sel_hi:[0,0]" : "=v"(hs) : "v"(u), "v"(l));
    } else if constexpr (!I) {
        asm("v_pk_add_f16 %0, %1, %2 neg_lo:[0,1] neg_hi:[1,0]" : "=v"(hc) : "v"(u), "v"(l));
        asm("v_pk_add_f16 %0, %1, %2 op_sel:[1,1] op_sel_hi:[0,0] neg_lo:[0,1] neg_hi:[0,1]"
            : "=v"(hs) : "v"(u), "v"(l));
    } else if constexpr (SG > 0) {
        asm("v_pk_add_f16 %0, %1, %2 op_sel:[0,1] op_sel_hi:[1,0] neg_lo:[0,1] neg_hi:[1,1]"
            : "=v"(hc) : "v"(u), "v"(l));
        asm("v_pk_add_f16 %0, %1, %2 op_sel:[1,0] op_sel_hi:[0,1] neg_hi:[0,1]" : "=v"(hs) : "v"(u), "v"(l));
    } else {
        asm("v_pk_add_f16 %0, %1, %2 op_sel:[0,1] op_sel_hi:[1,0] neg_hi:[1,0]" : "=v"(hc) : "v"(u), "v"(l));
        asm("v_pk_add_f16 %0, %1, %2 op_sel:[1,0] op_sel_hi:[0,1] neg_lo:[0,1]" : "=v"(hs) : "v"(u), "v"(l));
    }
}

// The four chains of one link row W (three entries) with both half-spinor
// components: Re and Im of W h0 and of W h1, each three v_dot2_f32_f16 from
// zero.  One block of assembly, since the compiler starts a chain by clearing
// a register (a tenth of the kernel's instructions) and since no instruction
// but another dot of the same kind (as its addend) may read the result of a
// dot for three wait states: the compiler keeps that distance only between
// instructions that it knows, so the block ends with the wait.
__device__ __forceinline__ void row_dots(float &ar, float &ai, float &br, float &bi, const hv2 *W, const hv2 *c0,
                                         const hv2 *s0, const hv2 *c1, const hv2 *s1)
{
    asm("v_dot2_f32_f16 %0, %4, %7, 0\n\t"
        "v_dot2_f32_f16 %1, %4, %10, 0\n\t"
        "v_dot2_f32_f16 %2, %4, %13, 0\n\t"
        "v_dot2_f32_f16 %3, %4, %16, 0\n\t"
        "v_dot2_f32_f16 %0, %5, %8, %0\n\t"
        "v_dot2_f32_f16 %1, %5, %11, %1\n\t"
        "v_dot2_f32_f16 %2, %5, %14, %2\n\t"
        "v_dot2_f32_f16 %3, %5, %17, %3\n\t"
        "v_dot2_f32_f16 %0, %6, %9, %0\n\t"
        "v_dot2_f32_f16 %1, %6, %12, %1\n\t"
        "v_dot2_f32_f16 %2, %6, %15, %2\n\t"
        "v_dot2_f32_f16 %3, %6, %18, %3\n\t"
        "s_nop 2"
        : "=&v"(ar), "=&v"(ai), "=&v"(br), "=&v"(bi)
        : "v"(W[0]), "v"(W[1]), "v"(W[2]), "v"(c0[0]), "v"(c0[1]), "v"(c0[2]), "v"(s0[0]), "v"(s0[1]), "v"(s0[2]),
          "v"(c1[0]), "v"(c1[1]), "v"(c1[2]), "v"(s1[0]), "v"(s1[1]), "v"(s1[2]));
}

template <int MU, int S>
__device__ __forceinline__ void half_hop(cx<float> w0[3], cx<float> w1[3], const hv2 W[9], const hv2 psi[12], float)
{
    hv2 c0[3], s0[3], c1[3], s1[3];
#pragma unroll
    for (int c = 0; c < 3; c++) {
        const hv2 u0 = psi[c], u1 = psi[3 + c], l0 = psi[6 + c], l1 = psi[9 + c];
        if (MU == 0) {          // h0 = u0 + S i l1, h1 = u1 + S i l0
            proj2<true, S>(u0, l1, c0[c], s0[c]);
            proj2<true, S>(u1, l0, c1[c], s1[c]);
        } else if (MU == 1) {   // h0 = u0 + S l1,   h1 = u1 - S l0
            proj2<false, S>(u0, l1, c0[c], s0[c]);
            proj2<false, -S>(u1, l0, c1[c], s1[c]);
        } else if (MU == 2) {   // h0 = u0 + S i l0, h1 = u1 - S i l1
            proj2<true, S>(u0, l0, c0[c], s0[c]);
            proj2<true, -S>(u1, l1, c1[c], s1[c]);
        } else {                // h0 = u0 - S l0,   h1 = u1 - S l1
            proj2<false, -S>(u0, l0, c0[c], s0[c]);
            proj2<false, -S>(u1, l1, c1[c], s1[c]);
        }
    }
#pragma unroll
    for (int r = 0; r < 3; r++)
        row_dots(w0[r].r, w0[r].i, w1[r].r, w1[r].i, W + 3 * r, c0, s0, c1, s1);
}

__device__ __forceinline__ hv2 ld_hv2(rsrc_t r, int voff, int soff)
{
    return __builtin_bit_cast(hv2, __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
}

// binary16 link as nine packed entries; the 12-parameter form rebuilds the
// third row conj(row0 x row1) with dot2 products (exact binary16 products,
// FP32 sums) rounded once to binary16, times the time-boundary factor on
// links that cross the boundary
template <bool REC>
__device__ __forceinline__ void load_link_h(hv2 W[9], rsrc_t lr, int vbytes, int voff, bool cross, float tbc)
{
    if constexpr (!REC) {
#pragma unroll
        for (int k = 0; k < 9; k++) W[k] = ld_hv2(lr, voff, k * vbytes);
    } else {
#pragma unroll
        for (int k = 0; k < 6; k++) W[k] = ld_hv2(lr, voff, k * vbytes);
        // conj(a b - c d): Re(a b) = dot2(a, conj b), Im(a b) = dot2(a, swap b)
        auto cr = [](hv2 a, hv2 b, hv2 c, hv2 d) {
            const hv2 nc = -c;
            const float re = __builtin_amdgcn_fdot2(nc, hv2{d.x, -d.y}, __builtin_amdgcn_fdot2(a, hv2{b.x, -b.y}, 0.f, false), false);
            const float im = __builtin_amdgcn_fdot2(nc, hv2{d.y, d.x}, __builtin_amdgcn_fdot2(a, hv2{b.y, b.x}, 0.f, false), false);
            return hv2{(_Float16)re, (_Float16)(-im)};
        };
        W[6] = cr(W[1], W[5], W[2], W[4]);
        W[7] = cr(W[2], W[3], W[0], W[5]);
        W[8] = cr(W[0], W[4], W[1], W[3]);
        if (cross) {
            const _Float16 f = (_Float16)tbc;
#pragma unroll
            for (int k = 6; k < 9; k++) W[k] = W[k] * f;
        }
    }
}

// how an instantiation holds links and spinors: FP16 spinors with binary16
// links in the packed form, everything else as components
template <typename SS, typename LS, typename T>
struct Held {
    static constexpr bool packed =
        std::is_same<SS, h2>::value && (std::is_same<LS, L12>::value || std::is_same<LS, h2>::value);
    using Link = std::conditional_t<packed, hv2, typename LinkEl<LS, T>::type>;
    using Spinor = std::conditional_t<packed, hv2, rawc<typename RawT<SS>::L>>;
};

// the link of direction dir (uniform) at half-site i; cross: the link crosses
// the time boundary
template <typename SS, typename LS, typename T>
__device__ __forceinline__ void load_dir_link(typename Held<SS, LS, T>::Link W[9], const DParams<T> &a, int dir, int i,
                                              bool cross)
{
    constexpr bool rec = std::is_same<LS, L12>::value || std::is_same<LS, L12D>::value || std::is_same<LS, L12F>::value;
    constexpr int np = std::is_same<LS, L8D>::value ? 4 : rec ? 6 : 9;
    using RS = std::conditional_t<std::is_same<LS, L12>::value, h2,
                                  std::conditional_t<std::is_same<LS, L12D>::value || std::is_same<LS, L8D>::value,
                                                     double2, std::conditional_t<std::is_same<LS, L12F>::value, float2, LS>>>;
    const RS *base = (const RS *)a.links + (size_t)dir * np * a.g.vh;
    const rsrc_t lr = make_rsrc(base, (size_t)np * a.g.vh * sizeof(RS));
    const int vb = a.g.vh * (int)sizeof(RS), vo = i * (int)sizeof(RS);
    if constexpr (Held<SS, LS, T>::packed)
        load_link_h<rec>(W, lr, vb, vo, cross, (float)a.t_bc);
    else if constexpr (std::is_same<LS, L8D>::value)
        load_link8<T>(W, lr, vb, vo, cross, (T)a.t_bc);
    else if constexpr (rec)
        load_link12<RS, T>(W, lr, vb, vo, cross, (T)a.t_bc);
    else
        load_link<LS, T>(W, lr, vb, vo);
}

template <typename SS, typename LS, typename T>
__device__ __forceinline__ void load_dir_spinor(typename Held<SS, LS, T>::Spinor psi[12], rsrc_t sr, int vb, int vo)
{
#pragma unroll
    for (int k = 0; k < 12; k++) {
        if constexpr (Held<SS, LS, T>::packed)
            psi[k] = ld_hv2(sr, vo, k * vb);
        else
            psi[k] = BufIO<SS>::ldraw(sr, vo, k * vb);
    }
}

// the spinor components that half-spinor component A of a hop along MU takes:
// spin A, then spin kLower<MU, A>
template <typename SS, int MU, int A, typename L>
__device__ __forceinline__ void load_half_spinor(rawc<L> p[6], rsrc_t sr, int vb, int vo)
{
#pragma unroll
    for (int c = 0; c < 3; c++) {
        p[c] = BufIO<SS>::ldraw(sr, vo, (3 * A + c) * vb);
        p[3 + c] = BufIO<SS>::ldraw(sr, vo, (3 * kLower<MU, A> + c) * vb);
    }
}

// value as stored in precision SS (what later kernels will read)
template <typename SS, typename T>
__device__ __forceinline__ cx<T> stored(cx<T> v)
{
    if constexpr (std::is_same<SS, double2>::value) {
        return v;
    } else if constexpr (std::is_same<SS, float2>::value) {
        return {(T)(float)v.r, (T)(float)v.i};
    } else if constexpr (std::is_same<SS, h2>::value) {
        return {(T)(float)(_Float16)(float)v.r, (T)(float)(_Float16)(float)v.i};
    } else {
        const b2 s = __builtin_bit_cast(b2, bf16_pair((float)v.r, (float)v.i));
        return {(T)bf16_to_f32(s.x), (T)bf16_to_f32(s.y)};
    }
}

template <typename T>
__device__ __forceinline__ double norm2c(cx<T> v)
{
    return (double)(v.r * v.r + v.i * v.i);
}

// Epilogue forms:
//   EPI_STORE  out = D_hop Hop[in] (+ D_own own)
//   EPI_NORM   as EPI_STORE, plus per-block partial |out|^2 per right-hand side
//   EPI_CG     s = D_hop Hop[in] + D_own q (own = q); then r -= alpha s,
//              rho -= alpha q in place (s is never stored), partial |r|^2 and
//              |rho|^2 -- the last half of Ahat^dag q fused with the CG updates;
//              rho = null: r only (the solver follows |rho|^2 by recurrence)
//   EPI_RES    out = b - (D_hop Hop[in] + D_own own) with b in `r`, partial
//              |out|^2; out = null: the norm only (exact links only).  Saves
//              the pass b - v (1.5 ms in FP64, 32^3 x 64, 12 right-hand sides)
//              and that of the norm (0.4 ms)
enum { EPI_STORE = 0, EPI_NORM = 1, EPI_CG = 2, EPI_RES = 3 };

// The half-spinors (w0, w1) of a right-hand side on their way from the wave
// of their direction to the wave of their colour.  KEEP: wave mu < 3, which
// sums colour mu itself, keeps that colour of its own two directions in
// registers, and 18 of the 24 (direction, colour) pairs go through LDS: four
// FP64 blocks fit a CU then instead of three.
template <typename T, bool KEEP>
struct Exchange {
    static constexpr int slots = KEEP ? 18 : 24;
    // first slot of a direction; colour c of direction dir is first(dir) + c,
    // without the kept colour
    static constexpr int first(int dir)
    {
        const int mu = dir & 3, half = dir >> 2;
        return !KEEP ? 3 * dir : mu < 3 ? 4 * mu + 2 * half : 12 + 3 * half;
    }
    // (w0, w1): one 16-byte access in FP32, one each in FP64
    alignas(16) cx<T> w[sizeof(T) == 4 ? 1 : 2][slots][kSites][sizeof(T) == 4 ? 2 : 1];
    // norm q of colour c in lane `lane`: the summing wave of that colour leaves
    // it in the slot of direction 3 that only it reads and only wave 3 writes,
    // and wave 3 sums the colours before its next hops.  Without memory of
    // their own six FP32 blocks fit a CU instead of five.
    typedef double __attribute__((may_alias)) lane_norm;
    __device__ __forceinline__ lane_norm &norm(int q, int c, int lane)
    {
        return reinterpret_cast<lane_norm *>(w[0][first(3) + c][lane])[q];
    }
};
template <int DIR, int A, bool KEEP>
__device__ __forceinline__ void put_comp(Exchange<double, KEEP> &x, int lane, const cx<double> w[3], cx<double> &kept)
{
#pragma unroll
    for (int c = 0, n = 0; c < 3; c++) {
        if (KEEP && c == (DIR & 3))
            kept = w[c];
        else
            *(double2 *)x.w[A][x.first(DIR) + n++][lane] = make_double2(w[c].r, w[c].i);
    }
}
template <int DIR, bool KEEP>
__device__ __forceinline__ void put_half(Exchange<float, KEEP> &x, int lane, const cx<float> w0[3], const cx<float> w1[3],
                                         cx<float> kept[2])
{
#pragma unroll
    for (int c = 0, n = 0; c < 3; c++) {
        if (KEEP && c == (DIR & 3))
            kept[0] = w0[c], kept[1] = w1[c];
        else
            *(float4 *)x.w[0][x.first(DIR) + n++][lane] = make_float4(w0[c].r, w0[c].i, w1[c].r, w1[c].i);
    }
}
// acc += colour c of direction DIR (kept: that of this wave's own directions)
template <int DIR, int S, typename T, bool KEEP>
__device__ __forceinline__ void add_half(cx<T> acc[4], const Exchange<T, KEEP> &x, const cx<T> kept[2][2], int c, int lane)
{
    constexpr int mu = DIR & 3;
    if (KEEP && mu < 3 && c == mu) {  // uniform
        rebuild<mu, S>(acc, kept[DIR >> 2][0], kept[DIR >> 2][1]);
        return;
    }
    const int slot = x.first(DIR) + (KEEP && mu < 3 && c > mu ? c - 1 : c);
    if constexpr (sizeof(T) == 4) {
        const float4 v = *(const float4 *)x.w[0][slot][lane];
        rebuild<mu, S>(acc, cx<T>{v.x, v.y}, cx<T>{v.z, v.w});
    } else {
        const double2 v0 = *(const double2 *)x.w[0][slot][lane], v1 = *(const double2 *)x.w[1][slot][lane];
        rebuild<mu, S>(acc, cx<T>{v0.x, v0.y}, cx<T>{v1.x, v1.y});
    }
}

// one per block, whatever forms a kernel calls (the persistent kernel runs four)
template <typename T, bool KEEP>
__device__ __forceinline__ Exchange<T, KEEP> &exchange()
{
    __shared__ Exchange<T, KEEP> x;
    return x;
}

// workgroup barrier that orders LDS accesses only: loads from memory stay in
// flight across it (__syncthreads would wait for them)
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// The two hops of wave MU for one right-hand side (field sr) into the
// exchange; vf / vk: byte offsets of its lanes' neighbours at +-MU.  The links
// come from flink and blink (a call each, so that one right-hand side need not
// hold both).
template <typename SS, typename LS, typename T, int MU, int SF, bool ONE, typename LF, typename LB>
__device__ __forceinline__ void wave_hops(Exchange<T, ONE> &ex, cx<T> kept[2][2], rsrc_t sr, int vb, int vf, int vk,
                                          int lane, LF &&flink, LB &&blink, T one)
{
    constexpr int SB = -SF;
    if constexpr (sizeof(T) == 8) {
        // a quarter of the two hops' input at a time, the next quarter's
        // loads issued before the arithmetic of the previous one: the two
        // links take 72 registers, a whole spinor 48
        cx<T> w[3];
        rawc<T> p0[6], p1[6];
        load_half_spinor<SS, MU, 0>(p0, sr, vb, vf);
        load_half_spinor<SS, MU, 1>(p1, sr, vb, vf);
        {
            const auto *W = flink();
            half_hop_comp<MU, SF, 0>(w, W, p0, p0 + 3, one);
            put_comp<MU, 0>(ex, lane, w, kept[0][0]);
            __builtin_amdgcn_sched_barrier(0);
            load_half_spinor<SS, MU, 0>(p0, sr, vb, vk);
            half_hop_comp<MU, SF, 1>(w, W, p1, p1 + 3, one);
            put_comp<MU, 1>(ex, lane, w, kept[0][1]);
            __builtin_amdgcn_sched_barrier(0);
        }
        load_half_spinor<SS, MU, 1>(p1, sr, vb, vk);
        const auto *W = blink();
        half_hop_comp<MU, SB, 0>(w, W, p0, p0 + 3, one);
        put_comp<4 + MU, 0>(ex, lane, w, kept[1][0]);
        __builtin_amdgcn_sched_barrier(0);
        half_hop_comp<MU, SB, 1>(w, W, p1, p1 + 3, one);
        put_comp<4 + MU, 1>(ex, lane, w, kept[1][1]);
    } else {
        typename Held<SS, LS, T>::Spinor pf[12], pb[12];
        load_dir_spinor<SS, LS, T>(pf, sr, vb, vf);
        load_dir_spinor<SS, LS, T>(pb, sr, vb, vk);
        const auto *Wf = flink();
        const auto *Wb = blink();
        cx<T> w0[3], w1[3];
        half_hop<MU, SF>(w0, w1, Wf, pf, one);
        put_half<MU>(ex, lane, w0, w1, kept[0]);
        half_hop<MU, SB>(w0, w1, Wb, pb, one);
        put_half<4 + MU>(ex, lane, w0, w1, kept[1]);
    }
}

// One block of the launch: bhw is the block's index within its instance's
// range of nhw blocks (that range starts at a multiple of 8, so bhw % 8 is
// still the XCD).  Block order: see map_block.  ONE: a single right-hand side
// per block, so that the links need not be kept past its hops.
template <typename SS, typename LS, typename T, int DAG, int OWN, int EPI, bool ONE = false>
__device__ __forceinline__ void dslash_block(const DParams<T> &a, int bhw, int nhw)
{
    Exchange<T, ONE> &ex = exchange<T, ONE>();
    int grp;
    const int sblk = map_block(bhw, nhw, a.ngroups, a.nb_t, grp);
    const int r0 = grp * a.rpb, r1 = min(r0 + a.rpb, a.nrhs);
    const int lane = threadIdx.x & 63;
    const int mu = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int i_raw = sblk * kSites + lane;
    const bool valid = i_raw < a.g.vh;
    const int i = valid ? i_raw : a.g.vh - 1;  // idle lanes take part in the barriers
    int x, y, z, t;
    eo_coords(a.g, a.p, i, x, y, z, t);
    // neighbours by the row strides; a wrap is one compare and select
    const int sy = a.g.lxh, sz = sy * a.g.L[1], st = a.g.vsh;
    int jf, jb;
    if (mu == 0) {
        const int xh = x >> 1;
        jf = x & 1 ? (xh == sy - 1 ? i - (sy - 1) : i + 1) : i;
        jb = x & 1 ? i : (xh == 0 ? i + (sy - 1) : i - 1);
    } else if (mu == 1) {
        jf = y == a.g.L[1] - 1 ? i - (sz - sy) : i + sy;
        jb = y == 0 ? i + (sz - sy) : i - sy;
    } else if (mu == 2) {
        jf = z == a.g.L[2] - 1 ? i - (st - sz) : i + sz;
        jb = z == 0 ? i + (st - sz) : i - sz;
    } else {
        jf = t == a.g.L[3] - 1 ? i - (a.g.vh - st) : i + st;
        jb = t == 0 ? i + (a.g.vh - st) : i - st;
    }
    // the links of this wave: held for all right-hand sides, or (ONE) loaded
    // where they are used
    using Link = typename Held<SS, LS, T>::Link;
    const bool cf = mu == 3 && t == a.g.L[3] - 1, cb = mu == 3 && t == 0;
    Link Wf[9], Wb[9];
    auto flink = [&]() -> const Link * {
        if constexpr (ONE) load_dir_link<SS, LS, T>(Wf, a, mu, i, cf);
        return Wf;
    };
    auto blink = [&]() -> const Link * {
        if constexpr (ONE) load_dir_link<SS, LS, T>(Wb, a, 4 + mu, i, cb);
        return Wb;
    };
    if constexpr (!ONE) {
        load_dir_link<SS, LS, T>(Wf, a, mu, i, cf);
        load_dir_link<SS, LS, T>(Wb, a, 4 + mu, i, cb);
    }

    // forward hops use (1 - gamma) for H and (1 + gamma) for H^dag
    constexpr int SF = DAG ? -1 : 1, SB = -SF;
    constexpr int NQ = EPI == EPI_CG ? 2 : 1;
    const size_t fbytes = (size_t)12 * a.g.hs * sizeof(SS);  // one right-hand side
    const int vb = a.g.hs * (int)sizeof(SS), vo = i * (int)sizeof(SS);
    const int vf = jf * (int)sizeof(SS), vk = jb * (int)sizeof(SS);
    const bool track_rho = EPI == EPI_CG && a.rho != nullptr;  // uniform
    auto field = [&](const void *base, int r) { return make_rsrc((const char *)base + r * fbytes, fbytes); };
#pragma unroll 1
    for (int r = r0; r < r1; r++) {
        const rsrc_t sr = field(a.in, r);
        cx<T> kept[2][2];
        if (mu == 0)
            wave_hops<SS, LS, T, 0, SF, ONE>(ex, kept, sr, vb, vf, vk, lane, flink, blink, a.one);
        else if (mu == 1)
            wave_hops<SS, LS, T, 1, SF, ONE>(ex, kept, sr, vb, vf, vk, lane, flink, blink, a.one);
        else if (mu == 2)
            wave_hops<SS, LS, T, 2, SF, ONE>(ex, kept, sr, vb, vf, vk, lane, flink, blink, a.one);
        else
            wave_hops<SS, LS, T, 3, SF, ONE>(ex, kept, sr, vb, vf, vk, lane, flink, blink, a.one);
        // the fields of the own site: ahead of the barrier when the links are
        // no longer needed, else after the sum (registers)
        const int c = mu;  // the colour that this wave sums
        const rsrc_t rr_r = field(a.r, r), rho_r = field(a.rho, r);
        cx<T> o[4], rl[4];
        auto load_own = [&]() {
#pragma unroll
            for (int sp = 0; sp < 4; sp++) {
                const int so = (3 * sp + c) * vb;
                if (OWN) o[sp] = BufIO<SS>::template ld<T>(field(a.own, r), vo, so);
                if constexpr (EPI == EPI_CG || EPI == EPI_RES) rl[sp] = BufIO<SS>::template ld<T>(rr_r, vo, so);
            }
        };
        if constexpr (ONE)
            if (mu < 3) load_own();
        lds_barrier();
        if (mu < 3) {
            // all loads first, then arithmetic and stores: the stores may
            // alias the loaded fields as far as the compiler knows
            cx<T> acc[4];
#pragma unroll
            for (int sp = 0; sp < 4; sp++) acc[sp] = {0, 0};
            if constexpr (!ONE && sizeof(T) == 4) load_own();
            add_half<0, SF>(acc, ex, kept, c, lane);
            add_half<1, SF>(acc, ex, kept, c, lane);
            add_half<2, SF>(acc, ex, kept, c, lane);
            add_half<3, SF>(acc, ex, kept, c, lane);
            add_half<4, SB>(acc, ex, kept, c, lane);
            add_half<5, SB>(acc, ex, kept, c, lane);
            add_half<6, SB>(acc, ex, kept, c, lane);
            add_half<7, SB>(acc, ex, kept, c, lane);
            if constexpr (!ONE && sizeof(T) == 8) {
                __builtin_amdgcn_sched_barrier(0);
                load_own();
            }
            T alpha = 0;
            if constexpr (EPI == EPI_CG) alpha = (T)cgdev::ld_coh(&a.sc[r].alpha);
            double nrm[NQ];
#pragma unroll
            for (int q = 0; q < NQ; q++) nrm[q] = 0;
#pragma unroll
            for (int sp = 0; sp < 4; sp++) {
                const int so = (3 * sp + c) * vb;
                cx<T> v = (sp < 2 ? a.hop_u : a.hop_l) * acc[sp];
                if (OWN) v = v + (sp < 2 ? a.own_u : a.own_l) * o[sp];
                if constexpr (EPI == EPI_CG) {
                    const cx<T> rv = rl[sp] - alpha * v;
                    if (valid) BufIO<SS>::template st<T>(rr_r, vo, so, rv);
                    nrm[0] += norm2c(stored<SS>(rv));
                } else if constexpr (EPI == EPI_RES) {
                    const cx<T> rv = rl[sp] - v;
                    if (valid && a.out) BufIO<SS>::template st<T>(field(a.out, r), vo, so, rv);
                    nrm[0] += norm2c(stored<SS>(rv));
                } else {
                    if (valid) BufIO<SS>::template st<T>(field(a.out, r), vo, so, v);
                    if constexpr (EPI == EPI_NORM) nrm[0] += norm2c(stored<SS>(v));
                }
            }
            if (track_rho) {
                cx<T> hl[4];
#pragma unroll
                for (int sp = 0; sp < 4; sp++) hl[sp] = BufIO<SS>::template ld<T>(rho_r, vo, (3 * sp + c) * vb);
#pragma unroll
                for (int sp = 0; sp < 4; sp++) {
                    const cx<T> hv = hl[sp] - alpha * o[sp];
                    if (valid) BufIO<SS>::template st<T>(rho_r, vo, (3 * sp + c) * vb, hv);
                    nrm[NQ - 1] += norm2c(stored<SS>(hv));
                }
            }
            if constexpr (EPI != EPI_STORE) {
#pragma unroll
                for (int q = 0; q < NQ; q++) ex.norm(q, c, lane) = valid ? nrm[q] : 0.0;
            }
        }
        if constexpr (!ONE || EPI != EPI_STORE) lds_barrier();
        if constexpr (EPI != EPI_STORE) {
            // the wave without a colour sums the block's norms (fixed order)
            // while the others go on; they reach the norms' slots again only
            // past the next barrier
            if (mu == 3) {
#pragma unroll
                for (int q = 0; q < NQ; q++) {
                    if (q == 1 && !track_rho) break;
                    const double s = cgdev::wave_sum(ex.norm(q, 0, lane) + ex.norm(q, 1, lane) + ex.norm(q, 2, lane));
                    if (lane == 0) cgdev::st_coh(a.part + ((size_t)q * a.nrhs + r) * a.nblk + sblk, s);
                }
            }
        }
        if constexpr (ONE) break;
    }
}

// The blocks past the launch's own nblk * ngroups, one per right-hand side:
// alpha, or the beta step, from the partial sums of an earlier launch, which the
// hops of this one do not read.  A launch of its own cost 3 to 5 us in the chain of an
// iteration.  True: block `over` had nothing else to do.
template <int DAG, int OWN, int EPI, typename T>
__device__ __forceinline__ bool alpha_block(const DParams<T> &a, int over)
{
    if (over < 0) return false;
    if constexpr (DAG == 1 && OWN == 0 && EPI == EPI_STORE)
        if (a.alpha > 0 && over < a.nrhs)
            cgdev::finish_alpha(const_cast<CGScalars *>(a.sc), a.part, a.nblk, a.alpha - 1, over);
    if constexpr (DAG == 0 && OWN == 0 && EPI == EPI_STORE)
        if (a.alpha < 0 && over < a.nrhs)
            cgdev::finish_beta(const_cast<CGScalars *>(a.sc), a.part, a.nblk, a.nrhs, a.delta, over);
    return true;
}
int alpha_blocks(const DslashCall &dc) { return dc.alpha > 0 || dc.beta > 0 ? dc.nrhs : 0; }

template <typename SS, typename LS, typename T, int DAG, int OWN, int EPI, bool ONE>
__global__ __launch_bounds__(kBlock, (waves_for<SS, LS, T, ONE>())) void k_dslash(DParams<T> a)
{
    const int nreal = a.nblk * a.ngroups;
    if (alpha_block<DAG, OWN, EPI>(a, (int)blockIdx.x - nreal)) return;
    dslash_block<SS, LS, T, DAG, OWN, EPI, ONE>(a, blockIdx.x, nreal);
}

// Several lattices in one launch: instance i owns hardware blocks
// [start[i], start[i+1]) (padded to multiples of 8; padding blocks exit).
// The records travel in the kernel-argument segment, like the single form's
// parameters: uniform, read-only scalar loads that the compiler may repeat
// after the epilogue's stores without going through the vector caches.
template <typename T>
struct MultiArgs {
    DParams<T> p[kMultiInst];
    int start[kMultiInst + 1];
    int n;
};
static_assert(sizeof(MultiArgs<double>) <= 4096, "kernel arguments exceed 4 KiB");

template <typename SS, typename LS, typename T, int DAG, int OWN, int EPI>
__global__ __launch_bounds__(kBlock, (waves_for<SS, LS, T>())) void k_dslash_multi(const MultiArgs<T> m)
{
    int i = 0;
    while (i + 1 < m.n && (int)blockIdx.x >= m.start[i + 1]) i++;
    const int local = (int)blockIdx.x - m.start[i];
    const int nreal = m.p[i].nblk * m.p[i].ngroups;
    if (alpha_block<DAG, OWN, EPI>(m.p[i], local - nreal)) return;
    dslash_block<SS, LS, T, DAG, OWN, EPI>(m.p[i], local, nreal);
}

// ---------------------------------------------------------------- persistent batch
// One launch runs `iters` CG iterations of every instance of a batch: the
// four half-Dslash stages, the CG scalars and the vector update, separated
// by grid-wide barriers.  The grid is sized so that every block is resident
// (cooperative launch).  Each Dslash stage walks the virtual blocks of all
// instances (the same (instance, site block, RHS group) decomposition and
// XCD mapping as the multi-instance kernel: the grid is a multiple of 8, so
// virtual block v runs on XCD v % 8); the scalar stages give one
// (instance, right-hand side) to a block and run the code of the
// stand-alone scalar kernels, so every instance follows its single solve
// bit for bit.  Per iteration:
//   S1 | S2 | S3 + alpha | S4 | beta | update |
// (alpha is summed while the third stage runs: that stage does not read it).

// Barrier state in device memory (zeroed before each launch), one 128-byte
// line per word: arrivals of the blocks with blockIdx % 8 == j, arrivals of
// the eight groups, the generation published to group j, the failure flag.
constexpr int kBarLine = 32;  // unsigned words per line
constexpr int kBarWords = 18 * kBarLine;
__device__ __forceinline__ unsigned *bar_cnt(unsigned *b, int j) { return b + j * kBarLine; }
__device__ __forceinline__ unsigned *bar_top(unsigned *b) { return b + 8 * kBarLine; }
__device__ __forceinline__ unsigned *bar_gen(unsigned *b, int j) { return b + (9 + j) * kBarLine; }
__device__ __forceinline__ unsigned *bar_fail(unsigned *b) { return b + 17 * kBarLine; }

// Launch parameters, kept in device memory (read-only during the launch):
// the stages index them with the instance number, which a kernel-argument
// block would have to copy to per-lane scratch memory.
template <typename T>
struct PersistArgs {
    // the stage forms of each instance: rows 0.. stage 1 per ring position,
    // kCgRing.. stage 2 per ring position, then stages 3 and 4
    DParams<T> st[2 * kCgRing + 2][kPersistInst];
    void *ring[kPersistInst][kCgRing];  // search directions, m of them
    int m;
    void *x[kPersistInst];           // solution accumulator (FP32)
    CGScalars *sc[kPersistInst];
    double delta[kPersistInst];
    int start[kPersistInst + 1];     // virtual Dslash blocks, multiples of 8
    int ustart[kPersistInst + 1];    // update work items (right-hand side x chunk)
    int uchunks[kPersistInst];       // chunks per right-hand side
    int fstart[kPersistInst + 1];    // scalar work items (right-hand sides)
    int n;
    unsigned *bar;                   // kBarWords words
};

constexpr int kUpdChunk = 8 * kBlock;  // elements per update work item

// Grid-wide barrier with a bounded wait, in two levels (the blocks of each
// of the eight residue classes of blockIdx, then the eight classes) so that
// no address takes more than G/8 arrivals or pollers.  Returns false (in
// every thread) when this or another block gave up; the caller then leaves
// the kernel.
__device__ __forceinline__ bool grid_sync(unsigned *bar, unsigned long long spin_limit)
{
    __shared__ int ok;
    // every wave waits until its own stores have reached the L2 (the
    // workgroup barrier alone does not wait for other waves' stores); the
    // release below then writes this L2's dirty lines back once per block
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (threadIdx.x == 0) {
        const int j = blockIdx.x & 7;
        const unsigned per = gridDim.x >> 3;  // the grid is a multiple of 8
        // release this block's results to the other XCDs (L2 write-back)
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        // the generation is read before arriving (acquire: the arrival below
        // cannot be performed first), so it cannot have advanced yet
        const unsigned g = __hip_atomic_load(bar_gen(bar, j), __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT);
        int good = 1;
        if (__hip_atomic_fetch_add(bar_cnt(bar, j), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1 == per) {
            // the class's counter is reset before the class arrives above (a
            // block of the class may arrive at the next barrier as soon as
            // the generation moves)
            __hip_atomic_store(bar_cnt(bar, j), 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __builtin_amdgcn_s_waitcnt(0);
            if (__hip_atomic_fetch_add(bar_top(bar), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1 == 8) {
                __hip_atomic_store(bar_top(bar), 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
                for (int k = 0; k < 8; k++)
                    __hip_atomic_fetch_add(bar_gen(bar, k), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        // poll about every 0.5 us, the failure flag every 32nd poll
        unsigned long long n = 0;
        while (__hip_atomic_load(bar_gen(bar, j), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == g) {
            if (++n > spin_limit ||
                ((n & 31) == 0 && __hip_atomic_load(bar_fail(bar), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))) {
                __hip_atomic_store(bar_fail(bar), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                good = 0;
                break;
            }
            __builtin_amdgcn_s_sleep(20);
        }
        if (__hip_atomic_load(bar_fail(bar), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) good = 0;
        // acquire the other blocks' results (invalidate this CU's L1 and
        // the stale L2 lines)
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        ok = good;
    }
    __syncthreads();
    return ok != 0;
}

// One Dslash stage over the virtual blocks of all instances; row k of the forms.
template <typename SS, typename LS, typename T, int DAG, int OWN, int EPI>
__device__ __forceinline__ void persist_stage(const PersistArgs<T> &a, int k)
{
    const int total = a.start[a.n];
    for (int vb = blockIdx.x; vb < total; vb += gridDim.x) {
        int i = 0;
        while (i + 1 < a.n && vb >= a.start[i + 1]) i++;
        const DParams<T> &p = a.st[k][i];
        const int local = vb - a.start[i];
        const int nreal = p.nblk * p.ngroups;
        if (local >= nreal) continue;
        dslash_block<SS, LS, T, DAG, OWN, EPI>(p, local, nreal);
    }
}

// The CG scalars of one right-hand side per block: alpha from the partial
// sums of stage 2 (BETA = false) or beta and the flags from those of stage 4.
template <typename T, bool BETA>
__device__ __forceinline__ void persist_scalars(const PersistArgs<T> &a, int pos)
{
    const int total = a.fstart[a.n];
    for (int w = blockIdx.x; w < total; w += gridDim.x) {
        int i = 0;
        while (i + 1 < a.n && w >= a.fstart[i + 1]) i++;
        const int r = w - a.fstart[i];
        if constexpr (BETA) {
            const DParams<T> &p = a.st[2 * kCgRing + 1][i];
            cgdev::finish_beta(a.sc[i], p.part, p.nblk, p.nrhs, a.delta[i], r);
        } else {
            const DParams<T> &p = a.st[kCgRing][i];
            cgdev::finish_alpha(a.sc[i], p.part, p.nblk, pos, r);
        }
    }
}

template <typename SS, typename T>
__device__ __forceinline__ void persist_update(const PersistArgs<T> &a, int pos)
{
    const int total = a.ustart[a.n];
    for (int w = blockIdx.x; w < total; w += gridDim.x) {
        int i = 0;
        while (i + 1 < a.n && w >= a.ustart[i + 1]) i++;
        const int local = w - a.ustart[i];
        const int r = local / a.uchunks[i], ch = local - r * a.uchunks[i];
        const DParams<T> &p3 = a.st[2 * kCgRing + 1][i];  // stage 4 updates r
        const size_t n = (size_t)12 * p3.g.hs;
        const size_t e0 = (size_t)ch * kUpdChunk, e1 = e0 + kUpdChunk < n ? e0 + kUpdChunk : n;
        const SS *rv = (const SS *)p3.r;
        float2 *x = (float2 *)a.x[i];
        void *const *ring = a.ring[i];
        const cgdev::NextBeta nb = cgdev::stored_beta(a.sc[i], r);
        if (pos < a.m - 1)
            cgdev::update_p((SS *)ring[pos + 1], (const SS *)ring[pos], rv, n, nb, r, e0 + threadIdx.x, e1,
                            (size_t)kBlock);
        else if (a.m == 8)
            cgdev::update_px<8, SS>(ring, rv, x, n, a.sc[i], nb, r, e0 + threadIdx.x, e1, (size_t)kBlock);
        else if (a.m == 4)
            cgdev::update_px<4, SS>(ring, rv, x, n, a.sc[i], nb, r, e0 + threadIdx.x, e1, (size_t)kBlock);
        else if (a.m == 2)
            cgdev::update_px<2, SS>(ring, rv, x, n, a.sc[i], nb, r, e0 + threadIdx.x, e1, (size_t)kBlock);
        else
            cgdev::update_px<1, SS>(ring, rv, x, n, a.sc[i], nb, r, e0 + threadIdx.x, e1, (size_t)kBlock);
    }
}

template <typename SS, typename LS, typename T>
__global__ __launch_bounds__(kBlock, (waves_for<SS, LS, T>())) void k_batch_persist(const PersistArgs<T> *__restrict__ pa,
                                                                             int iters,
                                                                             unsigned long long spin_limit)
{
    const PersistArgs<T> &a = *pa;
    for (int it = 0, pos = 0; it < iters; it++, pos = pos + 1 == a.m ? 0 : pos + 1) {
        persist_stage<SS, LS, T, 0, 0, EPI_STORE>(a, pos);            // t = R_oo^-1 H_oe p
        if (!grid_sync(a.bar, spin_limit)) return;
        persist_stage<SS, LS, T, 0, 1, EPI_NORM>(a, kCgRing + pos);   // q = R_ee p - H_eo t, |q|^2 partials
        if (!grid_sync(a.bar, spin_limit)) return;
        persist_stage<SS, LS, T, 1, 0, EPI_STORE>(a, 2 * kCgRing);    // t = R_oo^-1 H_oe^dag q
        persist_scalars<T, false>(a, pos);                            // alpha
        if (!grid_sync(a.bar, spin_limit)) return;
        persist_stage<SS, LS, T, 0, 1, EPI_CG>(a, 2 * kCgRing + 1);   // r -= alpha Ahat^dag q, partials
        if (!grid_sync(a.bar, spin_limit)) return;
        persist_scalars<T, true>(a, pos);                             // beta, flags
        if (!grid_sync(a.bar, spin_limit)) return;
        persist_update<SS, T>(a, pos);                                // p = r + beta p, at the ring's end x
        if (it + 1 < iters && !grid_sync(a.bar, spin_limit)) return;
    }
}

template <typename T>
cx<T> cvt(cx<double> v)
{
    return cx<T>{(T)v.r, (T)v.i};
}

// The fused epilogues belong to the second halves of the Schur operator
// (dag = 0 with the own-site term); the other forms store only.
//
// A single right-hand side per block has a form of its own (ONE: the links are
// loaded where they are used, the summing waves keep a colour in registers and
// load the fields of the own site ahead of the barrier) where that is the faster
// one: the CG update and the residual, which read two of those fields (FP64 with
// 8-parameter links, 32^3 x 64, one right-hand side: 361 us against 467);
// 12-parameter links, whose rebuilt rows then take no registers across the hops
// (BF16 Schur operator, 24^3 x 48, 40 us against 48); BF16 with binary16 links.
// Otherwise links with all their parameters, or with eight, are better loaded ahead
// of the spinors' arithmetic, as for several: Schur operator, 32^3 x 16, one
// right-hand side, FP32 90 us against 93, FP64 with 8 parameters 120 against 123,
// BF16 with FP32 links 72 against 74.
template <typename SS, typename LS, int EPI>
constexpr bool kOneForm = EPI == EPI_CG || EPI == EPI_RES || std::is_same<LS, L12>::value ||
                          std::is_same<LS, L12D>::value || std::is_same<LS, L12F>::value ||
                          (std::is_same<SS, b2>::value && std::is_same<LS, h2>::value);

template <typename SS, typename LS, typename T, int DAG, int OWN, int EPI>
void launch_form(dim3 grid, hipStream_t s, const DParams<T> &a)
{
    if constexpr (kOneForm<SS, LS, EPI>)
        if (a.rpb == 1) {
            hipLaunchKernelGGL((k_dslash<SS, LS, T, DAG, OWN, EPI, true>), grid, dim3(kBlock), 0, s, a);
            return;
        }
    hipLaunchKernelGGL((k_dslash<SS, LS, T, DAG, OWN, EPI, false>), grid, dim3(kBlock), 0, s, a);
}

template <typename SS, typename LS, typename T, int DAG, int OWN>
void launch_epi(const DslashCall &dc, dim3 grid, hipStream_t s, const DParams<T> &a)
{
    if constexpr (DAG == 0 && OWN == 1) {
        if (dc.epi == EPI_NORM) return launch_form<SS, LS, T, DAG, OWN, EPI_NORM>(grid, s, a);
        if (dc.epi == EPI_CG) return launch_form<SS, LS, T, DAG, OWN, EPI_CG>(grid, s, a);
        if constexpr (std::is_same<LS, double2>::value)
            if (dc.epi == EPI_RES) return launch_form<SS, LS, T, DAG, OWN, EPI_RES>(grid, s, a);
    }
    TM_REQUIRE(dc.epi == EPI_STORE, "fused epilogues need dag = 0 and the own-site term (residuals: the exact links)");
    launch_form<SS, LS, T, DAG, OWN, EPI_STORE>(grid, s, a);
}

// Right-hand sides per block (at most), for instances given as (site blocks,
// nrhs) and `slots` resident blocks (slots_one where a block takes a single
// right-hand side; BF16, 12 x 20 x 14 x 22, 5 right-hand sides: 24.9 us for the
// Schur operator at one per block, 27.2 at two, 31.3 at three, 28.8 at five):
// every instance splits its right-hand sides evenly over the fewest blocks that
// keep the limit.  More of them per block share one load and one rebuild of the
// links and keep the resident blocks on fewer sites, so that neighbouring blocks
// find each other's spinors in the L2; fewer fill the chip on small lattices.  The
// limit taken has the least (rounds of resident blocks) x (mean block length), a
// block's start and its links counting as one right-hand side: over 2970 calls 1.4%
// longer on average than the best split of each.  equal: only splits into blocks of
// one length.  TM_DSLASH_RHS_TILE and TM_BATCH_RHS_TILE in the environment fix the
// limit (results are bit-identical for any).
int even_split(int nrhs, int most)
{
    const int groups = (nrhs + most - 1) / most;
    return (nrhs + groups - 1) / groups;
}
int rhs_per_block(const std::vector<std::pair<int, int>> &inst, long slots, long slots_one, bool equal = false)
{
    int top = 1, best = 1;
    for (const auto &[nb, nrhs] : inst) top = std::max(top, nrhs);
    double least = 0;
    for (int lim = 1; lim <= top; lim++) {
        double blocks = 0, length = 0;
        int longest = 0;
        bool skip = false;
        for (const auto &[nb, nrhs] : inst) {
            const int rpb = even_split(nrhs, lim), g = (nrhs + rpb - 1) / rpb;
            skip |= equal && nrhs % rpb != 0;
            blocks += (double)nb * g;
            length += (double)nb * (g + nrhs);
            longest = std::max(longest, 1 + rpb);
        }
        if (skip) continue;
        const double cost = std::max((double)longest, std::ceil(blocks / (lim == 1 ? slots_one : slots)) * length / blocks);
        if (lim == 1 || cost < least) {
            least = cost;
            best = lim;
        }
    }
    return best;
}

// The blocks that the limit of one counts with (see kOneForm).  BF16: six per CU
// with 12-parameter links; 5.5 with full ones, where blocks of one load half as
// much again (32^3 x 64, 3 right-hand sides: 409 us for the Schur operator at one
// per block, 354 at three; counting six took one).  FP64: as for several,
// although four blocks fit instead of three, since each rebuilds its rows in FP64
// (16^3 x 32, 4 right-hand sides: 78 us at one per block, 74 at two; counting
// four made 21 of 290 calls slower, by up to 16%).
template <typename SS, typename LS, typename T>
long slots_of(const tm_ctx *c) { return (long)c->cus * waves_for<SS, LS, T>(); }
template <typename SS, typename LS, typename T>
long slots_of_one(const tm_ctx *c)
{
    if (sizeof(T) == 8) return slots_of<SS, LS, T>(c);
    const bool full = std::is_same<SS, b2>::value && std::is_same<LS, h2>::value;
    return (long)c->cus * waves_for<SS, LS, T, true>() - (full ? c->cus / 2 : 0);
}

template <typename SS, typename LS, typename T>
DParams<T> fill_params(tm_ctx *c, const DslashCall &dc, int most)
{
    const int rpb = even_split(dc.nrhs, most);
    DParams<T> a;
    a.out = dc.out;
    a.in = dc.in;
    a.own = dc.own;
    a.links = (std::is_same<LS, double2>::value ? c->links64
               : std::is_same<LS, h2>::value     ? c->links16
               : std::is_same<LS, L12>::value    ? c->links12
               : std::is_same<LS, L12D>::value   ? c->links12d
               : std::is_same<LS, L12F>::value   ? c->links12f
               : std::is_same<LS, L8D>::value    ? c->links8d
                                                 : c->links32)[dc.out_parity];
    a.g = c->geo;
    a.p = dc.out_parity;
    a.nrhs = dc.nrhs;
    a.rpb = rpb;
    a.ngroups = (dc.nrhs + rpb - 1) / rpb;
    a.own_u = cvt<T>(dc.d_own.u);
    a.own_l = cvt<T>(dc.d_own.l);
    a.hop_u = cvt<T>(dc.d_hop.u);
    a.hop_l = cvt<T>(dc.d_hop.l);
    a.one = (T)1;
    a.r = dc.r;
    if (dc.beta)
        a.delta = dc.delta;
    else
        a.rho = dc.rho;
    a.sc = dc.sc;
    a.part = dc.part;
    a.alpha = dc.beta ? -1 : dc.alpha;
    a.nblk = dslash_site_blocks(c);
    a.nb_t = (c->geo.vsh % kSites == 0 && (c->geo.vsh / kSites) % 8 == 0) ? c->geo.vsh / kSites : 0;
    a.t_bc = c->t_bc;
    return a;
}

template <typename SS, typename LS, typename T>
void launch_t(tm_ctx *c, const DslashCall &dc, hipStream_t s)
{
    // FP64, three or five right-hand sides: blocks of one length.  Blocks of two and
    // of one fill the chip unevenly (12^3 x 24, 3 right-hand sides, 18 / 12
    // parameters: Schur operator 29.0 / 26.2 us against 24.0 / 22.2 at one per block;
    // 20 x 16 x 18 x 24, 82.8 / 76.1 against 78.0 / 67.6 at three).  The 8-parameter
    // links, the dearest to rebuild, are shared all the same (12^3 x 24, 5: 38.3
    // against 41.8), and from seven on neither side is ahead throughout.
    const bool equal = sizeof(T) == 8 && !std::is_same<LS, L8D>::value && dc.nrhs <= 5;
    int rpb = rhs_per_block({{dslash_site_blocks(c), dc.nrhs}}, slots_of<SS, LS, T>(c), slots_of_one<SS, LS, T>(c), equal);
    if (const char *e = getenv("TM_DSLASH_RHS_TILE"))
        if (atoi(e) > 0) rpb = atoi(e);
    const DParams<T> a = fill_params<SS, LS, T>(c, dc, rpb);
    TM_REQUIRE(dc.alpha == 0 || (dc.dag && !dc.has_own), "alpha is summed beside the dag hops only");
    TM_REQUIRE(dc.beta == 0 || (!dc.dag && !dc.has_own), "beta is summed beside the plain hops only");
    dim3 grid((unsigned)(a.nblk * a.ngroups + alpha_blocks(dc)));
    // separate kernels per projector placement and per presence of the
    // own-site term (the x - H y forms read one more field)
    if (dc.dag) {
        if (dc.has_own)
            launch_epi<SS, LS, T, 1, 1>(dc, grid, s, a);
        else
            launch_epi<SS, LS, T, 1, 0>(dc, grid, s, a);
    } else {
        if (dc.has_own)
            launch_epi<SS, LS, T, 0, 1>(dc, grid, s, a);
        else
            launch_epi<SS, LS, T, 0, 0>(dc, grid, s, a);
    }
    TM_HIP(hipGetLastError());
}

template <typename SS, typename LS, typename T>
void multi_fill(MultiDslash &m, const std::vector<tm_ctx *> &cs, const std::vector<DslashCall> &dcs, int rpb)
{
    m.args.clear();
    m.grid.clear();
    for (size_t c0 = 0; c0 < cs.size(); c0 += kMultiInst) {
        MultiArgs<T> a{};
        const size_t c1 = std::min(cs.size(), c0 + kMultiInst);
        a.n = (int)(c1 - c0);
        a.start[0] = 0;
        for (size_t k = c0; k < c1; k++) {
            const int j = (int)(k - c0);
            a.p[j] = fill_params<SS, LS, T>(cs[k], dcs[k], rpb);
            const int nb = a.p[j].nblk * a.p[j].ngroups + alpha_blocks(dcs[k]);
            a.start[j + 1] = a.start[j] + (nb + 7) / 8 * 8;
        }
        const unsigned char *raw = reinterpret_cast<const unsigned char *>(&a);
        m.args.emplace_back(raw, raw + sizeof(a));
        m.grid.push_back(a.start[a.n]);
    }
}

template <typename SS, typename LS, typename T>
void multi_go(const MultiDslash &m, hipStream_t s)
{
    for (size_t c = 0; c < m.args.size(); c++) {
        TM_REQUIRE(m.args[c].size() == sizeof(MultiArgs<T>), "multi-instance arguments of another precision");
        MultiArgs<T> a;
        std::memcpy(&a, m.args[c].data(), sizeof(a));
        dim3 g(m.grid[c]), b(kBlock);
        // the four stage forms of a CG iteration on the Schur normal equations
        if (m.dag == 0 && m.own == 0 && m.epi == EPI_STORE)
            hipLaunchKernelGGL((k_dslash_multi<SS, LS, T, 0, 0, EPI_STORE>), g, b, 0, s, a);
        else if (m.dag == 1 && m.own == 0 && m.epi == EPI_STORE)
            hipLaunchKernelGGL((k_dslash_multi<SS, LS, T, 1, 0, EPI_STORE>), g, b, 0, s, a);
        else if (m.dag == 0 && m.own == 1 && m.epi == EPI_NORM)
            hipLaunchKernelGGL((k_dslash_multi<SS, LS, T, 0, 1, EPI_NORM>), g, b, 0, s, a);
        else if (m.dag == 0 && m.own == 1 && m.epi == EPI_CG)
            hipLaunchKernelGGL((k_dslash_multi<SS, LS, T, 0, 1, EPI_CG>), g, b, 0, s, a);
        else
            throw TmError{TM_ERR_UNSUPPORTED, "multi-instance Dslash form not instantiated"};
        TM_HIP(hipGetLastError());
    }
}

template <typename F>
void multi_dispatch(int prec, bool recon12, bool recon8, F &&f)
{
    auto with = [&](auto *tag) {
        using P3 = std::remove_pointer_t<decltype(tag)>;
        f.template operator()<typename P3::SS, typename P3::LS, typename P3::T>();
    };
    struct PD { using SS = double2; using LS = double2; using T = double; };
    struct PD12 { using SS = double2; using LS = L12D; using T = double; };
    struct PD8 { using SS = double2; using LS = L8D; using T = double; };
    struct PF { using SS = float2; using LS = float2; using T = float; };
    struct PF12 { using SS = float2; using LS = L12F; using T = float; };
    struct PH { using SS = h2; using LS = h2; using T = float; };
    struct PB { using SS = b2; using LS = h2; using T = float; };
    struct PH12 { using SS = h2; using LS = L12; using T = float; };
    struct PB12 { using SS = b2; using LS = L12; using T = float; };
    switch (prec) {
    case TM_F64:
        if (recon8)
            with((PD8 *)nullptr);
        else
            recon12 ? with((PD12 *)nullptr) : with((PD *)nullptr);
        break;
    case TM_F32: recon12 ? with((PF12 *)nullptr) : with((PF *)nullptr); break;
    case TM_F16: recon12 ? with((PH12 *)nullptr) : with((PH *)nullptr); break;
    case TM_BF16: recon12 ? with((PB12 *)nullptr) : with((PB *)nullptr); break;
    default: throw TmError{TM_ERR_ARG, "bad precision"};
    }
}

template <typename SS, typename LS, typename T>
void persist_fill(PersistBatch &pb, const std::vector<PersistInst> &v, hipStream_t s)
{
    if constexpr (sizeof(T) == 8) {
        throw TmError{TM_ERR_UNSUPPORTED, "the persistent batch kernel takes FP32-arithmetic solvers"};
    } else {
    PersistArgs<T> a{};
    a.n = (int)v.size();
    a.m = v[0].ring.m;
    for (int k = 0; k < a.n; k++) {
        const CgRing &ring = v[k].ring;
        TM_REQUIRE(ring.m == v[0].ring.m, "batched solves share the ring length");
        std::copy(ring.p, ring.p + kCgRing, a.ring[k]);
        auto form = [&](int stage, int pos) {
            DslashCall dc = v[k].st[stage];
            if (stage == 0) dc.in = ring.p[pos];
            if (stage == 1) dc.own = ring.p[pos];
            return fill_params<SS, LS, T>(v[k].c, dc, pb.rpb);
        };
        for (int pos = 0; pos < ring.m; pos++) {
            a.st[pos][k] = form(0, pos);
            a.st[kCgRing + pos][k] = form(1, pos);
        }
        a.st[2 * kCgRing][k] = form(2, 0);
        a.st[2 * kCgRing + 1][k] = form(3, 0);
        const int nb = a.st[0][k].nblk * a.st[0][k].ngroups;
        a.start[k + 1] = a.start[k] + (nb + 7) / 8 * 8;
        const size_t n = (size_t)12 * v[k].c->geo.hs;
        a.uchunks[k] = (int)((n + kUpdChunk - 1) / kUpdChunk);
        a.ustart[k + 1] = a.ustart[k] + a.uchunks[k] * v[k].st[0].nrhs;
        a.fstart[k + 1] = a.fstart[k] + v[k].st[0].nrhs;
        a.x[k] = v[k].x;
        a.sc[k] = v[k].sc;
        a.delta[k] = v[k].delta;
    }
    pb.work = std::max(a.start[a.n], a.ustart[a.n]);
    pb.sync_bytes = sizeof(unsigned) * kBarWords;
    pb.bar = ws_get(v[0].c, "persist_sync", pb.sync_bytes);
    a.bar = (unsigned *)pb.bar;
    pb.args_bytes = sizeof(a);
    // the table is rewritten only when no launch that reads it is in flight
    TM_HIP(hipStreamSynchronize(s));
    pb.dev_args = ws_get(v[0].c, "persist_args", sizeof(a));
    TM_HIP(hipMemcpy(pb.dev_args, &a, sizeof(a), hipMemcpyHostToDevice));
    // co-resident blocks of this instantiation: the grid of the cooperative launch
    int per_cu = 0;
    TM_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_batch_persist<SS, LS, T>, kBlock, 0));
    if (pb.blocks_per_cu > 0) per_cu = std::min(per_cu, pb.blocks_per_cu);
    const int cap = per_cu * v[0].c->cus / 8 * 8;
    TM_REQUIRE(cap >= 8, "the persistent batch kernel does not fit the device");
    // about eight work items per block, at least a block per CU: a grid barrier
    // takes longer the more blocks arrive (FP16, 16^3 x 32, 12^3 x 24 and 8^3 x 16,
    // one right-hand side each, 1412 items: 12.0 ms a batch with 256 blocks, 12.8
    // with 512, 21.0 with one per item; 12, 24 and 48 each, 5800 items: 46.3 with
    // 768, 53.1 with 1536)
    const int most = std::max(v[0].c->cus, pb.work / 8);
    pb.grid = std::min(cap, (std::min(most, pb.work) + 7) / 8 * 8);
    }
}

template <typename SS, typename LS, typename T>
bool persist_go(const PersistBatch &pb, hipStream_t s)
{
    if constexpr (sizeof(T) == 8) {
        return false;
    } else {
    TM_REQUIRE(pb.args_bytes == sizeof(PersistArgs<T>), "persistent batch arguments of another precision");
    const PersistArgs<T> *pa = (const PersistArgs<T> *)pb.dev_args;
    int iters = pb.iters;
    unsigned long long spin = pb.spin_limit;
    void *kargs[] = {&pa, &iters, &spin};
    if (hipLaunchCooperativeKernel((const void *)k_batch_persist<SS, LS, T>, dim3(pb.grid), dim3(kBlock), kargs,
                                   0, s) != hipSuccess) {
        (void)hipGetLastError();  // refused (e.g. the grid cannot be co-resident): nothing was launched
        return false;
    }
    return true;
    }
}

}  // namespace

void multi_dslash_prepare(MultiDslash &m, const std::vector<tm_ctx *> &cs, const std::vector<DslashCall> &dcs, int rpb,
                          hipStream_t s)
{
    TM_REQUIRE(!cs.empty() && cs.size() == dcs.size(), "bad multi-instance call");
    for (tm_ctx *c : cs)
        if (dcs[0].spinor_prec == TM_F16 || dcs[0].spinor_prec == TM_BF16)
            if (c->half_links_f32)
                throw TmError{TM_ERR_UNSUPPORTED, "batches read binary16 links for FP16/BF16 spinors"};
    m.prec = dcs[0].spinor_prec;
    m.dag = dcs[0].dag;
    m.own = dcs[0].has_own ? 1 : 0;
    m.epi = dcs[0].epi;
    m.n = (int)cs.size();
    m.recon8 = false;
    for (size_t k = 0; k < cs.size(); k++) {
        TM_REQUIRE(dcs[k].spinor_prec == m.prec && dcs[k].dag == m.dag && (dcs[k].has_own ? 1 : 0) == m.own &&
                       dcs[k].epi == m.epi,
                   "multi-instance calls must share precision and operator form");
        TM_REQUIRE(cs[k]->have_gauge, "no gauge field set");
        TM_REQUIRE(recon12_ok(cs[k], m.prec) == recon12_ok(cs[0], m.prec),
                   "multi-instance calls must share the link format");
        if (m.prec == TM_F32) {
            if (recon12_ok(cs[k], m.prec))
                ensure_links12f(cs[k], s);
            else
                ensure_links32(cs[k], s);
        }
        if (m.prec == TM_F64) {
            const bool r8 = recon8_wanted(cs[k]) && ensure_links8d(cs[k], s);
            TM_REQUIRE(k == 0 || r8 == m.recon8, "multi-instance calls must share the link format");
            m.recon8 = r8;
            if (!r8 && recon12_ok(cs[k], m.prec)) ensure_links12d(cs[k], s);
        }
        if (m.prec == TM_F16 || m.prec == TM_BF16) {
            if (recon12_ok(cs[k], m.prec))
                ensure_links12(cs[k], s);
            else
                ensure_links16(cs[k], s);
        }
    }
    m.recon12 = recon12_ok(cs[0], m.prec);
    multi_dispatch(m.prec, m.recon12, m.recon8,
                   [&]<typename SS, typename LS, typename T>() { multi_fill<SS, LS, T>(m, cs, dcs, rpb); });
}

void multi_dslash_launch(const MultiDslash &m, hipStream_t s)
{
    multi_dispatch(m.prec, m.recon12, m.recon8,
                   [&]<typename SS, typename LS, typename T>() { multi_go<SS, LS, T>(m, s); });
}

bool persist_supported(int device)
{
    int coop = 0;
    if (hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, device) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return coop != 0;
}

void persist_prepare(PersistBatch &pb, const std::vector<PersistInst> &v, int rpb, hipStream_t s)
{
    TM_REQUIRE(!v.empty() && (int)v.size() <= kPersistInst, "persistent batch: 1 to 4 instances");
    const int prec = v[0].st[0].spinor_prec;
    TM_REQUIRE(prec != TM_F64, "the persistent batch kernel takes FP32-arithmetic solvers");
    tm_ctx *c0 = v[0].c;
    bool recon8 = false;
    for (const auto &q : v) {
        // the link copies the stage forms read (the same choice as the
        // multi-instance launches of the same stages)
        MultiDslash m;
        std::vector<tm_ctx *> cs(1, q.c);
        for (int st = 0; st < 4; st++) {
            TM_REQUIRE(q.st[st].spinor_prec == prec, "batched solves share precision");
            multi_dslash_prepare(m, cs, std::vector<DslashCall>(1, q.st[st]), rpb, s);
        }
        TM_REQUIRE(recon12_ok(q.c, prec) == recon12_ok(c0, prec), "batched instances must share the link format");
        if (&q == &v[0]) recon8 = m.recon8;
        TM_REQUIRE(m.recon8 == recon8, "batched instances must share the link format");
    }
    pb.prec = prec;
    pb.rpb = rpb;
    pb.recon12 = recon12_ok(c0, prec);
    pb.recon8 = recon8;
    multi_dispatch(pb.prec, pb.recon12, pb.recon8,
                   [&]<typename SS, typename LS, typename T>() { persist_fill<SS, LS, T>(pb, v, s); });
}

bool persist_launch(PersistBatch &pb, int iters, unsigned long long spin_limit, hipStream_t s)
{
    TM_REQUIRE(iters >= 1, "iters must be >= 1");
    pb.iters = iters;
    pb.spin_limit = spin_limit;
    // the barrier state starts at zero (a launch that gave up may have left
    // it set)
    TM_HIP(hipMemsetAsync(pb.bar, 0, pb.sync_bytes, s));
    bool ok = false;
    multi_dispatch(pb.prec, pb.recon12, pb.recon8,
                   [&]<typename SS, typename LS, typename T>() { ok = persist_go<SS, LS, T>(pb, s); });
    return ok;
}

bool persist_failed(const PersistBatch &pb, hipStream_t s)
{
    unsigned fail = 0;
    TM_HIP(hipMemcpyAsync(&fail, (const unsigned *)pb.bar + 17 * kBarLine, sizeof(fail), hipMemcpyDeviceToHost, s));
    TM_HIP(hipStreamSynchronize(s));
    return fail != 0;
}

int dslash_site_blocks(tm_ctx *c) { return (c->geo.vh + kSites - 1) / kSites; }

// launches over several lattices take the form of several right-hand sides per
// block for one, too
int multi_rhs_per_block(const std::vector<std::pair<tm_ctx *, int>> &inst, int prec)
{
    std::vector<std::pair<int, int>> v;
    for (const auto &[c, nrhs] : inst) v.push_back({dslash_site_blocks(c), nrhs});
    tm_ctx *c = inst[0].first;
    long slots = 0;
    multi_dispatch(prec, recon12_ok(c, prec), recon8_wanted(c) && c->links8_usable,
                   [&]<typename SS, typename LS, typename T>() { slots = slots_of<SS, LS, T>(c); });
    return rhs_per_block(v, slots, slots);
}

void dslash_cost(tm_ctx *c, const DslashCall &dc, double &bytes, double &flops)
{
    const double sites = (double)c->geo.vh, n = dc.nrhs;
    const double sb = 12.0 * prec_bytes(dc.spinor_prec);  // one half-site spinor
    // link entries per site (8 directions) and bytes per complex entry
    double lb;
    const int par = recon12_ok(c, dc.spinor_prec) && !dc.links18 ? 6 : 9;
    switch (dc.spinor_prec) {
    case TM_F64: lb = !dc.links18 && recon8_wanted(c) && c->links8_usable ? 64.0 : 16.0 * par; break;
    case TM_F32: lb = 8.0 * par; break;
    default: lb = c->half_links_f32 ? 8.0 * 9 : 4.0 * par; break;
    }
    double per = 2 * sb;  // input once, output once
    double fl = 1320 + 72;
    if (dc.has_own) {
        per += sb;
        fl += 96;
    }
    if (dc.epi == 1) fl += 48;
    if (dc.epi == 3) {
        per += dc.out ? sb : 0;  // b read, out perhaps not written
        fl += 72;
    }
    if (dc.epi == 2) {
        per += sb;  // r read; the output is r itself (written once)
        fl += 96;
        if (dc.rho) {
            per += 2 * sb;
            fl += 96;
        }
    }
    bytes = sites * (n * per + 8 * lb);
    flops = sites * n * fl;
}

void launch_dslash(tm_ctx *c, const DslashCall &dc, hipStream_t s)
{
    TM_REQUIRE(c->have_gauge, "no gauge field set");
    {
        double b, f;
        dslash_cost(c, dc, b, f);
        account(c, b, f);
    }
    switch (dc.spinor_prec) {
    // FP64 (the plain solver and the reliable updates): 12-parameter FP64
    // links in the context's format, the third row rebuilt exactly up to rounding
    case TM_F64:
        if (!dc.links18 && recon8_wanted(c) && ensure_links8d(c, s)) {
            launch_t<double2, L8D, double>(c, dc, s);
        } else if (recon12_ok(c, TM_F64) && !dc.links18) {
            ensure_links12d(c, s);
            launch_t<double2, L12D, double>(c, dc, s);
        } else {
            launch_t<double2, double2, double>(c, dc, s);
        }
        break;
    case TM_F32:
        if (recon12_ok(c, TM_F32)) {
            ensure_links12f(c, s);
            launch_t<float2, L12F, float>(c, dc, s);
        } else {
            ensure_links32(c, s);
            launch_t<float2, float2, float>(c, dc, s);
        }
        break;
    // FP16/BF16 spinors: binary16 links in the context's format (all 18
    // parameters or 12 with the third row rebuilt; the solvers' choice)
    // unless the caller asked for the FP32 copy
    case TM_F16:
        if (c->half_links_f32) {
            ensure_links32(c, s);
            launch_t<h2, float2, float>(c, dc, s);
        } else if (recon12_ok(c, TM_F16)) {
            ensure_links12(c, s);
            launch_t<h2, L12, float>(c, dc, s);
        } else {
            ensure_links16(c, s);
            launch_t<h2, h2, float>(c, dc, s);
        }
        break;
    case TM_BF16:
        if (c->half_links_f32) {
            ensure_links32(c, s);
            launch_t<b2, float2, float>(c, dc, s);
        } else if (recon12_ok(c, TM_BF16)) {
            ensure_links12(c, s);
            launch_t<b2, L12, float>(c, dc, s);
        } else {
            ensure_links16(c, s);
            launch_t<b2, h2, float>(c, dc, s);
        }
        break;
    default: throw TmError{TM_ERR_ARG, "bad spinor precision"};
    }
}
