// Internal definitions of the gfx950 twisted-mass library: complex arithmetic,
// storage precisions, lattice geometry, the context and the kernel launchers.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <map>
#include <stdexcept>
#include <string>
#include <type_traits>
#include <vector>

#include "tm.h"

// ---------------------------------------------------------------- errors

struct TmError {
    int status;
    std::string msg;
};

#define TM_HIP(call)                                                                   \
    do {                                                                               \
        hipError_t e_ = (call);                                                        \
        if (e_ != hipSuccess)                                                          \
            throw TmError{TM_ERR_HIP, std::string(#call) + ": " + hipGetErrorString(e_)}; \
    } while (0)

#define TM_REQUIRE(cond, msg)                                 \
    do {                                                      \
        if (!(cond)) throw TmError{TM_ERR_ARG, (msg)};        \
    } while (0)

// ---------------------------------------------------------------- complex

template <typename T>
struct cx {
    T r, i;
};

template <typename T>
__host__ __device__ __forceinline__ cx<T> cmk(T r, T i) { return cx<T>{r, i}; }
template <typename T>
__host__ __device__ __forceinline__ cx<T> operator+(cx<T> a, cx<T> b) { return {a.r + b.r, a.i + b.i}; }
template <typename T>
__host__ __device__ __forceinline__ cx<T> operator-(cx<T> a, cx<T> b) { return {a.r - b.r, a.i - b.i}; }
template <typename T>
__host__ __device__ __forceinline__ cx<T> operator*(cx<T> a, cx<T> b)
{
    return {a.r * b.r - a.i * b.i, a.r * b.i + a.i * b.r};
}
template <typename T>
__host__ __device__ __forceinline__ cx<T> operator*(T s, cx<T> a) { return {s * a.r, s * a.i}; }
// a * i
template <typename T>
__host__ __device__ __forceinline__ cx<T> times_i(cx<T> a) { return {-a.i, a.r}; }
template <typename T>
__host__ __device__ __forceinline__ cx<T> conjg(cx<T> a) { return {a.r, -a.i}; }
// acc += a * b
template <typename T>
__host__ __device__ __forceinline__ void cmac(cx<T> &acc, cx<T> a, cx<T> b)
{
    acc.r = fma(a.r, b.r, acc.r);
    acc.r = fma(-a.i, b.i, acc.r);
    acc.i = fma(a.r, b.i, acc.i);
    acc.i = fma(a.i, b.r, acc.i);
}
// acc += conj(a) * b
template <typename T>
__host__ __device__ __forceinline__ void cmac_conj(cx<T> &acc, cx<T> a, cx<T> b)
{
    acc.r = fma(a.r, b.r, acc.r);
    acc.r = fma(a.i, b.i, acc.r);
    acc.i = fma(a.r, b.i, acc.i);
    acc.i = fma(-a.i, b.r, acc.i);
}

// ---------------------------------------------------------------- storage types

// IEEE binary16 pair and bfloat16 pair, 4 bytes per complex value.
// tag types of the 12-parameter link formats (Dslash template argument):
// binary16 rows and FP64 rows
struct L12 {};
struct L12D {};
struct L12F {};
// 8-parameter FP64 links (appendix A.1): [8 directions][4][vh] double2
struct L8D {};

struct alignas(4) h2 {
    _Float16 x, y;
};
struct alignas(4) b2 {
    uint16_t x, y;
};

__host__ __device__ __forceinline__ float bf16_to_f32(uint16_t v)
{
    union { uint32_t u; float f; } c;
    c.u = ((uint32_t)v) << 16;
    return c.f;
}
// two values as stored, x in the low half: round to nearest even, NaN stays NaN
// (one v_cvt_pk_bf16_f32; the same rounding in integer code was about twelve
// instructions a pair, and three of the four waves of a hopping block waited for
// them: Schur operator, 24^4, 12 right-hand sides, 207 us against 172)
__device__ __forceinline__ uint32_t bf16_pair(float x, float y)
{
    typedef __bf16 bv2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, bv2{(__bf16)x, (__bf16)y});
}

template <typename S>
struct StoreTraits;
template <>
struct StoreTraits<double2> {
    using real = double;
    __device__ __forceinline__ static cx<double> ld(const double2 *p, size_t k)
    {
        double2 v = p[k];
        return {v.x, v.y};
    }
    __device__ __forceinline__ static void st(double2 *p, size_t k, cx<double> v) { p[k] = make_double2(v.r, v.i); }
};
template <>
struct StoreTraits<float2> {
    using real = float;
    __device__ __forceinline__ static cx<float> ld(const float2 *p, size_t k)
    {
        float2 v = p[k];
        return {v.x, v.y};
    }
    __device__ __forceinline__ static void st(float2 *p, size_t k, cx<float> v) { p[k] = make_float2(v.r, v.i); }
};
template <>
struct StoreTraits<h2> {
    using real = float;
    __device__ __forceinline__ static cx<float> ld(const h2 *p, size_t k)
    {
        h2 v = p[k];
        return {(float)v.x, (float)v.y};
    }
    __device__ __forceinline__ static void st(h2 *p, size_t k, cx<float> v)
    {
        h2 o;
        o.x = (_Float16)v.r;
        o.y = (_Float16)v.i;
        p[k] = o;
    }
};
template <>
struct StoreTraits<b2> {
    using real = float;
    __device__ __forceinline__ static cx<float> ld(const b2 *p, size_t k)
    {
        b2 v = p[k];
        return {bf16_to_f32(v.x), bf16_to_f32(v.y)};
    }
    __device__ __forceinline__ static void st(b2 *p, size_t k, cx<float> v)
    {
        p[k] = __builtin_bit_cast(b2, bf16_pair(v.r, v.i));
    }
};

// load a complex of storage S converted to arithmetic type T
template <typename T, typename S>
__device__ __forceinline__ cx<T> ldT(const S *p, size_t k)
{
    auto v = StoreTraits<S>::ld(p, k);
    return {(T)v.r, (T)v.i};
}
template <typename T, typename S>
__device__ __forceinline__ void stT(S *p, size_t k, cx<T> v)
{
    if constexpr (std::is_same<S, h2>::value && std::is_same<T, double>::value) {
        // one rounding FP64 -> binary16 (not through FP32, whose rounding
        // could move a value onto a binary16 tie)
        h2 o;
        o.x = (_Float16)v.r;
        o.y = (_Float16)v.i;
        p[k] = o;
    } else {
        using R = typename StoreTraits<S>::real;
        StoreTraits<S>::st(p, k, cx<R>{(R)v.r, (R)v.i});
    }
}

static inline size_t prec_bytes(int prec)
{
    switch (prec) {
    case TM_F64: return 16;
    case TM_F32: return 8;
    case TM_F16: return 4;
    case TM_BF16: return 4;
    }
    return 0;
}

// ---------------------------------------------------------------- geometry

// Lattice geometry for kernels (passed by value).  Half-site index i of parity
// p is s >> 1 with s = x + Lx*(y + Ly*(z + Lz*t)); the row q = y + Ly*(z + Lz*t)
// gives i = (x >> 1) + (Lx/2) * q.
//
// The three divisions of that decomposition are by extents known on the host:
// n / d = (2n m >> 32) >> s for 0 <= n < 2^31 with s = ceil(log2 d) and
// m = floor(2^(31+s) / d) + 1, two instructions and a shift where a division
// by a run-time divisor is about twenty.
struct FastDiv {
    unsigned m, s;
};
inline FastDiv fast_div(int d)
{
    unsigned s = 0;
    while ((1ll << s) < d) s++;
    return FastDiv{(unsigned)((1ull << (31 + s)) / (unsigned)d + 1), s};
}
__host__ __device__ __forceinline__ int operator/(int n, FastDiv d)
{
    return (int)((unsigned)(((unsigned long long)(2u * (unsigned)n) * d.m) >> 32) >> d.s);
}

struct Geo {
    int L[4];
    int lxh;   // Lx / 2
    int vh;    // V / 2
    int vsh;   // half-sites per time slice, Lx*Ly*Lz / 2
    int hs;    // plane stride of half-site fields (sites), see half_stride
    FastDiv by_lxh, by_y, by_z;  // division by lxh, L[1], L[2]
};

// Half-site fields are stored [rhs][spin*3 + colour][hs] with hs >= vh; the
// hs - vh pad sites at the end of every plane are never read for a result
// (their contents are unspecified).  hs is vh rounded up to an odd multiple
// of 32 sites: with a power-of-two plane stride the 12 planes of a site (and
// the right-hand sides of a thread) fall on the same cache sets and memory
// channels, and the neighbour gathers of the hopping kernel lose ~7% of
// their bandwidth to the conflicts.
inline int half_stride(int vh)
{
    int q = (vh + 31) / 32;
    if (q % 2 == 0) q++;
    return 32 * q;
}

__device__ __forceinline__ void eo_coords(const Geo &g, int p, int i, int &x, int &y, int &z, int &t)
{
    const int q = i / g.by_lxh;
    const int xh = i - q * g.lxh;
    const int q2 = q / g.by_y;
    y = q - q2 * g.L[1];
    t = q2 / g.by_z;
    z = q2 - t * g.L[2];
    x = 2 * xh + ((p ^ (y + z + t)) & 1);
}

__device__ __forceinline__ int eo_index(const Geo &g, int x, int y, int z, int t)
{
    return (x >> 1) + g.lxh * (y + g.L[1] * (z + g.L[2] * t));
}

// Logical block index with contiguous chunks of blocks on each of the 8 XCDs:
// hardware dispatches consecutive workgroups round-robin over the XCDs, so
// block b runs on XCD b % 8; mapping it to chunk (b % 8) keeps lattice
// neighbours (nearby half-site indices) inside one XCD's L2.
__host__ __device__ __forceinline__ int xcd_block(int b, int nblk)
{
    // XCD k receives hardware blocks k, k+8, ...: base + (k < rem) of them
    int base = nblk >> 3, rem = nblk & 7;
    int k = b & 7, m = b >> 3;
    return k * base + (k < rem ? k : rem) + m;
}

// ---------------------------------------------------------------- context

struct DevBuf {
    void *p = nullptr;
    size_t bytes = 0;
};

struct tm_ctx {
    int device = 0;
    tm_lattice lat{};
    Geo geo{};
    long V = 0;
    double kappa = 0, eps = 0;
    int t_bc = -1;
    // internal links per parity of the output site: [8 directions][9][vh]
    // direction d < 4: U_d(x) (forward hop); d >= 4: U_{d-4}(x - d)^dag
    // (backward hop), boundary phase folded in
    void *links64[2] = {nullptr, nullptr};
    void *links32[2] = {nullptr, nullptr};
    void *links16[2] = {nullptr, nullptr};  // IEEE binary16 copy (FP16/BF16 spinors)
    // binary16 12-parameter copy: the first two rows, [8 directions][6][vh]
    void *links12[2] = {nullptr, nullptr};
    // FP64 and FP32 12-parameter copies, same layout
    void *links12d[2] = {nullptr, nullptr};
    void *links12f[2] = {nullptr, nullptr};
    // FP64 8-parameter copy (a2, a3, b1 or -c1, phases; see misc.hip), [8][4][vh]
    void *links8d[2] = {nullptr, nullptr};
    bool have_gauge = false;
    bool have_links32 = false;
    bool have_links16 = false;
    bool have_links12 = false;
    bool have_links12d = false;
    bool have_links12f = false;
    bool have_links8d = false;
    // the 8-parameter copy was built and every link's first row has
    // |a2|^2 + |a3|^2 >= kRecon8MinN (the reconstruction divides by it)
    bool links8_usable = false;
    // binary16 link format of the FP16/BF16-spinor kernels: 18 or 12
    // parameters (12 reads a third fewer link bytes; measured no slower at 12
    // RHS and 9-24% faster at 1-4 RHS per call)
    int link_recon = 12;
    // largest deviation of the gauge field from SU(3) measured at ingest,
    // max over links of max(|U U^dag - 1|, |det U - 1|) entrywise; the
    // 12-parameter format of a precision is used only while this stays
    // below that precision's rounding scale (recon12_ok)
    double su3_dev = 0;
    // FP16/BF16-spinor Dslash launches read the FP32 links instead of the
    // binary16 copy (set by tm_dslash for link_prec = TM_F32)
    bool half_links_f32 = false;
    // links of the FP16/BF16-spinor kernels when no call overrides them
    // (tm_set_half_spinor_links): false = binary16 copy, true = FP32 (18)
    bool half_links_f32_default = false;
    int cus = 256;  // compute units of the device (fewer in a partition)
    std::map<std::string, DevBuf> ws;
    size_t ws_total = 0;  // bytes in ws
    // bytes that ws may hold (0: no limit), TM_WORKSPACE_LIMIT in the environment
    // when the context is created; an allocation beyond it fails as on a full device
    size_t ws_limit = 0;
    int ring_users = 0;  // solves that hold the ring of search directions
    std::string err;
    hipStream_t stream = nullptr;  // stream of the current loop-driver call
    // pinned host staging for scalar read-back
    void *host_pinned = nullptr;
    size_t host_pinned_bytes = 0;
    void *host_up = nullptr;  // pinned slots of asynchronous uploads (host_upload_slot)
    size_t host_up_bytes = 0;
    // learned preconditioner (ptc.hip): channel count (0 = no weights),
    // Adam step counter, training-pair store (capacity, count, precision)
    int ptc_nc = 0;
    // network arithmetic, spin mixing on the matrix cores either way: TM_F32 (the
    // bits of FP32 FMA chains) or TM_BF16 (BF16 weights and activations, FP32
    // accumulation)
    int ptc_arith = TM_F32;
    long ptc_step = 0;
    int ptc_cap = 0, ptc_n = 0, ptc_store = TM_F32;
    // algorithmic work of the kernels launched on this context so far
    // (compulsory device-memory bytes and flops by the conventions of tm.h);
    // acct_pause > 0 while launches are recorded into a graph that is
    // accounted per replay instead
    double acct_bytes = 0, acct_flops = 0;
    int acct_pause = 0;
    // set for the duration of an allocation-free call: ws_get refuses to
    // allocate
    bool no_alloc = false;
};

// 12-parameter links for kernels of spinor precision prec: the format asks
// for 12 (or 8, which the FP64 kernels alone read, the others taking 12)
// and the links are special unitary to that precision's rounding (the third
// row is rebuilt from the first two assuming U in SU(3))
inline bool recon12_ok(const tm_ctx *c, int prec)
{
    if (c->link_recon != 12 && c->link_recon != 8) return false;
    const double lim = prec == TM_F64 ? 1e-12 : prec == TM_F32 ? 1e-6 : 1e-3;
    return c->su3_dev <= lim;
}

// smallest |a2|^2 + |a3|^2 (over the links) with which the 8-parameter form
// is used; fields with a link closer to diagonal (unit links) keep 12
constexpr double kRecon8MinN = 1e-10;

// the FP64 kernels read 8-parameter links: asked for, special unitary to
// FP64 rounding; links8_usable is settled when the copy is built
inline bool recon8_wanted(const tm_ctx *c) { return c->link_recon == 8 && c->su3_dev <= 1e-12; }

inline void account(tm_ctx *c, double bytes, double flops)
{
    if (c->acct_pause) return;
    c->acct_bytes += bytes;
    c->acct_flops += flops;
}

void *ws_get(tm_ctx *c, const std::string &name, size_t bytes);
// bytes that an allocation may take now
size_t ws_room(tm_ctx *c);
void *host_stage(tm_ctx *c, size_t bytes);
// Pinned staging slot `slot` (< kUpSlots) of `bytes` for an asynchronous
// upload on stream s.  A slot's previous copy must have completed before it
// is reused (the callers synchronise the stream in between).
constexpr int kUpSlots = 5;
void *host_upload_slot(tm_ctx *c, int slot, size_t bytes, hipStream_t s);
void ensure_links32(tm_ctx *c, hipStream_t s);
void ensure_links16(tm_ctx *c, hipStream_t s);
void ensure_links12(tm_ctx *c, hipStream_t s);
void ensure_links12d(tm_ctx *c, hipStream_t s);
// builds the 8-parameter copy if needed; true when the FP64 kernels use it
bool ensure_links8d(tm_ctx *c, hipStream_t s);
void ensure_links12f(tm_ctx *c, hipStream_t s);

// ---------------------------------------------------------------- dslash

// spin-diagonal operator: diag(u, u, l, l) in the chiral basis (R(eps),
// R^-1, gamma5 and their products are all of this form)
struct SpinDiag {
    cx<double> u, l;
};

static inline SpinDiag sd_scalar(double a) { return {{a, 0}, {a, 0}}; }
static inline SpinDiag sd_mul(SpinDiag a, SpinDiag b) { return {a.u * b.u, a.l * b.l}; }
static inline SpinDiag sd_twist(double eps)  // R = 1 + i eps gamma5
{
    return {{1.0, eps}, {1.0, -eps}};
}
static inline SpinDiag sd_twist_inv(double eps)  // R^-1 = (1 - i eps gamma5)/(1 + eps^2)
{
    double d = 1.0 / (1.0 + eps * eps);
    return {{d, -eps * d}, {d, eps * d}};
}
static inline SpinDiag sd_gamma5() { return {{1.0, 0}, {-1.0, 0}}; }

// out(x) = D_own own(x) + D_hop (Hop[in])(x),
// x over the half sites of parity out_parity; Hop is the hopping sum without
// the -kappa factor (fold it into D_hop).  dag selects the adjoint projector
// placement ((1+gamma) forward, (1-gamma) backward), i.e. Hop^dag.
struct DslashCall {
    void *out;
    const void *in;
    const void *own;  // may be null when D_own = 0
    int nrhs;
    int out_parity;
    int dag;
    int spinor_prec;  // TM_F64 with FP64 links, else FP32 links
    SpinDiag d_own, d_hop;
    bool has_own;
    // fused epilogue (0 store, 1 store + partial |out|^2, 2 CG update of r and
    // rho with partial |r|^2, |rho|^2, 3 residual r - result with its partial
    // norm; see dslash.hip)
    int epi = 0;
    void *r = nullptr, *rho = nullptr;
    const struct CGScalars *sc = nullptr;
    double *part = nullptr;  // [quantity][nrhs][dslash_site_blocks]
    // store forms with dag and without an own-site term: if > 0, one more block
    // per right-hand side sums `part` (|q|^2 of an earlier launch) and sets
    // alpha in sc, for ring position alpha - 1, while the others hop
    int alpha = 0;
    // store forms without dag and own-site term: if > 0, one more block per
    // right-hand side runs the beta step of the iteration before on `part`
    // ([2][nrhs][blocks]) with the threshold delta (which may be 0)
    int beta = 0;
    double delta = 0;
    // FP64 only: read all 18 parameters of the FP64 links whatever the
    // format (the exact operator for reliable updates and true residuals)
    bool links18 = false;
};

void launch_dslash(tm_ctx *c, const DslashCall &dc, hipStream_t s);
int dslash_site_blocks(tm_ctx *c);
// algorithmic bytes (each field and link read once, each output written
// once) and flops (1320 per site and RHS for the hopping term, 72 for its
// spin-diagonal coefficient, 96 for the own-site term, 48 per fused norm or
// update) of one launch of dc on this context's link format
void dslash_cost(tm_ctx *c, const DslashCall &dc, double &bytes, double &flops);

// One launch over several contexts (lattices), one DslashCall each; all
// share precision and operator form; rpb right-hand sides per block.  prepare() builds the launch arguments on the host;
// launch() is one kernel launch per chunk of instances (capturable).
struct MultiDslash {
    // per chunk of at most kMultiInst instances: the kernel-argument block
    // (instance records + block offsets) and the grid it covers
    std::vector<std::vector<unsigned char>> args;
    std::vector<int> grid;
    int prec = 0, dag = 0, own = 0, epi = 0, n = 0;
    bool recon12 = false;  // links in the 12-parameter format
    bool recon8 = false;   // FP64 links in the 8-parameter format
};
constexpr int kMultiInst = 16;  // instances per launch (kernel-argument space)
void multi_dslash_prepare(MultiDslash &m, const std::vector<tm_ctx *> &cs, const std::vector<DslashCall> &dcs, int rpb,
                          hipStream_t s);
// right-hand sides per block of a launch over several (context, nrhs) in prec
int multi_rhs_per_block(const std::vector<std::pair<tm_ctx *, int>> &inst, int prec);
void multi_dslash_launch(const MultiDslash &m, hipStream_t s);

// The low-precision solvers keep the search directions of up to kCgRing
// iterations in a ring of buffers and add them to the FP32 solution x together,
// in the order of the iterations (the same FP32 sums as one at a time): x and
// the directions move (4 m - 1) / m low-precision and 2 / m FP32 accesses per
// element and iteration instead of 3 and 2.  Bound: memory; FP16, 32^3 x 64, 12
// right-hand sides: 462 us per iteration for m = 8, 729 (5.8 TB/s) for
// m = 1, a mixed solve of 157 iterations 601 ms against 646.
constexpr int kCgRing = 8;
// The ring lives in the workspace "s_p_ring", which an allocation that would fail
// takes back from a context between its solves (ws_get).
// Ring of search directions: ring position q holds the direction of the q-th
// iteration since x was last brought up to date.
struct CgRing {
    int m = 1;                      // 1, 2, 4 or 8
    void *p[kCgRing] = {nullptr};
};

// Persistent batch: `iters` CG iterations of up to kPersistInst instances in
// one cooperative launch (grid barriers between the stages, bounded waits);
// solvers with FP32 arithmetic (FP32, FP16 or BF16 storage) only.
constexpr int kPersistInst = 4;
struct PersistInst {
    tm_ctx *c = nullptr;
    DslashCall st[4];       // the four stage forms of one CG iteration
    CgRing ring;            // directions (stages 1 and 2 read position 0 as given in st)
    void *x = nullptr;      // solution accumulator of the update
    CGScalars *sc = nullptr;
    double delta = 0;       // reliable-update threshold (0: none)
};
struct PersistBatch {
    void *dev_args = nullptr;          // launch parameters (device, owned by the first context)
    size_t args_bytes = 0, sync_bytes = 0;
    int grid = 0, work = 0, iters = 0;
    int blocks_per_cu = 0;             // cap on resident blocks per CU (0: as many as fit)
    int prec = 0, rpb = 1;
    bool recon12 = false, recon8 = false;
    void *bar = nullptr;               // barrier state (device)
    unsigned long long spin_limit = 0;
};
bool persist_supported(int device);
void persist_prepare(PersistBatch &pb, const std::vector<PersistInst> &v, int rpb, hipStream_t s);
// false if the runtime refused the cooperative launch (nothing launched)
bool persist_launch(PersistBatch &pb, int iters, unsigned long long spin_limit, hipStream_t s);
// reads the barrier state (synchronises the stream): true if a wait gave up
bool persist_failed(const PersistBatch &pb, hipStream_t s);

// ---------------------------------------------------------------- blas

// All vectors: half layout [nrhs][12][hs] of the given precision.
// Per-RHS scalars live in device memory (double).
void launch_spin_diag(tm_ctx *c, void *out, const void *in, int prec, int nrhs, SpinDiag d,
                      hipStream_t s);
void launch_copy_convert(tm_ctx *c, void *out, int out_prec, const void *in, int in_prec, int nrhs,
                         const double *dscale /* device per-rhs or null */, hipStream_t s);
// y = a*x + b*y with host scalars (same prec)
void launch_axpby_host(tm_ctx *c, void *y, const void *x, int prec, int nrhs, double a, double b,
                       hipStream_t s);
void launch_zero(tm_ctx *c, void *y, int prec, int nrhs, hipStream_t s);
// y[r] += a_dev[r] * x[r]
void launch_axpy_dev(tm_ctx *c, void *y, int yprec, const void *x, int xprec, int nrhs, const double *a_dev,
                     hipStream_t s);
// out = scale[r] in per right-hand side, converted, and the partial |out|^2 of
// the stored values into part[nrhs][norm_blocks]; out = null: the norm only.
// in_prec is out_prec or TM_F64.
void launch_convert_norm(tm_ctx *c, void *out, int out_prec, const void *in, int in_prec, int nrhs,
                         const double *dscale, double *part, hipStream_t s);
// partial |v|^2 into part[nrhs][norm_blocks]
int norm_blocks(tm_ctx *c);
void launch_partial_norm2(tm_ctx *c, const void *v, int prec, int nrhs, double *part, hipStream_t s);
// dev_out[k] = sum of part[k][0 .. nblk), k < n, in a fixed order
void launch_sum_partials(const double *part, int nblk, int n, double *dev_out, hipStream_t s);
// per-rhs |v|^2 into dev_out[nrhs] (device doubles), deterministic
void launch_norm2(tm_ctx *c, const void *v, int prec, int nrhs, double *dev_out, hipStream_t s);

// CG building blocks (blas.hip; the iteration itself is in runtime.hip).
struct CGScalars {
    double rr;       // |r|^2 (normal residual)
    double qq;       // |Ahat p|^2
    double alpha, beta;
    double hist[kCgRing];  // alpha per position of the ring
    double rho2;     // |rho|^2, iterated Schur residual
    double rho2_ref; // |rho|^2 at the last reliable update
    double target2;  // (tol |b|)^2 in the units of the vectors
    double sigma;    // scale of the low-precision vectors (MIXED/LOW)
    int active;
    int iters;
    int want_update; // reliable update requested
    int bad;         // NaN/Inf seen
};

void cg_finish_beta(tm_ctx *c, CGScalars *sc, const double *part, int nblk, int nrhs, double delta,
                    hipStream_t s);
// position pos < m - 1: p[pos + 1] = r + beta p[pos]; last position:
// x += sum_q hist[q] p[q], p[0] = r + beta p[m - 1].  A right-hand side that
// is no longer active keeps its last direction, in p[0] from the end of the
// ring on.  part: null, the beta step has run; else its partial sums, of nblk
// blocks: every block of the update forms beta itself, and the beta step follows
// later (with the next iteration's first launch).
void cg_update(tm_ctx *c, const CgRing &ring, int pos, const void *r, void *x, int prec, int xprec, int nrhs,
               const CGScalars *sc, hipStream_t s, const double *part = nullptr, int nblk = 0, double delta = 0);
// whether that form is the faster one for a solve's sizes
bool cg_beta_late(tm_ctx *c, int nrhs, int nblk, double delta);
// bytes and flops of cg_update per complex element at one position
void cg_update_cost(const CgRing &ring, int pos, int prec, int xprec, double &bytes, double &flops);
// x += sum of the first cnt directions, p[cnt] the current direction of every
// right-hand side (an incomplete round of the ring)
void cg_flush(tm_ctx *c, const CgRing &ring, int cnt, void *x, int prec, int xprec, int nrhs, const CGScalars *sc,
              hipStream_t s);

// The same scalar and vector steps for several lattices in one launch each
// (a batch's iteration): per lattice its context, CG scalars, partial sums
// and fields; all share prec and xprec.  Bit-identical to the per-lattice
// launches (the same device code per right-hand side and element).
struct CgTail {
    tm_ctx *c;
    CGScalars *sc;
    const double *partb;  // |r|^2 (and |rho|^2) partials (beta)
    int nblk;             // partial-sum blocks
    int nrhs;
    double delta;
    CgRing ring;  // the same length for all lattices
    const void *r;
    void *x;
};
void cg_tail_multi(const std::vector<CgTail> &t, int pos, int prec, int xprec, hipStream_t s);  // beta, then x and p

// ---------------------------------------------------------------- misc kernels

void launch_pack(tm_ctx *c, void *even, void *odd, const double *full, int nrhs, int prec,
                 const double *dscale, hipStream_t s);
void launch_unpack(tm_ctx *c, double *full, const void *even, const void *odd, int nrhs, int prec,
                   hipStream_t s);
void launch_gauge_ingest(tm_ctx *c, const double *U, hipStream_t s);
// max over the 4V links of the canonical field U (device) of
// max(|U U^dag - 1|, |det U - 1|) entrywise; synchronises s
double gauge_su3_deviation(tm_ctx *c, const double *U, hipStream_t s);
void launch_links_to_f32(tm_ctx *c, hipStream_t s);
void launch_links_to_f16(tm_ctx *c, hipStream_t s);
// first two rows of every link, rounded once to binary16: [8][6][vh] per parity
void launch_links_to_r12(tm_ctx *c, hipStream_t s);
// first two rows of every link in FP64: [8][6][vh] per parity
void launch_links_to_r12d(tm_ctx *c, hipStream_t s);
// builds links8d for both parities; returns the smallest |a2|^2 + |a3|^2
double launch_links_to_r8d(tm_ctx *c, hipStream_t s);
// first two rows of every link rounded once to FP32: [8][6][vh] per parity
void launch_links_to_r12f(tm_ctx *c, hipStream_t s);
// Z4 noise for noise index r into FP64 half fields: n_off x (12 with
// spin-colour dilution, else 1) RHS; with t_period > 0 RHS group q keeps the
// slices t = o_first + q (mod t_period) only (time dilution, coherent when
// t_period < Lt)
void launch_noise(tm_ctx *c, void *even, void *odd, uint64_t seed, long r, int dilution, hipStream_t s,
                  int t_period = 0, int o_first = 0, int n_off = 1);
// per time slice 4x4 colour-traced outer products C[b][a](t) = sum_x sum_c v_{bc} w*_{ac}
// accumulated over nrhs pairs and both parities, FP64; out device [Lt][16] complex.
// Only the slices t0, t0 + dt, ... are computed; the others are zero.
void launch_outer_slices(tm_ctx *c, const void *ve, const void *vo, const void *we, const void *wo,
                         int nrhs, double *dev_out /* [Lt][16][2] */, hipStream_t s, int t0 = 0, int dt = 1);
