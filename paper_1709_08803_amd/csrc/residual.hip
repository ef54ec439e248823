// Residual F(u) of the discretised boundary-integral system (Section 3.1) on gfx950.
//
// Four kernels, stream-ordered:
//   k_integrate   unpack u and integrate f_x along each slice (trapezoidal rule)
//   k_records     y-derivatives at the nodes; source-node records for S and B;
//                 collocation-point records at (x_{k+1/2}, y_l)
//   k_allpairs    the dense sums of eq. (new_finite_boundary_integral): every
//                 collocation point against every node of both boundaries and
//                 both y-images (hot loop)
//   k_finalize    reduction of the all-pairs partial sums, closed-form S2
//                 integral, 2 pi term, dynamic condition, radiation rows, and
//                 the row order of Appendix B
// The three node-level kernels take a PairDesc by value; their _batched forms
// serve many problems in one launch, each workgroup finding its problem from
// the first-workgroup offsets in the descriptors.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <type_traits>
#include <vector>

#include "bim_common.h"

namespace bim {

namespace {

constexpr double kTwoPi = 6.283185307179586476925286766559;

inline int cdiv(long a, long b) { return (int)((a + b - 1) / b); }

// ------------------------------------------------------------------ rsqrt
// FP32: the hardware reciprocal square root (about 1 ulp).
__device__ __forceinline__ float rsq(float x) { return __builtin_amdgcn_rsqf(x); }
// FP64: an estimate y refined by one Newton-Raphson step y (1 + e/2),
// e = 1 - x y^2, whose truncation error is (3/8) e^2 relative.  The estimate is
// the FP32 reciprocal square root of x rounded to FP32 (relative error ~1e-7,
// so the refined value is good to ~2e-14, far below the parity bound of the
// sums, 1e-12 of the sum of |terms|): on gfx950 the two conversions and
// v_rsq_f32 issue in ~10 cycles per wave against ~17 for v_rsq_f64, and one
// first-order step costs one FMA less than the second-order one the FP64
// estimate would otherwise get (the sums are bound by VALU issue).  x is a
// squared distance or a positive quadratic form well inside the FP32 range.
__device__ __forceinline__ double rsq(double x) {
    const double y = (double)__builtin_amdgcn_rsqf((float)x);
    const double e = fma(-x * y, y, 1.0);
    return fma(0.5 * y, e, y);
}

// ------------------------------------------------------------------ batched lookup
// Problem of workgroup b in a batched node-level launch: the number of
// problems whose first workgroup is <= b, minus one (a wave-wide count over
// the descriptors; uniform across the workgroup).  PART selects the launch.
template <int PART>
__device__ __forceinline__ int first_block(const PairDesc &D) {
    return PART == 0 ? D.blk_int : PART == 1 ? D.blk_rec : D.blk_fin;
}
template <int PART>
__device__ __forceinline__ int find_problem(const PairDesc *__restrict__ descs, int count, int b) {
    const int lane = threadIdx.x & 63;
    int n = 0;
    for (int base = 0; base < count; base += 64) {
        const int i = base + lane;
        const bool le = i < count && first_block<PART>(descs[i]) <= b;
        n += __popcll(__ballot(le));
    }
    return n - 1;
}

// ------------------------------------------------------------------ A1: unpack + x-integration
// f_{1,j} + trapezoidal integral of f_x along slice j (Section 3.1).  One wave
// per (field, slice): 64-wide inclusive scans of the trapezoid increments with
// the running total carried from one 64-node segment to the next.
__device__ __forceinline__ void integrate_body(const PairDesc &D, int idx) {
    const int N = D.N, M = D.M;
    const int f = idx / M, j = idx - f * M;  // idx = field * M + slice
    const int lane = threadIdx.x;
    const double *s = D.u + (size_t)f * (N + 1) * M + (size_t)j * (N + 1);
    double *o = D.nodes + ((size_t)f * M + j) * N;
    const double hdx = 0.5 * D.dx;
    double carry = s[0];
    for (int base = 0; base < N; base += 64) {
        const int i = base + lane;
        // increment into node i: (dx/2)(f_x,i-1 + f_x,i), zero for the first node
        double v = (i > 0 && i < N) ? hdx * (s[i] + s[i + 1]) : 0.0;
        for (int o2 = 1; o2 < 64; o2 <<= 1) {
            const double y = __shfl_up(v, o2, 64);
            if (lane >= o2) v += y;
        }
        if (i < N) o[i] = carry + v;
        carry += __shfl(v, 63, 64);
    }
}
__global__ __launch_bounds__(64) void k_integrate(PairDesc D) { integrate_body(D, blockIdx.x); }
__global__ __launch_bounds__(64) void k_integrate_batched(const PairDesc *__restrict__ descs, int count) {
    const PairDesc &D = descs[find_problem<0>(descs, count, blockIdx.x)];
    if (!D.active) return;
    integrate_body(D, blockIdx.x - D.blk_int);
}

// y-derivative of node field g at (j, i): central differences inside, the
// three-point one-sided stencil on the outer edge, zero on the symmetry line of
// a half domain (mirror of the outer stencil on a full domain).
__device__ __forceinline__ double ddy(const double *g, int j, int i, int N, int M, double dy, int half) {
    const double inv2 = 0.5 / dy;
    if (j > 0 && j < M - 1) return (g[(size_t)(j + 1) * N + i] - g[(size_t)(j - 1) * N + i]) * inv2;
    if (j == M - 1)
        return (3.0 * g[(size_t)j * N + i] - 4.0 * g[(size_t)(j - 1) * N + i] + g[(size_t)(j - 2) * N + i]) * inv2;
    if (half) return 0.0;
    return (-3.0 * g[i] + 4.0 * g[(size_t)N + i] - g[(size_t)2 * N + i]) * inv2;
}

// ------------------------------------------------------------------ records
// Node part (one thread per node of the mesh): y-derivatives of zeta and phi,
// and the source-node records of both boundaries.
template <typename T>
__device__ __forceinline__ void node_records(const PairDesc &D, int n) {
    const int N = D.N, M = D.M;
    const int j = n / N, i = n - j * N;
    const double dx = D.dx, dy = D.dy;
    const double *nodes = D.nodes;
    const double *zeta = nodes, *phi = nodes + (size_t)N * M, *psi = nodes + (size_t)2 * N * M;
    const double zy = ddy(zeta, j, i, N, M, dy, D.half);
    const double py = ddy(phi, j, i, N, M, dy, D.half);
    D.ydiv[n] = zy;
    D.ydiv[(size_t)N * M + n] = py;
    const double zx = D.u[(size_t)j * (N + 1) + 1 + i];
    const double x = D.x1 + i * dx;
    const double ci = (i == 0 || i == N - 1) ? 0.5 : 1.0;
    const double cj = (j == 0 || j == M - 1) ? 0.5 : 1.0;
    const double w = dx * dy * ci * cj;
    const bool linear = D.linear;
    // linear mode: the boundaries are the planes z = 0 and z = -1 (Section 4.2);
    // the layer densities are unchanged.
    // FP32 records are in grid units (lengths / dx, node x = its column index):
    // the double-layer and single-layer products are unchanged by the scaling
    // (w / dx^2 times K1 dx^2; w sigma / dx times K2 dx), the S2 sum carries a
    // factor 1 / dx that the all-pairs kernel removes, and s = x - x* is exact.
    const bool grid = sizeof(T) == 4;
    const double g = grid ? 1.0 / dx : 1.0;
    const double xr = grid ? (double)i : x;
    SrcRec<T> a;
    a.x = (T)xr;
    a.z = linear ? (T)0 : (T)(zeta[n] * g);
    a.zx = linear ? (T)0 : (T)zx;
    a.zy = linear ? (T)0 : (T)zy;
    a.wD = (T)(w * g * g * (phi[n] - x));
    a.ws = (T)(w * g * zx);
    a.w = (T)(w * g * g);
    a.pad = (T)0;
    ((SrcRec<T> *)D.srcS)[n] = a;
    // bottom: outward normal points down, so both layers enter with -w
    SrcRec<T> b;
    b.x = (T)xr;
    b.z = (T)((linear ? -1.0 : D.beta[n]) * g);
    b.zx = linear ? (T)0 : (T)D.beta_x[n];
    b.zy = linear ? (T)0 : (T)D.beta_y[n];
    b.wD = (T)(-w * g * g * (psi[n] - x));
    b.ws = (T)(-w * g * D.beta_x[n]);
    b.w = (T)(-w * g * g);
    b.pad = (T)0;
    ((SrcRec<T> *)D.srcB)[n] = b;
}

// Collocation part (one thread per collocation point).  tg layout: 8 arrays of
// 2 ntg entries: x*, y*, d, D*, A, B, C, sigma*; target t = st ntg + l (N-1) + k,
// st = 0 on the free surface, 1 on the bottom.  The FP32 copy tg32 holds the
// first 7 in grid units (x* = k + 1/2, y*, d / dx).  zeta_y at the two
// neighbouring nodes is formed here by the node part's own stencil.
__device__ __forceinline__ void target_records(const PairDesc &D, int t) {
    const int N = D.N, M = D.M;
    const int ntg = (N - 1) * M;
    const int st = t / ntg, r = t - st * ntg;
    const int l = r / (N - 1), k = r - l * (N - 1);
    const size_t n0 = (size_t)l * N + k, n1 = n0 + 1;
    const double dx = D.dx;
    const double xs = D.x1 + (k + 0.5) * dx, ys = D.y1 + l * D.dy;
    double d, Dst, ax, ay, sig;
    if (st == 0) {
        const double *zeta = D.nodes, *phi = D.nodes + (size_t)N * M;
        const double zx0 = D.u[(size_t)l * (N + 1) + 1 + k], zx1 = D.u[(size_t)l * (N + 1) + 2 + k];
        d = 0.5 * (zeta[n0] + zeta[n1]);
        Dst = 0.5 * (phi[n0] + phi[n1]) - xs;
        ax = 0.5 * (zx0 + zx1);
        ay = 0.5 * (ddy(zeta, l, k, N, M, D.dy, D.half) + ddy(zeta, l, k + 1, N, M, D.dy, D.half));
        sig = ax;
    } else {
        const double *psi = D.nodes + (size_t)2 * N * M;
        d = 0.5 * (D.beta[n0] + D.beta[n1]);
        Dst = 0.5 * (psi[n0] + psi[n1]) - xs;
        ax = 0.5 * (D.beta_x[n0] + D.beta_x[n1]);
        ay = 0.5 * (D.beta_y[n0] + D.beta_y[n1]);
        sig = -ax;
    }
    if (D.linear) {  // flat boundaries: elevation 0 or -1, S2 = 1/r
        d = st ? -1.0 : 0.0;
        ax = ay = 0.0;
    }
    const size_t T2 = (size_t)2 * ntg;
    const double v[8] = {xs, ys, d, Dst, 1.0 + ax * ax, 2.0 * ax * ay, 1.0 + ay * ay, sig};
    for (int q = 0; q < 8; ++q) D.tg64[q * T2 + t] = v[q];
    // FP32 copies in the grid units of the FP32 node records (x* = k + 1/2)
    const double g[7] = {0.0, 1.0 / dx, 1.0 / dx, 1.0, 1.0, 1.0, 1.0};
    for (int q = 0; q < 7; ++q) D.tg32[q * T2 + t] = (float)(q == 0 ? k + 0.5 : v[q] * g[q]);
}

// Workgroups [0, node_blocks) cover the nodes, the rest the collocation points.
__host__ __device__ __forceinline__ int node_blocks(int N, int M) { return (N * M + 255) / 256; }
__host__ __device__ __forceinline__ int record_blocks(int N, int M) {
    return node_blocks(N, M) + (2 * (N - 1) * M + 255) / 256;
}
template <typename T>
__device__ __forceinline__ void records_body(const PairDesc &D, int b) {
    const int nbn = node_blocks(D.N, D.M);
    if (b < nbn) {
        const int n = b * 256 + threadIdx.x;
        if (n < D.N * D.M) node_records<T>(D, n);
    } else {
        const int t = (b - nbn) * 256 + threadIdx.x;
        if (t < 2 * (D.N - 1) * D.M) target_records(D, t);
    }
}
template <typename T>
__global__ __launch_bounds__(256) void k_records(PairDesc D) { records_body<T>(D, blockIdx.x); }
template <typename T>
__global__ __launch_bounds__(256) void k_records_batched(const PairDesc *__restrict__ descs, int count) {
    const PairDesc &D = descs[find_problem<1>(descs, count, blockIdx.x)];
    if (!D.active) return;  // uniform over the workgroup
    records_body<T>(D, blockIdx.x - D.blk_rec);
}

// ------------------------------------------------------------------ A1 and records in one launch
// Inclusive scan over a wave of 64 in DPP steps (shifts within rows of 16 lanes,
// then the row broadcasts): a fraction of the latency of six FP64 shuffles.  Sums of two
// doubles (two-sum), as the rounding of a node's potential is most of a row's error: in one
// double, in this order, rows lay up to 1.4 times as far from extended precision as with the
// shuffles (rms at 31 x 11 8.9e-15 against 7.8e-15, 181 x 61 1.29e-14 / 1.24e-14; now 4.1e-15 and
// 8.2e-15, for 0.2 us).
struct Two {
    double hi, lo;
};
__device__ __forceinline__ Two two_add(Two a, Two b) {
    const double s = a.hi + b.hi, z = s - a.hi;
    return {s, (a.lo + b.lo) + ((a.hi - (s - z)) + (b.hi - z))};
}
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_move(double v) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)b, CTRL, ROWS, 0xf, false);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), CTRL, ROWS, 0xf, false);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
template <int CTRL, int ROWS>
__device__ __forceinline__ Two dpp_add(Two v) {
    return two_add(v, {dpp_move<CTRL, ROWS>(v.hi), dpp_move<CTRL, ROWS>(v.lo)});
}
__device__ __forceinline__ Two wave_scan(Two v) {
    v = dpp_add<0x111, 0xf>(v);  // row_shr 1, 2, 4, 8
    v = dpp_add<0x112, 0xf>(v);
    v = dpp_add<0x114, 0xf>(v);
    v = dpp_add<0x118, 0xf>(v);
    v = dpp_add<0x142, 0xa>(v);  // lane 15 of each row to the next (rows 1, 3)
    return dpp_add<0x143, 0xc>(v);  // lane 31 to rows 2, 3
}

// FP64, one problem: what k_integrate and k_records do, one workgroup per mesh row
// l.  Its y-differences need the node values of three rows of zeta and phi; each
// workgroup integrates those (7 slices with psi's) into LDS itself, which takes less
// than a second launch (bound by latency; 31 x 11: 2.8 + 3.9 -> 5.0 us; 181 x 61: 5.1 + 5.5 ->
// 9.5 us, and the gap between the launches).
__global__ __launch_bounds__(256) void k_prepare64(PairDesc D) {
    extern __shared__ double val[];  // [7][N]: zeta and phi on rows base .. base + 2, psi on row l
    const int N = D.N, M = D.M, l = blockIdx.x;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int base = l == 0 ? 0 : l == M - 1 ? M - 3 : l - 1, here = l - base;
    const double dx = D.dx, hdx = 0.5 * D.dx;
    for (int q = wave; q < 7; q += 4) {
        const int f = q < 3 ? 0 : q < 6 ? 1 : 2, j = q < 6 ? base + q % 3 : l;
        const double *s = D.u + ((size_t)f * M + j) * (N + 1);
        Two carry = {s[0], 0.0};
        for (int b0 = 0; b0 < N; b0 += 64) {
            const int i = b0 + lane;
            Two v = {0.0, 0.0};
            if (i > 0 && i < N) {  // hdx (s_i + s_i+1)
                const Two t = two_add({s[i], 0.0}, {s[i + 1], 0.0});
                v.hi = hdx * t.hi;
                v.lo = fma(hdx, t.lo, fma(hdx, t.hi, -v.hi));
            }
            v = two_add(carry, wave_scan(v));
            const double node = v.hi + v.lo;
            if (i < N) {
                val[q * N + i] = node;
                if (q == here || q == 3 + here || q == 6) D.nodes[((size_t)f * M + l) * N + i] = node;
            }
            carry = {__shfl(v.hi, 63, 64), __shfl(v.lo, 63, 64)};
        }
    }
    __syncthreads();
    // y-derivative at node i of the rows from q0: as ddy
    const double inv2 = 0.5 / D.dy;
    auto dydiff = [&](int q0, int i) {
        const double a = val[q0 * N + i], b = val[(q0 + 1) * N + i], c = val[(q0 + 2) * N + i];
        if (l > 0 && l < M - 1) return (c - a) * inv2;
        if (l == M - 1) return (3.0 * c - 4.0 * b + a) * inv2;
        return D.half ? 0.0 : (-3.0 * a + 4.0 * b - c) * inv2;
    };
    const double *zeta = val + here * N, *phi = val + (3 + here) * N, *psi = val + 6 * N;
    const double *zx = D.u + (size_t)l * (N + 1) + 1;
    const size_t nl = (size_t)l * N;
    const double *beta = D.beta + nl, *beta_x = D.beta_x + nl, *beta_y = D.beta_y + nl;
    const bool linear = D.linear;  // the planes z = 0 and z = -1; the layer densities are unchanged
    for (int i = threadIdx.x; i < N; i += 256) {
        const double zy = dydiff(0, i);
        D.ydiv[nl + i] = zy;
        D.ydiv[(size_t)N * M + nl + i] = dydiff(3, i);
        const double x = D.x1 + i * dx;
        const double w = dx * D.dy * ((i == 0 || i == N - 1) ? 0.5 : 1.0) * ((l == 0 || l == M - 1) ? 0.5 : 1.0);
        ((SrcRec<double> *)D.srcS)[nl + i] = {x,  linear ? 0.0 : zeta[i], linear ? 0.0 : zx[i], linear ? 0.0 : zy,
                                              w * (phi[i] - x), w * zx[i], w, 0.0};
        // bottom: outward normal points down, so both layers enter with -w
        ((SrcRec<double> *)D.srcB)[nl + i] = {x,  linear ? -1.0 : beta[i], linear ? 0.0 : beta_x[i],
                                              linear ? 0.0 : beta_y[i], -w * (psi[i] - x), -w * beta_x[i], -w, 0.0};
    }
    const size_t ntg = (size_t)(N - 1) * M, T2 = 2 * ntg;
    const double ys = D.y1 + l * D.dy;
    for (int e = threadIdx.x; e < 2 * (N - 1); e += 256) {
        const int st = e >= N - 1, k = e - st * (N - 1);
        const size_t t = st * ntg + (size_t)l * (N - 1) + k;
        const double xs = D.x1 + (k + 0.5) * dx;
        double d, Dst, ax, ay, sig;
        if (st == 0) {
            d = 0.5 * (zeta[k] + zeta[k + 1]);
            Dst = 0.5 * (phi[k] + phi[k + 1]) - xs;
            ax = 0.5 * (zx[k] + zx[k + 1]);
            ay = 0.5 * (dydiff(0, k) + dydiff(0, k + 1));
            sig = ax;
        } else {
            d = 0.5 * (beta[k] + beta[k + 1]);
            Dst = 0.5 * (psi[k] + psi[k + 1]) - xs;
            ax = 0.5 * (beta_x[k] + beta_x[k + 1]);
            ay = 0.5 * (beta_y[k] + beta_y[k + 1]);
            sig = -ax;
        }
        if (linear) {
            d = st ? -1.0 : 0.0;
            ax = ay = 0.0;
        }
        const double v[8] = {xs, ys, d, Dst, 1.0 + ax * ax, 2.0 * ax * ay, 1.0 + ay * ay, sig};
        for (int q = 0; q < 8; ++q) D.tg64[q * T2 + t] = v[q];
    }
}
constexpr size_t kPrepareLds = 64 << 10;  // rows of up to 1170 nodes; longer ones take the two launches

// ------------------------------------------------------------------ A2: all-pairs sums (hot loop)
// The sums read through address-space qualified pointers.  Per-lane arrays are
// global memory.  Node records are read-only for a whole launch; the batched
// kernel, whose pointers come from a descriptor in memory and so carry no
// address space (flat loads, which count on the same counter as the scalar
// loads and break the record prefetch), reads them through the constant
// address space, where a wave-uniform address gives a scalar load.  The
// single-problem kernel keeps the kernel-argument pointers: the compiler infers
// them as global and keeps several FP64 record loads in flight, which it does
// not do for constant-space loads (measured: 3% on the FP64 sums).
template <typename T>
using ConstPtr = const __attribute__((address_space(4))) T *;
template <typename T>
using GlobalPtr = __attribute__((address_space(1))) T *;

// One source record as a single 8-wide vector load (one scalar load per node).
template <typename T>
struct RecVec;
template <>
struct RecVec<float> {
    typedef float type __attribute__((ext_vector_type(8)));
};
template <>
struct RecVec<double> {
    typedef double type __attribute__((ext_vector_type(8)));
};
template <typename T, bool CREC>
struct RecPtrs {  // generic pointers
    typedef const SrcRec<T> *rec;
    typedef const typename RecVec<T>::type *vec;
};
template <typename T>
struct RecPtrs<T, true> {  // constant address space
    typedef ConstPtr<SrcRec<T>> rec;
    typedef ConstPtr<typename RecVec<T>::type> vec;
};
template <typename T, bool CREC>
using RecPtr = typename RecPtrs<T, CREC>::rec;

template <typename T, bool CREC>
__device__ __forceinline__ SrcRec<T> load_rec(RecPtr<T, CREC> p) {
    const typename RecVec<T>::type v = *reinterpret_cast<typename RecPtrs<T, CREC>::vec>(p);
    SrcRec<T> r;
    r.x = v[0];
    r.z = v[1];
    r.zx = v[2];
    r.zy = v[3];
    r.wD = v[4];
    r.ws = v[5];
    r.w = v[6];
    r.pad = v[7];
    return r;
}

// Walk the N source records of one row in groups of UNROLL with the next
// group's scalar loads in flight while the current group is computed.  Scalar
// loads may return out of order, so a wait covers every load issued before
// it: the next group is loaded into separate registers and handed over only
// after the current group's arithmetic, which is where the single wait falls.
// The prefetch reads up to UNROLL records past the end of a row; the record
// arrays carry kRecPad spare records so that this stays inside them (the
// values read there are never used).
// FP64 records (two scalar loads of 16 dwords per pair of records) gain
// nothing from it (measured), so they keep the plain loop.
// body(p, slot) does the first part of record p's work (distances and every
// reciprocal square root) and returns the rest (the accumulations) as a
// closure; a group runs every record's first part before any second part, so
// the independent rsq of the group are issued ahead of their uses (second
// parts in reverse record order).  slot (a compile-time constant: the record's
// position in the group, mod 2) picks one of two FP32 running sums, so that
// each sums half of the row's terms.
// The FP32 walk is one loop: any fold of the running sums inside a row piece
// (a branch per segment, or a loop nest per segment) measured 6 - 12% slower.
template <int U, int K = 0, typename Body, typename Rec>
__device__ __forceinline__ void run_group(Body &body, const Rec *cur) {
    if constexpr (K < U) {
        auto rest = body(cur[K], std::integral_constant<int, K % 2>{});
        run_group<U, K + 1>(body, cur);
        rest();
    }
}
template <typename T, int UNROLL, bool CREC, typename Body>
__device__ __forceinline__ void walk_row(RecPtr<T, CREC> src, int N, Body &&body) {
    static_assert(UNROLL <= kRecPad, "prefetch beyond the record padding");
    if constexpr (sizeof(T) == 8) {
#pragma unroll UNROLL
        for (int i = 0; i < N; ++i) body(load_rec<T, CREC>(src + i), std::integral_constant<int, 0>{})();
        return;
    }
    const int full = N - N % UNROLL;
    SrcRec<T> cur[UNROLL];
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) cur[u] = load_rec<T, CREC>(src + u);
    for (int i0 = 0; i0 < full; i0 += UNROLL) {
        SrcRec<T> nxt[UNROLL];
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) nxt[u] = load_rec<T, CREC>(src + i0 + UNROLL + u);
        __builtin_amdgcn_sched_barrier(0);  // keep the loads ahead of the arithmetic
        run_group<UNROLL>(body, cur);
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) cur[u] = nxt[u];
    }
    // the tail indexes cur[] with constants only (a runtime index would put the
    // array in private memory)
#pragma unroll
    for (int u = 0; u < UNROLL - 1; ++u)
        if (u < N - full) body(cur[u], std::integral_constant<int, 0>{})();
}

// One wave = 64 collocation points of one boundary: consecutive entries of
// the list of (row group, x*_k) points of that boundary, where a row group is
// TPL mesh rows handled by the same lane (so rows need not fill whole waves).
// The wave walks a chunk of source rows (boundary, y-row) and, for each, all N
// nodes of that row.  Source records are read with wave-uniform addresses
// (scalar loads) and shared by the TPL targets of a lane; every y-dependent
// term is hoisted per source row.  On a half domain each record serves both
// images (x, y_j) and (x, -y_j), which share s, dz, s^2 + dz^2 and the
// x-part of the double-layer numerator.
// Per pair:
//   own boundary:   w (D - D*) K1 + w sigma K2  and  w S2   (two rsqrt)
//   other boundary: w D K1 + w sigma K2                      (one rsqrt)
// written as  ri (coef num ri^2 + w sigma)  with ri = 1/R.
// FP32C: two FP32 running sums per row piece (alternate nodes), combined across
// pieces with Neumaier's compensated summation; the chunk result is written in
// FP64.
template <typename T, int NI>
struct TargetState {
    double ys;                                   // y* (FP64, physical units)
    T d, Dst, A, B, C;                           // collocation data
    T t[NI], ti[NI], t2[NI], Bt[NI], Ct2[NI];    // per source row and image
    T acc[2], acc2[2];                           // per source row piece (two running sums each)
    T sum, comp, s2sum, s2comp;                  // across rows
};

// Folds the running sums of a row piece into the across-row sums (Neumaier's
// compensated summation in FP32C).  S2: the piece also carries the S2 sum (only
// rows of the target's own boundary).
template <typename T>
__device__ __forceinline__ void neumaier_add(T &sum, T &comp, T x) {
    const T t = sum + x;
    comp += (fabs(sum) >= fabs(x)) ? ((sum - t) + x) : ((x - t) + sum);
    sum = t;
}
template <typename T, bool COMP, int NI, bool S2 = true>
__device__ __forceinline__ void row_end(TargetState<T, NI> &g) {
    if (COMP) {
        neumaier_add(g.sum, g.comp, g.acc[0]);
        neumaier_add(g.sum, g.comp, g.acc[1]);
        if (S2) {
            neumaier_add(g.s2sum, g.s2comp, g.acc2[0]);
            neumaier_add(g.s2sum, g.s2comp, g.acc2[1]);
        }
    } else {  // FP64: one running sum (slot 0)
        g.sum += g.acc[0];
        if (S2) g.s2sum += g.acc2[0];
    }
}

// NI = 2: half domain (both images per source row); NI = 1: full domain.
// FP32 (grid units): t = (y_j - y*) / dx is formed in FP64 for every source row
// and the S2 sum is multiplied by dx on output; FP64 works in physical units.
// LIN: the linearised residual (Section 4.2), whose boundaries are the planes
// z = 0 and z = -1 with zero slopes.  On a record of the target's own plane the
// double-layer numerator is exactly zero, so the general body adds exactly
// w sigma / R, and the S2 radicand is exactly s^2 + t^2; on the other plane the
// numerator is exactly the plane separation.  The LIN bodies drop those zero
// terms and give bit-identical sums.
// S2SUM: the item also forms the S2 sum (and writes both sums per target); without
// it, the single-problem FP64 sums, whose S2 sums s2_item forms.
template <typename T, bool COMP, int TPL, int UNROLL, int NI, bool CREC, bool LIN = false, bool S2SUM = true>
__device__ __forceinline__ void pair_item(const SrcRec<T> *__restrict__ srcS, const SrcRec<T> *__restrict__ srcB,
                                          const T *__restrict__ tg, const double *__restrict__ tg64, int N, int M,
                                          double y1, double dx, double dy, int tiles_per_bnd, int row_groups,
                                          int chunks, double *__restrict__ part, int tt, int c, int lane) {
    const RecPtr<T, CREC> recS = (RecPtr<T, CREC>)srcS, recB = (RecPtr<T, CREC>)srcB;
    const GlobalPtr<const T> gtg = (GlobalPtr<const T>)tg;
    const GlobalPtr<const double> gtg64 = (GlobalPtr<const double>)tg64;
    const double gi = (sizeof(T) == 4) ? 1.0 / dx : 1.0;
    const int ntg = (N - 1) * M;
    const size_t T2 = (size_t)2 * ntg;
    const int st = tt / tiles_per_bnd;
    const int npts = row_groups * (N - 1);
    const int idx = (tt - st * tiles_per_bnd) * 64 + lane;
    const bool valid = idx < npts;
    const int ic = valid ? idx : npts - 1;
    const int lg = ic / (N - 1);
    const int k = ic - lg * (N - 1);
    TargetState<T, NI> ts[TPL];
    T xs = 0;
#pragma unroll
    for (int q = 0; q < TPL; ++q) {
        const int l = min(lg * TPL + q, M - 1);
        const int tid = st * ntg + l * (N - 1) + k;
        xs = gtg[0 * T2 + tid];
        ts[q].ys = gtg64[1 * T2 + tid];
        ts[q].d = gtg[2 * T2 + tid];
        ts[q].Dst = gtg[3 * T2 + tid];
        ts[q].A = gtg[4 * T2 + tid];
        ts[q].B = gtg[5 * T2 + tid];
        ts[q].C = gtg[6 * T2 + tid];
        ts[q].sum = ts[q].comp = ts[q].s2sum = ts[q].s2comp = 0;
    }
    // chunk c: nodes [e0, e1) of the 2 M N source nodes in visit order (row r =
    // 2 j + boundary, so that every chunk mixes both boundaries); a chunk may
    // start and end inside a row.
    // (balanced split: the first nsrc % chunks chunks take one node more; 32-bit
    // arithmetic, as 2 M N is far below 2^31 for any mesh that fits the GPU)
    const int nsrc = 2 * M * N;
    const int q = nsrc / chunks, rem = nsrc - q * chunks;
    const int e0 = c * q + min(c, rem), e1 = e0 + q + (c < rem ? 1 : 0);
    for (int r = e0 / N; r * N < e1; ++r) {
        const int i0 = max(e0 - r * N, 0);
        const int i1 = min(e1 - r * N, N);
        const int ss = r & 1;
        const int j = r >> 1;
        const double yj = y1 + j * dy;
#pragma unroll
        for (int q = 0; q < TPL; ++q) {
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                // image i = 1 is (x, -y_j): a_y changes sign, which ti carries
                const T t = (T)((((i == 0) ? yj : -yj) - ts[q].ys) * gi);
                ts[q].t[i] = t;
                ts[q].ti[i] = (i == 0) ? t : -t;
                ts[q].t2[i] = t * t;
                ts[q].Bt[i] = ts[q].B * t;
                ts[q].Ct2[i] = ts[q].C * (t * t);
            }
            ts[q].acc[0] = ts[q].acc[1] = 0;
            ts[q].acc2[0] = ts[q].acc2[1] = 0;
        }
        const RecPtr<T, CREC> src = (ss ? recB : recS) + (size_t)j * N + i0;
        if (LIN && ss == st) {
            walk_row<T, UNROLL, CREC>(src, i1 - i0, [&](const SrcRec<T> &p, auto slot) {
                constexpr int a = decltype(slot)::value;
                const T s = p.x - xs;
                T ri[TPL][NI], rq[TPL][NI];
#pragma unroll
                for (int q = 0; q < TPL; ++q) {
                    const TargetState<T, NI> &e = ts[q];
                    const T dz = p.z - e.d;  // exactly zero: both points lie on one plane
                    const T base = (NI == 2) ? fma(s, s, dz * dz) : fma(s, s, e.t2[0]);
#pragma unroll
                    for (int i = 0; i < NI; ++i) {
                        ri[q][i] = rsq((NI == 2) ? base + e.t2[i] : fma(dz, dz, base));
                        // A = C = 1, B = 0: the S2 radicand is s^2 + t^2, in one rounding
                        rq[q][i] = (NI == 2) ? rsq(fma(s, s, e.t2[i])) : ri[q][i];
                    }
                }
                return [&, p, ri, rq]() {
#pragma unroll
                    for (int q = 0; q < TPL; ++q) {
                        TargetState<T, NI> &e = ts[q];
#pragma unroll
                        for (int i = 0; i < NI; ++i) {
                            e.acc[a] = fma(p.ws, ri[q][i], e.acc[a]);
                            e.acc2[a] = fma(p.w, rq[q][i], e.acc2[a]);
                        }
                    }
                };
            });
        } else if (ss == st) {
            walk_row<T, UNROLL, CREC>(src, i1 - i0, [&](const SrcRec<T> &p, auto slot) {
                constexpr int a = decltype(slot)::value;
                const T s = p.x - xs;
                T nb0[TPL], coef[TPL], ri[TPL][NI], rq[TPL][NI];
#pragma unroll
                for (int q = 0; q < TPL; ++q) {
                    const TargetState<T, NI> &e = ts[q];
                    const T dz = p.z - e.d;
                    const T base = (NI == 2) ? fma(s, s, dz * dz) : fma(s, s, e.t2[0]);
                    nb0[q] = fma(-s, p.zx, dz);
                    coef[q] = fma(-e.Dst, p.w, p.wD);
#pragma unroll
                    for (int i = 0; i < NI; ++i) {
                        ri[q][i] = rsq((NI == 2) ? base + e.t2[i] : fma(dz, dz, base));
                        if constexpr (S2SUM) rq[q][i] = rsq(fma(s, fma(e.A, s, e.Bt[i]), e.Ct2[i]));
                    }
                }
                return [&, p, nb0, coef, ri, rq]() {
#pragma unroll
                    for (int q = 0; q < TPL; ++q) {
                        TargetState<T, NI> &e = ts[q];
#pragma unroll
                        for (int i = 0; i < NI; ++i) {
                            const T num = fma(-e.ti[i], p.zy, nb0[q]);
                            const T bsum = fma(coef[q] * num, ri[q][i] * ri[q][i], p.ws);
                            e.acc[a] = fma(bsum, ri[q][i], e.acc[a]);
                            if constexpr (S2SUM) e.acc2[a] = fma(p.w, rq[q][i], e.acc2[a]);
                        }
                    }
                };
            });
        } else {
            walk_row<T, UNROLL, CREC>(src, i1 - i0, [&](const SrcRec<T> &p, auto slot) {
                constexpr int a = decltype(slot)::value;
                const T s = p.x - xs;
                T nb0[TPL], ri[TPL][NI];
#pragma unroll
                for (int q = 0; q < TPL; ++q) {
                    const TargetState<T, NI> &e = ts[q];
                    const T dz = p.z - e.d;
                    const T base = (NI == 2) ? fma(s, s, dz * dz) : fma(s, s, e.t2[0]);
                    nb0[q] = LIN ? dz : fma(-s, p.zx, dz);
#pragma unroll
                    for (int i = 0; i < NI; ++i) ri[q][i] = rsq((NI == 2) ? base + e.t2[i] : fma(dz, dz, base));
                }
                return [&, p, nb0, ri]() {
#pragma unroll
                    for (int q = 0; q < TPL; ++q) {
                        TargetState<T, NI> &e = ts[q];
#pragma unroll
                        for (int i = 0; i < NI; ++i) {
                            const T num = LIN ? nb0[q] : fma(-e.ti[i], p.zy, nb0[q]);
                            const T bsum = fma(p.wD * num, ri[q][i] * ri[q][i], p.ws);
                            e.acc[a] = fma(bsum, ri[q][i], e.acc[a]);
                        }
                    }
                };
            });
        }
#pragma unroll
        for (int q = 0; q < TPL; ++q) row_end<T, COMP, NI, S2SUM>(ts[q]);
    }
#pragma unroll
    for (int q = 0; q < TPL; ++q) {
        const int l = lg * TPL + q;
        if (valid && l < M) {
            const int tid = st * ntg + l * (N - 1) + k;
            if constexpr (!S2SUM) {
                ((GlobalPtr<double>)part)[(size_t)c * T2 + tid] = ts[q].sum;
                continue;
            }
            const GlobalPtr<double> o = (GlobalPtr<double>)part + ((size_t)c * T2 + tid) * 2;
            o[0] = (double)ts[q].sum + (double)ts[q].comp;
            o[1] = ((double)ts[q].s2sum + (double)ts[q].s2comp) * ((sizeof(T) == 4) ? dx : 1.0);
        }
    }
}

template <typename T, bool COMP, int TPL, int UNROLL, bool CREC, bool LIN = false>
__device__ __forceinline__ void pair_item_any(const SrcRec<T> *__restrict__ srcS, const SrcRec<T> *__restrict__ srcB,
                                              const T *__restrict__ tg, const double *__restrict__ tg64, int N,
                                              int M, int nimg, double y1, double dx, double dy, int tiles_per_bnd,
                                              int row_groups, int chunks, double *__restrict__ part, int tt,
                                              int c, int lane) {
    if (nimg == 2)
        pair_item<T, COMP, TPL, UNROLL, 2, CREC, LIN>(srcS, srcB, tg, tg64, N, M, y1, dx, dy, tiles_per_bnd,
                                                      row_groups, chunks, part, tt, c, lane);
    else
        pair_item<T, COMP, TPL, UNROLL, 1, CREC, LIN>(srcS, srcB, tg, tg64, N, M, y1, dx, dy, tiles_per_bnd,
                                                      row_groups, chunks, part, tt, c, lane);
}

// Resident waves per SIMD asked of the compiler: 8 for the FP32 variants whose
// registers allow it (the scalar registers of the record prefetch otherwise
// push the count to 7; what the limit moves out of scalar registers is spilled
// to vector lanes outside the inner loops), none (1) for the others.  Not used
// for the batched kernel, whose descriptor values would then be spilled inside
// its inner loops.
template <typename T, int TPL, int UNROLL>
constexpr int kMinWaves = (sizeof(T) == 4 && TPL == 1 && UNROLL <= 4) ? 8 : 1;

// Single problem: one wave per (target tile, source chunk).  LIN: the
// linearised residual (one launch shape per precision).
template <typename T, bool COMP, int TPL, int UNROLL, bool LIN = false>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(kMinWaves<T, TPL, UNROLL>))) void k_allpairs(
    const SrcRec<T> *__restrict__ srcS, const SrcRec<T> *__restrict__ srcB, const T *__restrict__ tg,
    const double *__restrict__ tg64, int N, int M, int nimg, double y1, double dx, double dy, int tiles_per_bnd,
    int row_groups, int target_tiles, int chunks, double *__restrict__ part) {
    const int lane = threadIdx.x & 63;
    // the wave index is uniform: keep it (and everything derived) in scalar registers
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = blockIdx.x * 4 + wave;
    const int tt = g % target_tiles, c = g / target_tiles;
    if (c >= chunks) return;
    pair_item_any<T, COMP, TPL, UNROLL, false, LIN>(srcS, srcB, tg, tg64, N, M, nimg, y1, dx, dy, tiles_per_bnd,
                                                    row_groups, chunks, part, tt, c, lane);
}

// ------------------------------------------------------------------ S2 sums in FP64
// The trapezoidal sum of w S2 over every node and image, S2 = (A s^2 + B s t + C
// t^2)^(-1/2), depends on a target's (A, B, C) and its mesh indices only, and away
// from the target a row of it is its integral plus Euler-Maclaurin corrections at
// the ends:
//   sum' f(s_i) dx = int f ds + sum_m B_2m / (2m)! dx^2m [f^(2m-1)]
// up to e^(-2 pi eta / dx), eta the distance of f's branch points s_c +- i eta from
// the real axis (s_c = -B t / 2A, eta = |t| sqrt(4AC - B^2) / 2A), and the
// derivatives of Q^(-1/2) are Legendre polynomials:
//   f^(n) = n! P_n(c) (A/Q)^(n/2) Q^(-1/2),  c = -(2As + Bt) / (2 sqrt(A Q)).
// In units of dx, a row with eta >= 8 takes its two ends, any other row also the
// nodes within sqrt(8^2 - eta^2) of s_c one by one (about 200 of them in all rows),
// with a segment of the corrected integral on each side: every end then lies 8 or
// more from the branch points (or the sum runs to the mesh edge node by node), where
// six corrections leave 1e-13 of one end's term and 1.5e-15 of the sum, and three
// suffice from 32 on.  The segments' integrals are (1/sqrt A) ln of a ratio; a
// wave multiplies the ratios of 16 rows before it takes a logarithm.
// A target costs about 16 thousand FP64 instructions (29 thousand in all) instead of the 220
// thousand of its 22082 pairs at 181 x 61 (launches of the sums by HIP events 613 -> 495 us;
// full 151 x 151 1570 -> 1142).
constexpr double kS2Reach = 8.0;   // node-by-node distance, in dx
constexpr int kS2Flush = 16;       // rows per logarithm, fewer where their product passes kS2Wide
// Range of the products: numerators and denominators of a row are 1 or more and the
// numerator is the larger one.  With A, C <= kS2Steep (slopes up to 10^6) and dy <= kS2Aspect
// dx it is below (4 kS2Steep (N + 2 M kS2Aspect))^2 < 10^50 (N M <= 2^26), so that no product
// passes 10^150; steeper targets, and meshes of larger dy, are summed node by node.  (16 rows
// without the check pass 10^308 from slopes of about 2800 on, half domain, 281 x 141.)
constexpr double kS2Wide = 1e100, kS2Steep = 1e12, kS2Aspect = 1e3;
constexpr int kS2Chunks = 16;      // most row chunks per tile of targets (rows c, c + chunks, ..)

// Closed form of the integral of (A s^2 + B s t + C t^2)^(-1/2) over a rectangle
// from the antiderivative of Section 3.1; a term with a zero prefactor is its
// limit, zero.
__device__ double s2_antideriv(double A, double B, double C, double s, double t) {
    const double Q = A * s * s + B * s * t + C * t * t;
    double g = 0.0;
    if (t != 0.0) g += t / sqrt(A) * log(2.0 * A * s + B * t + 2.0 * sqrt(A * Q));
    if (s != 0.0) g += s / sqrt(C) * log(2.0 * C * t + B * s + 2.0 * sqrt(C * Q));
    return g;
}

// The same without the cancellation in the logarithm: with p = 2 A s + B t and
// q = 2 sqrt(A Q), q^2 - p^2 = (4 A C - B^2) t^2, so p + q = (q^2 - p^2) / (q - p) where
// p < 0 (3 x 900: the row's error 5e-12 -> 1e-15 of its terms).
__device__ double s2_antideriv_stable(double A, double B, double C, double s, double t) {
    const double Q = A * s * s + B * s * t + C * t * t, det = 4.0 * A * C - B * B;
    const double p = 2.0 * A * s + B * t, q = 2.0 * sqrt(A * Q);
    const double p2 = 2.0 * C * t + B * s, q2 = 2.0 * sqrt(C * Q);
    double g = 0.0;
    if (t != 0.0) g += t / sqrt(A) * log(p < 0.0 ? det * t * t / (q - p) : p + q);
    if (s != 0.0) g += s / sqrt(C) * log(p2 < 0.0 ? det * s * s / (q2 - p2) : p2 + q2);
    return g;
}

// The part of the closed-form integral that row chunk c of `chunks` subtracts from
// its sum: corners c, c + chunks, .. of the rectangle [x_1, x_N] x [y_lo, y_M] relative
// to point (k, l), from mesh indices: the offset to an edge through the target is
// exactly zero (y_lo = -y_M on a half domain, where y_1 = 0; y_1 on a full one).
__device__ __forceinline__ double s2_corners(double A, double B, double C, int N, int M, int nimg, double dx, double dy,
                                             int k, int l, int c, int chunks) {
    double g = 0.0;
    for (int w = c; w < 4; w += chunks) {
        const double sc = (w & 1) ? -(k + 0.5) * dx : (N - 1.5 - k) * dx;
        const double tc = (w & 2) ? (nimg == 2 ? -(double)(M - 1 + l) * dy : -(double)l * dy) : (double)(M - 1 - l) * dy;
        const double v = s2_antideriv_stable(A, B, C, sc, tc);
        g += (w == 0 || w == 3) ? v : -v;
    }
    return g;
}

// 1/sqrt(x) to rounding: the estimate refined twice
__device__ __forceinline__ double rsq_full(double x) {
    double y = (double)__builtin_amdgcn_rsqf((float)x);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const double e = fma(-x * y, y, 1.0);
        y = fma(0.5 * y, e, y);
    }
    return y;
}

// Coefficients of one target's form (in units of dx) at one row: B t and C t^2.
struct S2Row {
    double A, sqA, Bt, Ct2;  // sqA: sqrt(A)
};

// One end of a segment: g = |u| + 2 sqrt(A Q), u = 2 A s + B t, and the corrections
// of the first K orders as they enter at an upper end:
//   sum_m (B_2m / 2m) eps^(2m-1) P_2m-1(c) / sqrt(Q),  eps = sqrt(A / Q).
// With X = eps c = -u / 2Q and y = eps^2, eps^n P_n(c) is a polynomial in X and y;
// the sum is X times a polynomial of degree K - 1 in (X^2, y), by Horner in both.
template <int K>
__device__ __forceinline__ double s2_end(const S2Row &r, double s, double &g, double &u) {
    // row j: the coefficients of y^j, by powers of X^2
    constexpr double q[6][6] = {
        {1.0 / 12, -1.0 / 48, 1.0 / 32, -143.0 / 1280, 1105.0 / 1536, -223193.0 / 30720},
        {1.0 / 80, -5.0 / 144, 231.0 / 1280, -195.0 / 128, 2455123.0 / 129024},
        {5.0 / 672, -21.0 / 256, 273.0 / 256, -129217.0 / 7168},
        {7.0 / 768, -35.0 / 128, 7601.0 / 1024},
        {105.0 / 5632, -7601.0 / 6144},
        {7601.0 / 133120}};
    const double Q = fma(s, fma(r.A, s, r.Bt), r.Ct2), rq = rsq(Q), rq2 = rq * rq;
    u = fma(2.0 * r.A, s, r.Bt);
    g = fma(2.0 * r.sqA, Q * rq, fabs(u));
    const double X = -0.5 * u * rq2, y = r.A * rq2, z = X * X;
    double sum = 0.0;
#pragma unroll
    for (int j = K - 1; j >= 0; --j) {
        double h = q[j][K - 1 - j];
#pragma unroll
        for (int i = K - 2 - j; i >= 0; --i) h = fma(h, z, q[j][i]);
        sum = j == K - 1 ? h : fma(sum, y, h);
    }
    return sum * X * rq;
}

// Ratio num / den whose logarithm over sqrt(A) is the integral between two ends.
__device__ __forceinline__ void s2_ratio(double g1, double u1, double g2, double u2, double w2, double &num,
                                         double &den) {
    const bool cross = u1 < 0.0 && u2 >= 0.0;
    num = cross ? g1 * g2 : u1 >= 0.0 ? g2 : g1;
    den = cross ? w2 : u1 >= 0.0 ? g1 : g2;
}

// The S2 sums of 64 targets (tile tt of the flattened points of both boundaries)
// over the lattice rows c, c + chunks, ..: rows -(M-1) .. M-1 on a half domain (the
// images; the doubled row on the symmetry line counts once whole), less this
// chunk's part of the closed-form integral.  Node by node:
__device__ __forceinline__ void s2_nodes_item(const double *__restrict__ tg64, int N, int M, int nimg, double dx,
                                              double dy, int tiles_per_bnd, int tt, int c, int chunks,
                                              double *__restrict__ out, int lane) {
    const GlobalPtr<const double> tg = (GlobalPtr<const double>)tg64;
    const int ntg = (N - 1) * M;
    const size_t T2 = (size_t)2 * ntg;
    const int st = tt / tiles_per_bnd, idx = (tt - st * tiles_per_bnd) * 64 + lane;
    const int ic = min(idx, ntg - 1), l = ic / (N - 1), k = ic - l * (N - 1);
    const int tid = st * ntg + ic;
    const double A = tg[4 * T2 + tid], B = tg[5 * T2 + tid], C = tg[6 * T2 + tid];
    const int rows = nimg == 2 ? 2 * M - 1 : M, off = nimg == 2 ? M - 1 + l : l;
    const double ry = dy / dx, s0 = -(k + 0.5);
    double acc = 0.0;
    for (int jr = c; jr < rows; jr += chunks) {
        const double t = (jr - off) * ry, Bt = B * t, Ct2 = C * (t * t);
        const double wy = (jr == 0 || jr == rows - 1) ? 0.5 : 1.0;
        double row = 0.0;
#pragma unroll 4
        for (int i = 0; i < N; ++i) {
            const double sn = s0 + i, f = rsq(fma(sn, fma(A, sn, Bt), Ct2));
            row = fma((i == 0 || i == N - 1) ? 0.5 : 1.0, f, row);
        }
        acc = fma(wy, row, acc);
    }
    const double sum = dy * acc - s2_corners(A, B, C, N, M, nimg, dx, dy, k, l, c, chunks);
    if (idx < ntg) ((GlobalPtr<double>)out)[(size_t)c * T2 + tid] = sum;
}

// The same in segments, for dy <= kS2Aspect dx.
__device__ __forceinline__ void s2_item(const double *__restrict__ tg64, int N, int M, int nimg, double dx, double dy,
                                        int tiles_per_bnd, int tt, int c, int chunks, double *__restrict__ out,
                                        int lane) {
    const GlobalPtr<const double> tg = (GlobalPtr<const double>)tg64;
    const int ntg = (N - 1) * M;
    const size_t T2 = (size_t)2 * ntg;
    const int st = tt / tiles_per_bnd, idx = (tt - st * tiles_per_bnd) * 64 + lane;
    const int ic = min(idx, ntg - 1), l = ic / (N - 1), k = ic - l * (N - 1);
    const int tid = st * ntg + ic;
    const double B = tg[5 * T2 + tid], C = tg[6 * T2 + tid];
    S2Row r;
    r.A = tg[4 * T2 + tid];
    if (!__all(r.A <= kS2Steep && C <= kS2Steep)) {
        s2_nodes_item(tg64, N, M, nimg, dx, dy, tiles_per_bnd, tt, c, chunks, out, lane);
        return;
    }
    const double isqA = rsq_full(r.A);
    r.sqA = r.A * isqA;
    const double D4 = fma(4.0 * r.A, C, -B * B);
    const double cen = -0.5 * B / r.A, et2 = D4 / (4.0 * r.A * r.A);  // s_c / t, eta^2 / t^2
    const int rows = nimg == 2 ? 2 * M - 1 : M, off = nimg == 2 ? M - 1 + l : l;
    const double ry = dy / dx, s0 = -(k + 0.5), sN = N - 1.5 - k, last = N - 1;
    constexpr double H2 = kS2Reach * kS2Reach, far3 = 32.0 * 32.0;
    double acc = 0.0, logs = 0.0, num = 1.0, den = 1.0;
    int pending = 0;
    for (int jr = c; jr < rows; jr += chunks) {
        const double t = (jr - off) * ry, t2 = t * t;
        const bool edge = jr == 0 || jr == rows - 1;
        const double wy = edge ? 0.5 : 1.0;
        r.Bt = B * t;
        r.Ct2 = C * t2;
        const double eta2 = et2 * t2, w2 = D4 * t2;
        double rn = 1.0, rd = 1.0;  // the row's ratio
        if (__all(eta2 >= H2)) {
            // the whole row as one segment
            const double Q0 = fma(s0, fma(r.A, s0, r.Bt), r.Ct2), Q1 = fma(sN, fma(r.A, sN, r.Bt), r.Ct2);
            double g1, g2, u1, u2, e1, e2;
            if (__all(Q0 >= far3 * r.A && Q1 >= far3 * r.A)) {
                e1 = s2_end<3>(r, s0, g1, u1);
                e2 = s2_end<3>(r, sN, g2, u2);
            } else {
                e1 = s2_end<6>(r, s0, g1, u1);
                e2 = s2_end<6>(r, sN, g2, u2);
            }
            acc = fma(wy, e2 - e1, acc);
            s2_ratio(g1, u1, g2, u2, w2, rn, rd);
        } else {
            // nodes a .. b one by one (a trapezoid of its own), segments 0 .. a and b .. N-1
            const double W = sqrt(fmax(H2 - eta2, 0.0)), sc = cen * t - s0;
            const bool far = eta2 >= H2;
            double fa = floor(sc - W), fb = ceil(sc + W);
            fa = far ? last : fa < 1.0 ? 0.0 : fmin(fa, last);
            fb = far || fb > last - 1.0 ? last : fmax(fb, 0.0);
#pragma unroll 1
            for (int side = 0; side < 2; ++side) {
                const double e1 = side ? fb : 0.0, e2 = side ? last : fa;
                double g1, g2, u1, u2, n1, d1;
                const double c1 = s2_end<6>(r, s0 + e1, g1, u1), c2 = s2_end<6>(r, s0 + e2, g2, u2);
                s2_ratio(g1, u1, g2, u2, w2, n1, d1);
                const bool there = e2 > e1;
                rn *= there ? n1 : 1.0;
                rd *= there ? d1 : 1.0;
                acc = fma(there ? wy : 0.0, c2 - c1, acc);
            }
            const int cnt = (int)(fb - fa);
            double sa = s0 + fa;
            for (int j = 0; __any(j <= cnt && cnt > 0); ++j) {
                const double f = rsq(fma(sa, fma(r.A, sa, r.Bt), r.Ct2));
                const double wj = (j > cnt || cnt <= 0) ? 0.0 : (j == 0 || j == cnt) ? 0.5 * wy : wy;
                acc = fma(wj, f, acc);
                sa += j < cnt ? 1.0 : 0.0;
            }
        }
        if (edge) {  // half weight: half the logarithm
            rn = sqrt(rn);
            rd = sqrt(rd);
        }
        num *= rn;
        den *= rd;
        if (++pending == kS2Flush || __any(num > kS2Wide)) {
            logs += log(num / den);
            num = den = 1.0;
            pending = 0;
        }
    }
    if (pending) logs += log(num / den);
    const double sum = dy * fma(logs, isqA, acc) - s2_corners(r.A, B, C, N, M, nimg, dx, dy, k, l, c, chunks);
    if (idx < ntg) ((GlobalPtr<double>)out)[(size_t)c * T2 + tid] = sum;
}

__global__ __launch_bounds__(256) void k_s2_sums(const double *__restrict__ tg, int N, int M, int nimg, double dx,
                                                 double dy, int s2_chunks, double *__restrict__ out) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = blockIdx.x * 4 + wave, tpb = ((N - 1) * M + 63) / 64;
    const int tt = g / s2_chunks, c = g - tt * s2_chunks;
    if (tt >= 2 * tpb) return;
    s2_item(tg, N, M, nimg, dx, dy, tpb, tt, c, s2_chunks, out, lane);
}

// The single-problem FP64 pair sums, one wave per (target tile, source chunk);
// part: [chunks][targets].  NODES: the first s2_blocks workgroups form the S2 sums
// node by node, behind the pair sums; otherwise k_s2_sums does (whose segments need
// twice the registers of the pair sums: in one launch they cost these a third of
// their resident waves, 506 -> 552 us at 181 x 61).
template <int TPL, int UNROLL, bool NODES>
__global__ __launch_bounds__(256) void k_allpairs64(const SrcRec<double> *__restrict__ srcS,
                                                    const SrcRec<double> *__restrict__ srcB,
                                                    const double *__restrict__ tg, int N, int M, int nimg, double y1,
                                                    double dx, double dy, int tiles_per_bnd, int row_groups,
                                                    int target_tiles, int chunks, double *__restrict__ part,
                                                    int s2_blocks, int s2_chunks) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int g = blockIdx.x * 4 + wave;
    if constexpr (NODES) {
        if ((int)blockIdx.x < s2_blocks) {
            const int tpb = ((N - 1) * M + 63) / 64, t2 = g / s2_chunks;
            if (t2 < 2 * tpb)
                s2_nodes_item(tg, N, M, nimg, dx, dy, tpb, t2, g - t2 * s2_chunks, s2_chunks,
                              part + (size_t)chunks * 2 * (N - 1) * M, lane);
            return;
        }
        g -= 4 * s2_blocks;
    }
    const int tt = g % target_tiles, c = g / target_tiles;
    if (c >= chunks) return;
    if (nimg == 2)
        pair_item<double, false, TPL, UNROLL, 2, false, false, false>(srcS, srcB, tg, tg, N, M, y1, dx, dy, tiles_per_bnd,
                                                                      row_groups, chunks, part, tt, c, lane);
    else
        pair_item<double, false, TPL, UNROLL, 1, false, false, false>(srcS, srcB, tg, tg, N, M, y1, dx, dy, tiles_per_bnd,
                                                                      row_groups, chunks, part, tt, c, lane);
}

// Many problems in one persistent launch: the work items (target tile, source
// chunk) of all active problems form one list; every wave walks it with a fixed
// stride, so the schedule (and each problem's fixed-order reduction) is
// deterministic.  An inactive problem owns no items (its item0 equals the next
// problem's), so the walk never selects it.
template <typename T, bool COMP, int TPL, int UNROLL>
__global__ __launch_bounds__(256) void k_allpairs_batched(const PairDesc *__restrict__ descs, int count) {
    const long total_items = descs[0].batch_items;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const long nwaves = (long)gridDim.x * 4;
    int inst = 0;
    for (long item = (long)blockIdx.x * 4 + wave; item < total_items; item += nwaves) {
        while (inst + 1 < count && descs[inst + 1].item0 <= item) ++inst;  // items grow monotonically
        const PairDesc &D = descs[inst];
        const int local = (int)(item - D.item0);
        const int tt = local % D.target_tiles, c = local / D.target_tiles;
        pair_item_any<T, COMP, TPL, UNROLL, true>((const SrcRec<T> *)D.srcS, (const SrcRec<T> *)D.srcB,
                                            (const T *)D.tg, D.tg64, D.N, D.M, D.nimg, D.y1, D.dx, D.dy,
                                            D.tiles_per_bnd, D.row_groups, D.chunks, D.part, tt, c, lane);
    }
}

// ------------------------------------------------------------------ A3 + A4: finalize

// Workgroups [0, bie_blocks) hold 64 boundary-integral rows each (4 waves: wave
// w sums a quarter of the source chunks' partial sums and the w-th corner term
// of the closed-form S2 integral; wave 0 combines them in a fixed order), the
// rest one dynamic or radiation row per thread.
__host__ __device__ __forceinline__ int bie_blocks(int N, int M) { return (2 * (N - 1) * M + 63) / 64; }
__host__ __device__ __forceinline__ int finalize_blocks(int N, int M) {
    return bie_blocks(N, M) + ((N + 1) * M + 4 * M + 255) / 256;
}

__device__ __forceinline__ void finalize_bie(const PairDesc &D, int b, double (*red)[3][64]) {
    const int N = D.N, M = D.M;
    const int ntg = (N - 1) * M;
    const size_t T2 = (size_t)2 * ntg;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int tid = b * 64 + lane;
    const bool valid = tid < 2 * ntg;
    const int t = valid ? tid : 2 * ntg - 1;
    // partial sums of chunks [c0, c1), in chunk order, eight loads in flight
    const int chunks = D.chunks;
    const int c0 = (w * chunks) >> 2, c1 = ((w + 1) * chunks) >> 2;
    const double2 *pp = (const double2 *)D.part + t;
    double acc = 0.0, acc2 = 0.0;
    int c = c0;
    for (; c + 8 <= c1; c += 8) {
        double2 v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = pp[(size_t)(c + q) * T2];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            acc += v[q].x;
            acc2 += v[q].y;
        }
    }
    for (; c < c1; ++c) {
        const double2 v = pp[(size_t)c * T2];
        acc += v.x;
        acc2 += v.y;
    }
    // corner w of the rectangle [x_1, x_N] x [y_lo, y_M] relative to the target,
    // from mesh indices: the offset to an edge through the target is exactly zero
    // (y_lo = -y_M on a half domain, where y_1 = 0; y_1 on a full one)
    const double *tg = D.tg64;
    const double A = tg[4 * T2 + t], B = tg[5 * T2 + t], C = tg[6 * T2 + t];
    const int tl = (t % ntg) / (N - 1), tk = (t % ntg) - tl * (N - 1);
    const double sc = (w & 1) ? -(tk + 0.5) * D.dx : (N - 1.5 - tk) * D.dx;
    const double tc = (w & 2) ? (D.half ? -(double)(M - 1 + tl) * D.dy : -(double)tl * D.dy)
                              : (double)(M - 1 - tl) * D.dy;
    const double corner = s2_antideriv(A, B, C, sc, tc);
    if (w > 0) {
        red[w - 1][0][lane] = acc;
        red[w - 1][1][lane] = acc2;
        red[w - 1][2][lane] = corner;
    }
    __syncthreads();
    if (w > 0 || !valid) return;
    acc = ((acc + red[0][0][lane]) + red[1][0][lane]) + red[2][0][lane];
    acc2 = ((acc2 + red[0][1][lane]) + red[1][1][lane]) + red[2][1][lane];
    // corners in the order (xhi, yhi) - (xlo, yhi) - (xhi, ylo) + (xlo, ylo)
    const double I2 = ((corner - red[0][2][lane]) - red[1][2][lane]) + red[2][2][lane];
    const int st = t / ntg, r = t - st * ntg;
    const int l = r / (N - 1), k = r - l * (N - 1);
    const int row = (st + 1) * (N + 1) * M + l * (N + 1) + k + 2;
    const double s2 = st ? -acc2 : acc2;  // bottom records carry -w
    const double Dst = tg[3 * T2 + t], sig = tg[7 * T2 + t];
    D.F[row] = acc - sig * s2 + sig * I2 - kTwoPi * Dst;
}

// Dynamic rows (block 0, columns >= 2) and radiation rows (columns 0, 1 of the
// three blocks); r enumerates block 0 and then the radiation pairs of blocks 1, 2.
// Second y-difference of the node field g (zeta: block 0 of the node array) at
// (l, i): central inside; on the symmetry line of a half domain the mirror node
// stands for row -1; one-sided four-point stencils on an outer edge (M >= 4).
__device__ __forceinline__ double y_second_diff(const double *g, int l, int i, int N, int M, double dy, int half) {
    const double c = 1.0 / (dy * dy);
    auto at = [&](int j) { return g[(size_t)j * N + i]; };
    if (l > 0 && l < M - 1) return c * (at(l + 1) - 2.0 * at(l) + at(l - 1));
    if (l == M - 1) return c * (2.0 * at(M - 1) - 5.0 * at(M - 2) + 4.0 * at(M - 3) - at(M - 4));
    return half ? c * 2.0 * (at(1) - at(0)) : c * (2.0 * at(0) - 5.0 * at(1) + 4.0 * at(2) - at(3));
}

__device__ __forceinline__ void finalize_rows(const PairDesc &D, int r) {
    const int N = D.N, M = D.M;
    const int nblk = (N + 1) * M;
    if (r >= nblk + 4 * M) return;
    int blk, l, col;
    if (r < nblk) {
        blk = 0;
        l = r / (N + 1);
        col = r - l * (N + 1);
    } else {
        const int q = r - nblk;
        blk = 1 + q / (2 * M);
        const int e = q - (blk - 1) * 2 * M;
        l = e >> 1;
        col = e & 1;
    }
    const int row = blk * nblk + l * (N + 1) + col;
    const double dx = D.dx, x1 = D.x1;
    const double *u = D.u, *nodes = D.nodes, *ydiv = D.ydiv;
    const double *fx = u + (size_t)blk * nblk + (size_t)l * (N + 1) + 1;  // (f_x)_{., l}
    const double *fv = nodes + ((size_t)blk * M + l) * N;                  // f_{., l}
    if (col < 2) {
        // radiation rows (eqs. scullen1-6 as discretised in Appendix B)
        const double fxx = (fx[1] - fx[0]) / dx;
        const double n_decay = D.n_decay;
        double v;
        if (blk == 0) {
            v = (col == 0) ? x1 * fx[0] + n_decay * fv[0] : x1 * fxx + n_decay * fx[0];
        } else {
            v = (col == 0) ? x1 * (fx[0] - 1.0) + n_decay * (fv[0] - x1) : x1 * fxx + n_decay * (fx[0] - 1.0);
        }
        D.F[row] = v;
        return;
    }
    // dynamic condition, eq. (new_finite_dynamic), at (x_{k+1/2}, y_l)
    const int k = col - 2;
    const size_t n0 = (size_t)l * N + k, n1 = n0 + 1;
    const double *zx = u + (size_t)l * (N + 1) + 1;
    const double *px = u + (size_t)nblk + (size_t)l * (N + 1) + 1;
    const double z = 0.5 * (nodes[n0] + nodes[n1]);
    const double a = 0.5 * (zx[k] + zx[k + 1]);
    const double b = 0.5 * (ydiv[n0] + ydiv[n1]);
    const double p = 0.5 * (px[k] + px[k + 1]);
    const double q = 0.5 * (ydiv[(size_t)N * M + n0] + ydiv[(size_t)N * M + n1]);
    const double kin = 0.5 * ((1.0 + a * a) * q * q + (1.0 + b * b) * p * p - 2.0 * a * b * p * q) /
                       (1.0 + a * a + b * b);
    const double fr2 = D.froude * D.froude;
    // linear mode: eq. (linear_dynamic2), phi*_x + zeta*/F^2 - 1
    double f1 = D.linear ? p + z / fr2 - 1.0 : kin + z / fr2 - 0.5;
    if (D.tau != 0.0) {
        // surface tension (Section 6): -tau K, K = div(grad zeta / |(1, grad zeta)|) from the
        // half-mesh slopes, the cell differences of zeta_x and zeta_y and the mean of the
        // node second y-differences; linear mode: -tau (zeta_xx + zeta_yy)
        const double zxx = (zx[k + 1] - zx[k]) / dx;
        const double zyy = 0.5 * (y_second_diff(nodes, l, k, N, M, D.dy, D.half) +
                                  y_second_diff(nodes, l, k + 1, N, M, D.dy, D.half));
        if (D.linear) {
            f1 -= D.tau * (zxx + zyy);
        } else {
            const double zxy = (ydiv[n1] - ydiv[n0]) / dx;
            const double qq = 1.0 + a * a + b * b;
            f1 -= D.tau * ((1.0 + b * b) * zxx - 2.0 * a * b * zxy + (1.0 + a * a) * zyy) / (qq * sqrt(qq));
        }
    }
    D.F[row] = f1;
}

// The boundary-integral rows from the single-problem FP64 sums: pair sums [chunks]
// [targets] and, behind them, [s2_chunks][targets] (at most 16) S2 sums less the
// closed-form integral.  64 rows per workgroup, a quarter of the chunks per wave; the
// logarithms of the closed form are taken in the S2 sums, where other waves hide
// them (12.2 -> 4.8 us at 31 x 11, 8.0 -> 5.3 at 181 x 61).
__device__ __forceinline__ void finalize_bie64(const PairDesc &D, int b, int s2_chunks, double (*red)[2][64]) {
    const int N = D.N, M = D.M;
    const int ntg = (N - 1) * M;
    const size_t T2 = (size_t)2 * ntg;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int tid = b * 64 + lane;
    const bool valid = tid < 2 * ntg;
    const int t = valid ? tid : 2 * ntg - 1;
    const int chunks = D.chunks;
    const int c0 = (w * chunks) >> 2, c1 = ((w + 1) * chunks) >> 2;
    const double *pp = D.part + t, *p2 = D.part + (size_t)chunks * T2 + t;
    const double Dst = D.tg64[3 * T2 + t], sig = D.tg64[7 * T2 + t];
    // this wave's four S2 chunks, then its quarter of the pair sums, eight loads in flight
    double q2[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) q2[q] = 4 * w + q < s2_chunks ? p2[(size_t)(4 * w + q) * T2] : 0.0;
    double acc = 0.0;
    int c = c0;
    for (; c + 8 <= c1; c += 8) {
        double v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = pp[(size_t)(c + q) * T2];
#pragma unroll
        for (int q = 0; q < 8; ++q) acc += v[q];
    }
    for (; c < c1; ++c) acc += pp[(size_t)c * T2];
    double acc2 = (q2[0] + q2[1]) + (q2[2] + q2[3]);
    if (w > 0) {
        red[w - 1][0][lane] = acc;
        red[w - 1][1][lane] = acc2;
    }
    __syncthreads();
    if (w > 0 || !valid) return;
    acc = ((acc + red[0][0][lane]) + red[1][0][lane]) + red[2][0][lane];
    acc2 = ((acc2 + red[0][1][lane]) + red[1][1][lane]) + red[2][1][lane];
    const int st = t / ntg, r = t - st * ntg;
    const int l = r / (N - 1), k = r - l * (N - 1);
    const int row = (st + 1) * (N + 1) * M + l * (N + 1) + k + 2;
    D.F[row] = acc - sig * acc2 - kTwoPi * Dst;
}
__global__ __launch_bounds__(256) void k_finalize64(PairDesc D, int s2_chunks) {
    __shared__ double red[3][2][64];
    const int nb = bie_blocks(D.N, D.M), b = blockIdx.x;
    if (b < nb) finalize_bie64(D, b, s2_chunks, red);
    else finalize_rows(D, (b - nb) * 256 + threadIdx.x);
}

__device__ __forceinline__ void finalize_body(const PairDesc &D, int b) {
    __shared__ double red[3][3][64];
    const int nb = bie_blocks(D.N, D.M);
    if (b < nb) finalize_bie(D, b, red);
    else finalize_rows(D, (b - nb) * 256 + threadIdx.x);
}
__global__ __launch_bounds__(256) void k_finalize(PairDesc D) { finalize_body(D, blockIdx.x); }
__global__ __launch_bounds__(256) void k_finalize_batched(const PairDesc *__restrict__ descs, int count) {
    const PairDesc &D = descs[find_problem<2>(descs, count, blockIdx.x)];
    if (!D.active) return;  // uniform over the workgroup
    finalize_body(D, blockIdx.x - D.blk_fin);
}

}  // namespace


size_t residual_work_bytes(const Dims &d, const PairLaunch &pl) {
    auto al = [](size_t b) { return (b + 255) & ~(size_t)255; };
    size_t b = 0;
    b += al(sizeof(double) * 3 * d.nnode);
    b += al(sizeof(double) * 2 * d.nnode);
    b += al(sizeof(double) * 8 * 2 * d.ntg);
    b += al(sizeof(float) * 7 * 2 * d.ntg);
    b += 2 * al(sizeof(SrcRec<double>) * (d.nnode + kRecPad));
    b += al(sizeof(double) * 2 * 2 * (size_t)d.ntg * pl.chunks);
    b += al(sizeof(double) * 4);
    return b;
}

void residual_work_carve(void *base, const Dims &d, const PairLaunch &pl, ResidualWork *w) {
    auto al = [](size_t b) { return (b + 255) & ~(size_t)255; };
    char *p = (char *)base;
    w->nodes = (double *)p; p += al(sizeof(double) * 3 * d.nnode);
    w->ydiv = (double *)p; p += al(sizeof(double) * 2 * d.nnode);
    w->tg = (double *)p; p += al(sizeof(double) * 8 * 2 * d.ntg);
    w->tg32 = (float *)p; p += al(sizeof(float) * 7 * 2 * d.ntg);
    w->srcS = p; p += al(sizeof(SrcRec<double>) * (d.nnode + kRecPad));
    w->srcB = p; p += al(sizeof(SrcRec<double>) * (d.nnode + kRecPad));
    w->part = (double *)p; p += al(sizeof(double) * 2 * 2 * (size_t)d.ntg * pl.chunks);
    w->scal = (double *)p; p += al(sizeof(double) * 4);
    w->bytes = (size_t)(p - (char *)base);
}

namespace {

PairDesc make_desc(const bim_problem *p, const Dims &d, const PairLaunch &pl, const ResidualWork &w,
                   const double *u, double *F, int prec, int linear) {
    PairDesc D{};
    D.srcS = w.srcS;
    D.srcB = w.srcB;
    D.tg = (prec == BIM_FP64) ? (const void *)w.tg : (const void *)w.tg32;
    D.tg64 = w.tg;
    D.part = w.part;
    D.N = d.N;
    D.M = d.M;
    D.nimg = d.nimg;
    D.y1 = p->y1;
    D.dx = p->dx;
    D.dy = p->dy;
    D.tiles_per_bnd = pl.tiles_per_bnd;
    D.row_groups = pl.row_groups;
    D.target_tiles = pl.target_tiles;
    D.chunks = pl.chunks;
    D.item0 = 0;
    D.batch_items = 0;
    D.active = 1;
    D.u = u;
    D.F = F;
    D.nodes = w.nodes;
    D.ydiv = w.ydiv;
    D.tg32 = w.tg32;
    D.beta = p->beta;
    D.beta_x = p->beta_x;
    D.beta_y = p->beta_y;
    D.x1 = p->x1;
    D.n_decay = p->n_decay;
    D.froude = p->froude;
    D.tau = p->tau;
    D.half = p->half_domain ? 1 : 0;
    D.linear = linear;
    return D;
}

}  // namespace

// Meshes whose S2 sums are formed node by node, in the pair sums' launch: up to about
// 10^7 targets times lattice nodes the segments' own launch and latency cost more
// (whole evaluation, nodes / segments in us: 31 x 11 22 / 28, 61 x 21 34 / 36, 76 x 26 45 /
// 48, 91 x 31 70 / 68, 121 x 41 156 / 137, 181 x 61 660 / 511; full 51 x 51 51 / 55,
// 61 x 61 74.5 / 72.5, 101 x 101 358 / 302).  A row costs its N nodes one way and two ends
// and up to 17 nodes the other, so that the line rises as rows get shorter than about 45
// (3 x 900 58 / 101, 8 x 900 277 / 337, 12 x 900 599 / 599, 16 x 300 139 / 148, 16 x 900 1042 / 979,
// 24 x 121 63 / 68, 24 x 300 281 / 264, 31 x 121 93 / 90, 40 x 61 49 / 53, 50 x 61 67 / 66).
static bool s2_by_nodes(const Dims &d, const bim_problem *p) {
    const double row = std::max(1.0, 45.0 / d.N);
    return (double)d.nnode * d.nnode * d.nimg < 1.1e7 * row * row || p->dy > kS2Aspect * p->dx;
}

int residual_enqueue(const bim_problem *p, const double *u, double *F, int prec, const PairLaunch &pl,
                     const ResidualWork &w, hipStream_t s, hipEvent_t *ev_pair, int linear,
                     const double *lin_tables) {
    const Dims d(p);
    const int N = d.N, M = d.M;
    PairDesc D = make_desc(p, d, pl, w, u, F, prec, linear);
    if (lin_tables) D.chunks = lin_conv_chunks(d, pl.chunks);
    // FP64 with its own sums (not pair by pair with S2's)
    const bool pairs64 = prec == BIM_FP64 && !linear && !pl.s2_with_pairs;
    const bool own64 = pairs64 || lin_tables;
    const size_t prep_lds = sizeof(double) * 7 * (size_t)N;
    if (own64 && prep_lds <= kPrepareLds) {
        hipLaunchKernelGGL(k_prepare64, dim3(M), dim3(256), prep_lds, s, D);
    } else {
        hipLaunchKernelGGL(k_integrate, dim3(3 * M), dim3(64), 0, s, D);
        if (prec == BIM_FP64)
            hipLaunchKernelGGL(k_records<double>, dim3(record_blocks(N, M)), dim3(256), 0, s, D);
        else
            hipLaunchKernelGGL(k_records<float>, dim3(record_blocks(N, M)), dim3(256), 0, s, D);
    }
    if (ev_pair) BIM_HIP(hipEventRecord(ev_pair[0], s));
#define BIM_LAUNCH_PAIRS(T, COMP, TPL, UNR, TG)                                                         \
    hipLaunchKernelGGL((k_allpairs<T, COMP, TPL, UNR>), dim3(pl.blocks), dim3(256), 0, s,               \
                       (const SrcRec<T> *)w.srcS, (const SrcRec<T> *)w.srcB, TG, w.tg, N, M, d.nimg,    \
                       p->y1, p->dx, p->dy, pl.tiles_per_bnd, pl.row_groups, pl.target_tiles, pl.chunks, \
                       w.part)
    const int vsel = (pl.tpl == 2 ? 3 : 0) + (pl.unroll == 2 ? 0 : pl.unroll == 4 ? 1 : 2);
    // FP64: the S2 sums' row chunks share the partial-sum buffer (two values per chunk
    // and target) with the pair sums; on small meshes they are summed node by node in
    // the same launch (s2_by_nodes)
    const bool by_nodes = s2_by_nodes(d, p);
    const int s2_chunks = std::min(kS2Chunks, pl.chunks);
    const int s2_blocks = cdiv((long)2 * cdiv((long)(N - 1) * M, 64) * s2_chunks, 4);
    if (lin_tables) {
        if (int rc = lin_conv_enqueue(D, lin_tables, s)) return rc;
    } else if (linear) {
        // the same source chunks (the partial-sum buffer and the finalize use
        // pl.chunks), one target row per lane and the default unroll
        const PairLaunch ll = pair_launch(d, 1, prec == BIM_FP64 ? 4 : 2, pl.chunks);
        if (prec == BIM_FP64)
            hipLaunchKernelGGL((k_allpairs<double, false, 1, 4, true>), dim3(ll.blocks), dim3(256), 0, s,
                               (const SrcRec<double> *)w.srcS, (const SrcRec<double> *)w.srcB, w.tg, w.tg, N, M,
                               d.nimg, p->y1, p->dx, p->dy, ll.tiles_per_bnd, ll.row_groups, ll.target_tiles,
                               ll.chunks, w.part);
        else
            hipLaunchKernelGGL((k_allpairs<float, true, 1, 2, true>), dim3(ll.blocks), dim3(256), 0, s,
                               (const SrcRec<float> *)w.srcS, (const SrcRec<float> *)w.srcB, w.tg32, w.tg, N, M,
                               d.nimg, p->y1, p->dx, p->dy, ll.tiles_per_bnd, ll.row_groups, ll.target_tiles,
                               ll.chunks, w.part);
    } else if (pairs64) {
#define BIM_LAUNCH_PAIRS64(TPL, UNR, NODES)                                                                       \
    hipLaunchKernelGGL((k_allpairs64<TPL, UNR, NODES>), dim3(pl.blocks + (NODES ? s2_blocks : 0)), dim3(256), 0, s,    \
                       (const SrcRec<double> *)w.srcS, (const SrcRec<double> *)w.srcB, w.tg, N, M, d.nimg, p->y1, p->dx, \
                       p->dy, pl.tiles_per_bnd, pl.row_groups, pl.target_tiles, pl.chunks, w.part, s2_blocks, s2_chunks)
        if (by_nodes) {
            switch (vsel) {
                case 0: BIM_LAUNCH_PAIRS64(1, 2, true); break;
                case 1: BIM_LAUNCH_PAIRS64(1, 4, true); break;
                case 2: BIM_LAUNCH_PAIRS64(1, 8, true); break;
                case 3: BIM_LAUNCH_PAIRS64(2, 2, true); break;
                case 4: BIM_LAUNCH_PAIRS64(2, 4, true); break;
                default: BIM_LAUNCH_PAIRS64(2, 8, true); break;
            }
        } else {
            hipLaunchKernelGGL(k_s2_sums, dim3(s2_blocks), dim3(256), 0, s, w.tg, N, M, d.nimg, p->dx, p->dy, s2_chunks,
                               w.part + (size_t)pl.chunks * 2 * d.ntg);
            switch (vsel) {
                case 0: BIM_LAUNCH_PAIRS64(1, 2, false); break;
                case 1: BIM_LAUNCH_PAIRS64(1, 4, false); break;
                case 2: BIM_LAUNCH_PAIRS64(1, 8, false); break;
                case 3: BIM_LAUNCH_PAIRS64(2, 2, false); break;
                case 4: BIM_LAUNCH_PAIRS64(2, 4, false); break;
                default: BIM_LAUNCH_PAIRS64(2, 8, false); break;
            }
        }
#undef BIM_LAUNCH_PAIRS64
    } else if (prec == BIM_FP64) {
        switch (vsel) {
            case 0: BIM_LAUNCH_PAIRS(double, false, 1, 2, w.tg); break;
            case 1: BIM_LAUNCH_PAIRS(double, false, 1, 4, w.tg); break;
            case 2: BIM_LAUNCH_PAIRS(double, false, 1, 8, w.tg); break;
            case 3: BIM_LAUNCH_PAIRS(double, false, 2, 2, w.tg); break;
            case 4: BIM_LAUNCH_PAIRS(double, false, 2, 4, w.tg); break;
            default: BIM_LAUNCH_PAIRS(double, false, 2, 8, w.tg); break;
        }
    } else {
        switch (vsel) {
            case 0: BIM_LAUNCH_PAIRS(float, true, 1, 2, w.tg32); break;
            case 1: BIM_LAUNCH_PAIRS(float, true, 1, 4, w.tg32); break;
            case 2: BIM_LAUNCH_PAIRS(float, true, 1, 8, w.tg32); break;
            case 3: BIM_LAUNCH_PAIRS(float, true, 2, 2, w.tg32); break;
            case 4: BIM_LAUNCH_PAIRS(float, true, 2, 4, w.tg32); break;
            default: BIM_LAUNCH_PAIRS(float, true, 2, 8, w.tg32); break;
        }
    }
#undef BIM_LAUNCH_PAIRS
    if (ev_pair) BIM_HIP(hipEventRecord(ev_pair[1], s));
    if (pairs64)
        hipLaunchKernelGGL(k_finalize64, dim3(finalize_blocks(N, M)), dim3(256), 0, s, D, s2_chunks);
    else
        hipLaunchKernelGGL(k_finalize, dim3(finalize_blocks(N, M)), dim3(256), 0, s, D);
    return hip_check(hipGetLastError(), "residual kernel launch");
}


BatchShape residual_batched_shape(const bim_problem *probs, int count, const PairLaunch *pls, int max_blocks) {
    BatchShape sh{pls[0].tpl, pls[0].unroll, 0, 0, 0, 1};
    long total = 0;
    for (int i = 0; i < count; ++i) {
        const Dims d(&probs[i]);
        sh.b_int += 3 * d.M;
        sh.b_rec += record_blocks(d.N, d.M);
        sh.b_fin += finalize_blocks(d.N, d.M);
        total += (long)pls[i].target_tiles * pls[i].chunks;
    }
    const long want = (total + 3) / 4;
    sh.blocks = (int)std::max(1L, std::min(want, (long)(max_blocks > 0 ? max_blocks : 2048)));
    return sh;
}

int residual_batched_fill(const bim_problem *probs, int count, const int *active, const double *const *u,
                          double *const *F, int prec, const PairLaunch *pls, const ResidualWork *ws,
                          PairDesc *descs, long *total_items) {
    const int tpl = pls[0].tpl, unroll = pls[0].unroll;
    long total = 0;
    int b_int = 0, b_rec = 0, b_fin = 0;
    for (int i = 0; i < count; ++i) {
        const bim_problem *p = &probs[i];
        const Dims d(p);
        const PairLaunch &pl = pls[i];
        if (pl.tpl != tpl || pl.unroll != unroll) return fail(BIM_EINVAL, "batched launch needs one kernel variant");
        const int on = active ? active[i] : 1;
        if (on && (!u[i] || !F[i])) return fail(BIM_EINVAL, "an active problem needs u and F");
        PairDesc &D = descs[i];
        D = make_desc(p, d, pl, ws[i], on ? u[i] : nullptr, on ? F[i] : nullptr, prec, 0);
        D.active = on;
        D.item0 = total;
        if (on) total += (long)pl.target_tiles * pl.chunks;
        D.blk_int = b_int;
        D.blk_rec = b_rec;
        D.blk_fin = b_fin;
        b_int += 3 * d.M;
        b_rec += record_blocks(d.N, d.M);
        b_fin += finalize_blocks(d.N, d.M);
    }
    for (int i = 0; i < count; ++i) descs[i].batch_items = total;
    *total_items = total;
    return BIM_OK;
}

int residual_batched_launch(const PairDesc *descs_dev, int count, int prec, const BatchShape &sh, hipStream_t s,
                            hipEvent_t *ev_pair) {
    if (count <= 0) return BIM_OK;
    hipLaunchKernelGGL(k_integrate_batched, dim3(sh.b_int), dim3(64), 0, s, descs_dev, count);
    if (prec == BIM_FP64)
        hipLaunchKernelGGL(k_records_batched<double>, dim3(sh.b_rec), dim3(256), 0, s, descs_dev, count);
    else
        hipLaunchKernelGGL(k_records_batched<float>, dim3(sh.b_rec), dim3(256), 0, s, descs_dev, count);
    if (ev_pair) BIM_HIP(hipEventRecord(ev_pair[0], s));
#define BIM_LAUNCH_BATCH(T, COMP, TPL, UNR) \
    hipLaunchKernelGGL((k_allpairs_batched<T, COMP, TPL, UNR>), dim3(sh.blocks), dim3(256), 0, s, descs_dev, count)
    const int vsel = (sh.tpl == 2 ? 3 : 0) + (sh.unroll == 2 ? 0 : sh.unroll == 4 ? 1 : 2);
    if (prec == BIM_FP64) {
        switch (vsel) {
            case 0: BIM_LAUNCH_BATCH(double, false, 1, 2); break;
            case 1: BIM_LAUNCH_BATCH(double, false, 1, 4); break;
            case 2: BIM_LAUNCH_BATCH(double, false, 1, 8); break;
            case 3: BIM_LAUNCH_BATCH(double, false, 2, 2); break;
            case 4: BIM_LAUNCH_BATCH(double, false, 2, 4); break;
            default: BIM_LAUNCH_BATCH(double, false, 2, 8); break;
        }
    } else {
        switch (vsel) {
            case 0: BIM_LAUNCH_BATCH(float, true, 1, 2); break;
            case 1: BIM_LAUNCH_BATCH(float, true, 1, 4); break;
            case 2: BIM_LAUNCH_BATCH(float, true, 1, 8); break;
            case 3: BIM_LAUNCH_BATCH(float, true, 2, 2); break;
            case 4: BIM_LAUNCH_BATCH(float, true, 2, 4); break;
            default: BIM_LAUNCH_BATCH(float, true, 2, 8); break;
        }
    }
#undef BIM_LAUNCH_BATCH
    if (ev_pair) BIM_HIP(hipEventRecord(ev_pair[1], s));
    hipLaunchKernelGGL(k_finalize_batched, dim3(sh.b_fin), dim3(256), 0, s, descs_dev, count);
    return hip_check(hipGetLastError(), "batched residual launch");
}

int residual_batched_enqueue(const bim_problem *probs, int count, const double *const *u, double *const *F,
                             int prec, const PairLaunch *pls, const ResidualWork *ws, PairDesc *descs_dev,
                             int max_blocks, hipStream_t s, hipEvent_t *ev_pair) {
    if (count <= 0) return BIM_OK;
    std::vector<PairDesc> descs(count);
    long total = 0;
    int rc = residual_batched_fill(probs, count, nullptr, u, F, prec, pls, ws, descs.data(), &total);
    if (rc) return rc;
    BIM_HIP(hipMemcpyAsync(descs_dev, descs.data(), sizeof(PairDesc) * count, hipMemcpyHostToDevice, s));
    return residual_batched_launch(descs_dev, count, prec, residual_batched_shape(probs, count, pls, max_blocks), s,
                                   ev_pair);
}

}  // namespace bim
