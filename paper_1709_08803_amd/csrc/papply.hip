// The FP64-stored preconditioner's apply z = P^-1 r on one problem: the parts that
// are not the Schur complement's inverse.
//
// The dense blocks of P are banded convolutions.  On the planes z = 0 and
// z = -1 of the linearised problem the kernels depend on a node only through
// its offset from the collocation point, so that the row of P21 (K5 = 1/r), P31
// (K7 = (r^2+1)^(-1/2)) and P23 = P32 (K6 = (r^2+1)^(-3/2) on node values) for
// target (k, l) and source slice m is
//   sum_i w_i,m [tab_K(|m - l|, i - k - 1/2) + tab_K(m + l, i - k - 1/2)] f_i,m
// (the second table row is the mirror image, on a half domain), w the trapezoid
// weight.  The tables hold 3 (2M - 1)(N - 1) values (0.5 MB at 181 x 61) where
// the blocks themselves are 3 M (2h+1) s^2 (1.0 GB at 181 x 61, h = 10, and
// another 0.34 GB for G = P33^-1 (P32 - P31 E)), and products with the stored
// blocks are bound by reading them (250 of the 422 us of an apply at 181 x 61).
// Formed from the tables the same products read a few MB and are bound by FP64
// FMAs, LDS reads and launches: 422 -> 237 us per apply at 181 x 61, of which
// 166 us were the two triangular products of the Schur inverse (122 us in groups of
// slices, precond_groups: 197 us per apply).  The tables
// hold the exact mesh offsets, where the blocks were formed from rounded node
// coordinates (a difference of 1e-14 relative next to the target).  (The lockstep
// solver and the FP32-stored operator go on with the stored blocks: the latter's
// elements are the rounded blocks themselves, G's rounding not being that of
// its factors.)
//
// Sequence (E = P11^-1 P12; D22^-1 the inverse of the slice block P22 = P33; T
// the trapezoidal node values of a slice; conv(K, q) the banded convolution):
//   k_pc_slice<0>  a1 = P11^-1 r1,  q1 = w a1_x
//   k_pc_conv<0>   p1 = conv(K7, q1), p2 = conv(K5, q1)
//   k_pc_a3        a3 = D22^-1 (r3 - p1),  q1 = w T a3
//   k_pc_conv<1>   p1 = conv(K6, q1)
//   k_pc_rhs       t2 = r2 - p2 + corr (..) - p1      (the right-hand side of S)
//   [z2 = S^-1 t2: block-triangular products]
//   k_pc_slice<2>  e = E z2:  z1 = a1 - e,  q2 = w e_x,  q1 = w T z2
//   k_pc_conv<2>   p1 = conv(K6, q1) - conv(K7, q2)
//   k_pc_slice<3>  z3 = a3 - D22^-1 p1                (G z2 without G)
#include <hip/hip_runtime.h>

#include <algorithm>

#include "bim_common.h"
#include "precond.h"

namespace bim {

namespace {

template <typename T>
using ConstPtr = const __attribute__((address_space(4))) T *;
template <typename T>
using GlobalPtr = __attribute__((address_space(1))) T *;
typedef double d2_t __attribute__((ext_vector_type(2)));

inline int cdiv(long a, long b) { return (int)((a + b - 1) / b); }

// ------------------------------------------------------------------ banded convolutions
// One wave: targets k0 .. k0 + R - 1 of slice l in every lane (k0 = R lane + 64 R
// kb: all N - 1 of them for N <= 64 R + 1) against an equal share of the nodes
// of the band's source slices (chunks x 4 waves share them; a share may start
// and end inside a slice).  The slice's table, both images added, lies in the
// wave's own part of LDS; from node i to i + 1 every target's entry moves by
// one, so a lane reads one new entry per node and table and keeps the other
// R - 1 in registers (R FMAs per LDS read; with one target per lane the LDS
// reads bound the loop).  The weighted sources are uniform: scalar loads, the
// next batch in flight during the current one.  The four waves' sums are added in
// LDS and the chunks' by the reader, in a fixed order.
// Nodes per scalar-load batch (a multiple of R): 12, with two sources half of it,
// as the current and the next batch of both fill the scalar registers.
template <int MODE, int R>
constexpr int kBatch = MODE != 2 ? 12 : R == 4 ? 4 : 6;
constexpr int kFront = 4;    // entries before the first node's (R - 1 are read)
constexpr int kPiece = 512;  // nodes of a slice per table window
constexpr int kFill = 6;     // table entries per lane in flight
constexpr int kMaxChunks = 8;  // a reader adds at most so many partial sums

// entries of a wave's table window: those a piece of a slice can meet in 64 R targets
__host__ __device__ __forceinline__ int conv_window(int N, int R) {
    return (N < kPiece ? N : kPiece) + 64 * R + kFront + 12;
}

extern __shared__ double conv_lds[];

template <int MODE, int R>
__global__ __launch_bounds__(256) void k_pc_conv(PcDesc D) {
    const int b = blockIdx.x;
    double *tabs = conv_lds;
    constexpr int NT = MODE == 1 ? 1 : 2;      // tables
    constexpr int NA = MODE == 0 ? 2 : 1;      // accumulators per target
    constexpr int NQ = MODE == 2 ? 2 : 1;      // sources
    const int N = D.N, M = D.M, h = D.h, nk = N - 1;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int kbs = (nk + 64 * R - 1) / (64 * R);
    const int c = b % D.chunks, rest = b / D.chunks;
    const int kb = rest % kbs, l = rest / kbs;
    if (l >= M) return;  // uniform in the workgroup
    const int LT = conv_window(N, R);
    double *tw = tabs + (size_t)wave * NT * LT;
    // table order: mode 0: K7, K5; mode 1: K6; mode 2: K6, K7
    const size_t tsz = (size_t)(2 * M - 1) * nk;
    const GlobalPtr<const double> tab = (GlobalPtr<const double>)D.tab;
    const GlobalPtr<const double> tk[2] = {tab + (MODE == 0 ? 2 : 1) * tsz, tab + (MODE == 0 ? 0 : 2) * tsz};
    const ConstPtr<double> q1 = (ConstPtr<double>)D.q1, q2 = (ConstPtr<double>)D.q2;
    constexpr int KB = kBatch<MODE, R>;
    const int kbase = kb * 64 * R, k0 = kbase + lane * R;
    const int m0 = max(0, l - h), m1 = min(M - 1, l + h);
    const int nsrc = (m1 - m0 + 1) * N, parts = 4 * D.chunks, part = c * 4 + wave;
    const int e0 = (int)((long)nsrc * part / parts), e1 = (int)((long)nsrc * (part + 1) / parts);
    double acc[NA][R] = {};
    for (int e = e0; e < e1;) {
        // nodes [i0, i1) of source slice m
        const int row = e / N, m = m0 + row;
        const int i0 = e - row * N, i1 = min(min(e1 - row * N, N), i0 + kPiece);
        e += i1 - i0;
        const size_t o1 = (size_t)abs(m - l) * nk, o2 = (size_t)(m + l) * nk;
        // window entry t is the kernel at offset d - 1/2 = i - k - 1/2, d = dlo + t; zero
        // where no target and node have that offset
        const int dlo = i0 - (kbase + 64 * R - 1) - kFront;
        // (kFill entries per lane at a time, their loads unconditional at clamped
        // indices and all in flight together: one by one, a wave waited for L2 at
        // every 64 entries)
        const int need = i1 - i0 + 64 * R + kFront + 12;
        for (int t0 = lane; t0 < need; t0 += 64 * kFill) {
            double v[NT][kFill], w[NT][kFill];
#pragma unroll
            for (int f = 0; f < kFill; ++f) {
                const int d = dlo + t0 + 64 * f;
                const int en = min(d >= 1 ? d - 1 : -d, nk - 1);
#pragma unroll
                for (int q = 0; q < NT; ++q) {
                    v[q][f] = tk[q][o1 + en];
                    w[q][f] = tk[q][o2 + en];
                }
            }
#pragma unroll
            for (int f = 0; f < kFill; ++f) {
                const int t = t0 + 64 * f, d = dlo + t;
                const bool in = (d >= 1 ? d - 1 : -d) < nk;
                if (t < need)
#pragma unroll
                    for (int q = 0; q < NT; ++q)
                        tw[q * LT + t] = in ? (D.half ? v[q][f] + w[q][f] : v[q][f]) : 0.0;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        // node i0 + i of target k0: entry kFront + i + 64 R - 1 - R lane
        const double *tl = tw + kFront + 64 * R - 1 - R * lane;
        const ConstPtr<double> s1 = q1 + (size_t)m * N + i0, s2 = q2 + (size_t)m * N + i0;
        const int len = i1 - i0;
        double old[NT][R];  // old[q][x] = entry of node i - x for target k0, x = 1 .. R - 1
#pragma unroll
        for (int q = 0; q < NT; ++q)
#pragma unroll
            for (int x = 1; x < R; ++x) old[q][x] = tl[q * LT - x];
        // A batch: its table entries and sources, loaded during the batch before (both
        // count on the wave's one LDS and scalar-load counter, so one wait at the
        // hand-over covers them; loads past the piece read spare entries, not used).
        struct Batch {
            double t[NT][KB], s[NQ][KB];
        };
        auto fetch = [&](Batch &b, int i) {
            i = min(i, len - 1);
#pragma unroll
            for (int j = 0; j < KB; ++j) {
                b.s[0][j] = s1[i + j];
                if (NQ == 2) b.s[NQ - 1][j] = s2[i + j];
            }
#pragma unroll
            for (int q = 0; q < NT; ++q)
#pragma unroll
                for (int j = 0; j < KB; ++j) b.t[q][j] = tl[q * LT + i + j];
        };
        auto batch = [&](Batch &b, Batch &next, int i) {
            fetch(next, i + KB);
            if (i + KB > len) {  // nodes past the piece count zero
#pragma unroll
                for (int j = 0; j < KB; ++j)
#pragma unroll
                    for (int q = 0; q < NQ; ++q) b.s[q][j] = i + j < len ? b.s[q][j] : 0.0;
            }
            __builtin_amdgcn_sched_barrier(0);  // the loads stay ahead of the FMAs
#pragma unroll
            for (int g = 0; g < KB; g += R) {
#pragma unroll
                for (int j = 0; j < R; ++j)
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        const double v0 = j >= r ? b.t[0][j >= r ? g + j - r : 0] : old[0][j >= r ? 0 : r - j];
                        acc[0][r] = fma(v0, b.s[0][g + j], acc[0][r]);
                        if (NT == 2) {
                            const double v1 =
                                j >= r ? b.t[NT - 1][j >= r ? g + j - r : 0] : old[NT - 1][j >= r ? 0 : r - j];
                            if (MODE == 0) acc[NA - 1][r] = fma(v1, b.s[0][g + j], acc[NA - 1][r]);
                            else acc[0][r] = fma(-v1, b.s[NQ - 1][g + j], acc[0][r]);
                        }
                    }
#pragma unroll
                for (int q = 0; q < NT; ++q)
#pragma unroll
                    for (int x = 1; x < R; ++x) old[q][x] = b.t[q][g + R - x];
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        Batch b0, b1;
        fetch(b0, 0);
        for (int i = 0; i < len; i += 2 * KB) {
            batch(b0, b1, i);
            if (i + KB < len) batch(b1, b0, i + KB);
        }
        __builtin_amdgcn_wave_barrier();  // the next piece overwrites the window
    }
    // the four waves' sums through the windows' memory (no longer read)
    __syncthreads();
    double(*red)[NA * R][64] = reinterpret_cast<double(*)[NA * R][64]>(conv_lds);
    if (wave > 0) {
#pragma unroll
        for (int a = 0; a < NA; ++a)
#pragma unroll
            for (int r = 0; r < R; ++r) red[wave - 1][a * R + r][lane] = acc[a][r];
    }
    __syncthreads();
    if (wave > 0) return;
    const size_t at = ((size_t)c * M + l) * nk;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (k0 + r >= nk) continue;
#pragma unroll
        for (int a = 0; a < NA; ++a) {
            const double v = ((acc[a][r] + red[0][a * R + r][lane]) + red[1][a * R + r][lane]) + red[2][a * R + r][lane];
            ((GlobalPtr<double>)(a == 0 ? D.p1 : D.p2))[at + k0 + r] = v;
        }
    }
}

// ------------------------------------------------------------------ slice products
// Rows of the s x s slice blocks (and of the node-value map stacked below E) times
// one slice of a vector that is formed on the way in; the same block serves every
// slice (it stays in L2: 0.3 MB at s = 182, where a copy per slice was 16 MB).
constexpr int kMaxSlice = 1024;
constexpr int kRowsPerGroup = 16;

__device__ __forceinline__ double weight(const PcDesc &D, int l, int i) {
    const double ci = (i == 0 || i == D.N - 1) ? 0.5 : 1.0, cl = (l == 0 || l == D.M - 1) ? 0.5 : 1.0;
    return D.dx * D.dy * ci * cl;
}

__device__ __forceinline__ double chunk_sum(GlobalPtr<const double> p, int chunks, size_t stride, size_t at) {
    double q[kMaxChunks];  // all loads in flight
#pragma unroll
    for (int c = 0; c < kMaxChunks; ++c) q[c] = p[min(c, chunks - 1) * stride + at];
    double v = q[0];
#pragma unroll
    for (int c = 1; c < kMaxChunks; ++c) v += c < chunks ? q[c] : 0.0;
    return v;
}

// Rows r0 .. r0 + 3 (below `rows`) of A (leading dimension s) times x (LDS): the
// result of row r0 + lane in lanes 0 .. 3.
__device__ __forceinline__ double rows4(GlobalPtr<const double> A, int s, int rows, int r0, const double *x, int lane) {
    double acc[4] = {};
    if (s % 2 == 0) {  // rows aligned to two elements
        for (int q = lane; q < s / 2; q += 64) {
            const d2_t xv = *reinterpret_cast<const d2_t *>(x + 2 * q);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const d2_t a = *(GlobalPtr<const d2_t>)(A + (size_t)min(r0 + e, rows - 1) * s + 2 * q);
                acc[e] = fma(a[0], xv[0], acc[e]);
                acc[e] = fma(a[1], xv[1], acc[e]);
            }
        }
    } else {
        for (int c = lane; c < s; c += 64)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[e] = fma(A[(size_t)min(r0 + e, rows - 1) * s + c], x[c], acc[e]);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
        acc[e] = wave_sum64(acc[e]);
    double v = acc[0];
#pragma unroll
    for (int e = 1; e < 4; ++e) v = lane == e ? acc[e] : v;
    return v;
}

// Slice l's value c of the convolution sums in p1 (zero on the radiation rows).
__device__ __forceinline__ double conv_value(const PcDesc &D, int l, int c) {
    if (c < 2) return 0.0;
    return chunk_sum((GlobalPtr<const double>)D.p1, D.chunks, (size_t)D.M * (D.N - 1), (size_t)l * (D.N - 1) + c - 2);
}

// 16 rows per workgroup, four per wave.  MODE 0: a1; 2: z1 and the sources of
// the last convolutions; 3: z3.
template <int MODE>
__host__ __device__ __forceinline__ int slice_rows(int N) { return MODE == 2 ? 2 * N + 1 : N + 1; }

template <int MODE>
__global__ __launch_bounds__(256) void k_pc_slice(PcDesc D) {
    __shared__ __align__(16) double x[kMaxSlice];
    const int N = D.N, s = D.s;
    const int rows = slice_rows<MODE>(N), rb = (rows + kRowsPerGroup - 1) / kRowsPerGroup;
    const int l = blockIdx.x / rb;
    const size_t ls = (size_t)l * s;
    for (int c = threadIdx.x; c < s; c += 256)
        x[c] = MODE == 0   ? ((GlobalPtr<const double>)D.r)[ls + c]
               : MODE == 2 ? ((GlobalPtr<const double>)D.z)[D.n + ls + c]
                           : conv_value(D, l, c);
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r0 = (blockIdx.x - l * rb) * kRowsPerGroup + 4 * wave;
    if (r0 >= rows) return;
    const GlobalPtr<const double> A = (GlobalPtr<const double>)(MODE == 0 ? D.iD11 : MODE == 2 ? D.ETs : D.iD22);
    const double v = rows4(A, s, rows, r0, x, lane);
    const int row = r0 + lane;
    if (lane >= 4 || row >= rows) return;
    const GlobalPtr<double> q1 = (GlobalPtr<double>)D.q1, q2 = (GlobalPtr<double>)D.q2;
    if (MODE == 0) {
        ((GlobalPtr<double>)D.a1)[ls + row] = v;
        if (row >= 1) q1[(size_t)l * N + row - 1] = weight(D, l, row - 1) * v;
    } else if (MODE == 3) {
        ((GlobalPtr<double>)D.z)[2 * D.n + ls + row] = ((GlobalPtr<const double>)D.a3)[ls + row] - v;
    } else if (row >= s) {
        q1[(size_t)l * N + row - s] = weight(D, l, row - s) * v;
    } else {
        ((GlobalPtr<double>)D.z)[ls + row] = ((GlobalPtr<const double>)D.a1)[ls + row] - v;
        if (row >= 1) q2[(size_t)l * N + row - 1] = weight(D, l, row - 1) * v;
    }
}

// a3 = D22^-1 (r3 - p1) and the weighted node values of the a3 that was computed
// (a product with the node values of D22^-1's columns would be one kernel's
// rows like the others, but leaves a3's own rounding, up to 1e5 of the result
// on fine meshes, out of the right-hand side of S): one workgroup per slice.
__global__ __launch_bounds__(1024) void k_pc_a3(PcDesc D) {
    __shared__ __align__(16) double x[kMaxSlice];
    __shared__ double y[kMaxSlice];
    const int N = D.N, s = D.s, l = blockIdx.x;
    const size_t ls = (size_t)l * s;
    for (int c = threadIdx.x; c < s; c += 1024)
        x[c] = ((GlobalPtr<const double>)D.r)[2 * D.n + ls + c] - conv_value(D, l, c);
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int r0 = 4 * wave; r0 < s; r0 += 64) {
        const double v = rows4((GlobalPtr<const double>)D.iD22, s, s, r0, x, lane);
        if (lane < 4 && r0 + lane < s) {
            y[r0 + lane] = v;
            ((GlobalPtr<double>)D.a3)[ls + r0 + lane] = v;
        }
    }
    __syncthreads();
    if (wave > 0) return;
    // node values by the trapezoidal rule: 64-wide scans, the total carried on
    const double hdx = 0.5 * D.dx;
    double carry = y[0];
    for (int base = 0; base < N; base += 64) {
        const int i = base + lane;
        double v = (i > 0 && i < N) ? hdx * (y[i] + y[i + 1]) : 0.0;
        for (int o = 1; o < 64; o <<= 1) {
            const double t = __shfl_up(v, o, 64);
            if (lane >= o) v += t;
        }
        if (i < N) ((GlobalPtr<double>)D.q1)[(size_t)l * N + i] = weight(D, l, i) * (carry + v);
        carry += __shfl(v, 63, 64);
    }
}

// t2 = r2 - P21 a1 - P23 a3; P21 carries the singular subtraction of the K5 sum
// on the target's own slice, corr = (sum of w K5 - integral of K5) / 2
__global__ __launch_bounds__(256) void k_pc_rhs(PcDesc D) {
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e >= D.n) return;
    const int nk = D.N - 1, l = e / D.s, c = e - l * D.s;
    double v = ((GlobalPtr<const double>)D.r)[D.n + e];
    if (c >= 2) {
        const size_t at = (size_t)l * nk + c - 2, pst = (size_t)D.M * nk;
        const GlobalPtr<const double> a1 = (GlobalPtr<const double>)D.a1;
        v -= chunk_sum((GlobalPtr<const double>)D.p2, D.chunks, pst, at) -
             ((GlobalPtr<const double>)D.corr)[at] * (a1[e - 1] + a1[e]);
        v -= chunk_sum((GlobalPtr<const double>)D.p1, D.chunks, pst, at);
    }
    ((GlobalPtr<double>)D.t2)[e] = v;
}

// ------------------------------------------------------------------ setup pieces
// tab[K][o][e]: K5, K6, K7 at the offset ((e + 1/2) dx, o dy)
__global__ void k_pc_tables(double *tab, int N, int M, double dx, double dy) {
    const long nk = N - 1, tsz = (2L * M - 1) * nk;
    const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= tsz) return;
    const int o = (int)(t / nk), e = (int)(t - o * nk);
    const double s = (e + 0.5) * dx, tt = o * dy, r2 = s * s + tt * tt;
    const double q = 1.0 / sqrt(r2 + 1.0);
    tab[t] = 1.0 / sqrt(r2);
    tab[tsz + t] = q * q * q;
    tab[2 * tsz + t] = q;
}
__global__ void k_pc_corr(const double *rowsum, const double *I5, double *corr, int ntg) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t < ntg) corr[t] = 0.5 * (rowsum[t] - I5[t]);
}
// [A; T]: the s rows of A and, below, the N rows of the node-value map of a slice
__global__ void k_pc_stack(const double *A, double *out, int N, double dx) {
    const int s = N + 1;
    const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (long)(s + N) * s) return;
    const int r = (int)(t / s), c = (int)(t - (long)r * s);
    double v;
    if (r < s) v = A[t];
    else if (c == 0) v = 1.0;
    else {  // coefficient of (f_x)_{c-1} in the value at node r - s
        const int i = r - s, j = c - 1;
        v = (i == 0 || j > i) ? 0.0 : (j == 0 || j == i) ? 0.5 * dx : dx;
    }
    out[t] = v;
}

// Targets per lane of the convolutions: the R of 1 .. 4 with the least work per
// node, blocks of 64 R targets times R FMAs and one LDS read (0.7 of an FMA's
// issue time on the shared LDS port).
int pc_conv_targets(int N) {
    int best = 1;
    double cost = 1e30;
    for (int R = 1; R <= 4; ++R) {
        const double c = cdiv(N - 1, 64 * R) * (R + 0.7);
        if (c < cost) {
            cost = c;
            best = R;
        }
    }
    return best;
}

template <int MODE>
int conv_launch(const PcDesc &D, hipStream_t st) {
    const int R = pc_conv_targets(D.N);
    const dim3 grid(D.M * cdiv(D.N - 1, 64 * R) * D.chunks);
    // the windows; at least the reduction's 3 R x 64 values per accumulator
    const size_t lds =
        sizeof(double) * std::max(4 * (MODE == 1 ? 1 : 2) * conv_window(D.N, R), 3 * (MODE == 0 ? 2 : 1) * R * 64);
    switch (R) {
        case 1: hipLaunchKernelGGL((k_pc_conv<MODE, 1>), grid, dim3(256), lds, st, D); break;
        case 2: hipLaunchKernelGGL((k_pc_conv<MODE, 2>), grid, dim3(256), lds, st, D); break;
        case 3: hipLaunchKernelGGL((k_pc_conv<MODE, 3>), grid, dim3(256), lds, st, D); break;
        default: hipLaunchKernelGGL((k_pc_conv<MODE, 4>), grid, dim3(256), lds, st, D); break;
    }
    return BIM_OK;
}
template <int MODE>
void slice_launch(const PcDesc &D, hipStream_t st) {
    hipLaunchKernelGGL(k_pc_slice<MODE>, dim3(D.M * cdiv(slice_rows<MODE>(D.N), kRowsPerGroup)), dim3(256), 0, st, D);
}

}  // namespace

// Source chunks: about 512 workgroups (2048 waves, two per SIMD), with at least 96
// nodes per wave, as a wave spends about that many nodes' time on its table
// window, and at most kMaxChunks.  Measured at 181 x 61 (three convolutions of
// an apply): 49 us with 244 workgroups, 40 with 488, 38 with 976, whose readers
// lose more than that on the partial sums.
int pc_conv_chunks(int N, int M, int h) {
    const int R = pc_conv_targets(N);
    const int fill = cdiv(512, (long)M * cdiv(N - 1, 64 * R)), most = std::max(1, (2 * h + 1) * N / (4 * 96));
    return std::max(1, std::min({kMaxChunks, fill, most}));
}

int pc_before_schur(const PcDesc &D, hipStream_t st) {
    slice_launch<0>(D, st);
    conv_launch<0>(D, st);
    hipLaunchKernelGGL(k_pc_a3, dim3(D.M), dim3(1024), 0, st, D);
    conv_launch<1>(D, st);
    hipLaunchKernelGGL(k_pc_rhs, dim3(cdiv(D.n, 256)), dim3(256), 0, st, D);
    return hip_check(hipGetLastError(), "preconditioner apply launch");
}

int pc_after_schur(const PcDesc &D, hipStream_t st) {
    slice_launch<2>(D, st);
    conv_launch<2>(D, st);
    slice_launch<3>(D, st);
    return hip_check(hipGetLastError(), "preconditioner apply launch");
}

int kernel_tables_enqueue(double *tab, int N, int M, double dx, double dy, hipStream_t st) {
    hipLaunchKernelGGL(k_pc_tables, dim3(cdiv((2L * M - 1) * (N - 1), 256)), dim3(256), 0, st, tab, N, M, dx, dy);
    return hip_check(hipGetLastError(), "kernel tables launch");
}

int pc_corr_enqueue(const double *rowsum, const double *I5, double *corr, int N, int M, hipStream_t st) {
    hipLaunchKernelGGL(k_pc_corr, dim3(cdiv((long)(N - 1) * M, 256)), dim3(256), 0, st, rowsum, I5, corr, (N - 1) * M);
    return hip_check(hipGetLastError(), "preconditioner correction launch");
}

int pc_stack_enqueue(const double *A, double *out, int N, double dx, hipStream_t st) {
    hipLaunchKernelGGL(k_pc_stack, dim3(cdiv((2L * N + 1) * (N + 1), 256)), dim3(256), 0, st, A, out, N, dx);
    return hip_check(hipGetLastError(), "preconditioner node map launch");
}

}  // namespace bim
