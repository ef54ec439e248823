// The sums of the linearised residual (Section 4.2) in FP64 as convolutions.
//
// On the planes z = 0 and z = -1 the kernels depend on a source node only through
// its offset (s, t) from the collocation point, s = (i - k - 1/2) dx and t = (+-j
// - l) dy, so that with the tables K5 = 1/r, K7 = (r^2 + 1)^(-1/2) and K6 = K7^3 by
// offset (3 (2M - 1)(N - 1) values, two images added on a half domain) the rows are
//   surface:  sum  w sigma_S K5 - w sigma_B K7 + w D_B K6      S2: sum w K5
//   bottom:   sum -w sigma_B K5 + w sigma_S K7 + w D_S K6      S2: sum -w K5
// (sigma_S = zeta_x, sigma_B = beta_x, D = phi - x, psi - x: the weighted values of
// the node records).  A pair of slices costs 7 FMAs per target and node for both
// boundaries and both images, against 8 reciprocal square roots with ~60 FP64
// operations in the pairwise form: 513 -> 54 us for the sums at 181 x 61.
//
// One wave takes R targets per lane of slice l (k0 .. k0 + R - 1, k0 = 64 R kb + R
// lane) against an equal share of all 2-D nodes; the window of the three tables
// lies in the wave's part of LDS, moves by one entry per node, and a lane reads one
// new entry per table and node (21 FMAs per 3 reads at R = 3: bound by FP64 issue,
// 84 cycles per wave and node, 24 us at 181 x 61, and by filling the windows).  The node values are scalar loads, one batch
// ahead.  Partial sums go to [chunk][target][2] as the pairwise kernel's do.
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

constexpr int kPiece = 256;  // nodes of a slice per table window
constexpr int kFront = 4;    // entries before the first node's (R - 1 are read)
constexpr int kFill = 4;     // table entries per lane in flight (of each of the three tables)
template <int R>
constexpr int kBatch = R == 3 ? 3 : 4;  // nodes per batch: a multiple of R

__host__ __device__ __forceinline__ int window(int N, int R) {
    return (N < kPiece ? N : kPiece) + 64 * R + kFront + 4;
}

extern __shared__ double lin_lds[];

template <int R>
__global__ __launch_bounds__(256) void k_lin_conv(PairDesc D, const double *__restrict__ tables, int chunks) {
    constexpr int KB = kBatch<R>;
    const int N = D.N, M = D.M, nk = N - 1;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int kbs = (nk + 64 * R - 1) / (64 * R);
    const int c = blockIdx.x % chunks, rest = blockIdx.x / chunks;
    const int kb = rest % kbs, l = rest / kbs;
    const int LT = window(N, R);
    double *tw = lin_lds + (size_t)wave * 3 * LT;
    const size_t tsz = (size_t)(2 * M - 1) * nk;
    const GlobalPtr<const double> tab = (GlobalPtr<const double>)tables;  // K5, K6, K7
    // {w D, w sigma} of the node records
    const ConstPtr<d2_t> recS = (ConstPtr<d2_t>)D.srcS + 2, recB = (ConstPtr<d2_t>)D.srcB + 2;
    const int kbase = kb * 64 * R, k0 = kbase + lane * R;
    const int nsrc = M * N, parts = 4 * chunks, part = c * 4 + wave;
    const int e0 = (int)((long)nsrc * part / parts), e1 = (int)((long)nsrc * (part + 1) / parts);
    double aS[R] = {}, aB[R] = {}, a2[R] = {};
    for (int e = e0; e < e1;) {
        // nodes [i0, i1) of source slice m
        const int m = e / N;
        const int i0 = e - m * N, i1 = min(min(e1 - m * N, N), i0 + kPiece), len = i1 - i0;
        e += len;
        const size_t o1 = (size_t)abs(m - l) * nk, o2 = (size_t)(m + l) * nk;
        // window entry t: the kernels at offset d - 1/2 = i - k - 1/2, d = dlo + t; zero
        // where no target and node have that offset
        const int dlo = i0 - (kbase + 64 * R - 1) - kFront;
        const int need = len + 64 * R + kFront + 4;
        for (int t0 = lane; t0 < need; t0 += 64 * kFill) {
            double v[3][kFill], w[3][kFill];
#pragma unroll
            for (int f = 0; f < kFill; ++f) {
                const int d = dlo + t0 + 64 * f;
                const int en = min(d >= 1 ? d - 1 : -d, nk - 1);
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    v[q][f] = tab[q * tsz + o1 + en];
                    w[q][f] = tab[q * tsz + o2 + en];
                }
            }
#pragma unroll
            for (int f = 0; f < kFill; ++f) {
                const int t = t0 + 64 * f, d = dlo + t;
                const bool in = (d >= 1 ? d - 1 : -d) < nk;
                if (t < need)
#pragma unroll
                    for (int q = 0; q < 3; ++q) tw[q * LT + t] = in ? (D.half ? v[q][f] + w[q][f] : v[q][f]) : 0.0;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        // node i0 + i of target k0: entry kFront + i + 64 R - 1 - R lane
        const double *tl = tw + kFront + 64 * R - 1 - R * lane;
        const ConstPtr<d2_t> sS = recS + ((size_t)m * N + i0) * 4, sB = recB + ((size_t)m * N + i0) * 4;
        double old[3][R], s2[R] = {};  // old[q][x] = entry of node i - x for target k0
#pragma unroll
        for (int q = 0; q < 3; ++q)
#pragma unroll
            for (int x = 1; x < R; ++x) old[q][x] = tl[q * LT - x];
        // A batch: its table entries and node values, loaded during the batch before
        // (both count on the wave's one LDS and scalar-load counter, so one wait at the
        // hand-over covers them; loads past the piece read the window's spare entries
        // and the next slice's or the spare records, and are not used).
        struct Batch {
            double t[3][KB];
            d2_t S[KB], B[KB];
        };
        auto fetch = [&](Batch &b, int i) {
            i = min(i, len - 1);
#pragma unroll
            for (int j = 0; j < KB; ++j) {
                b.S[j] = sS[4 * (i + j)];
                b.B[j] = sB[4 * (i + j)];
            }
#pragma unroll
            for (int q = 0; q < 3; ++q)
#pragma unroll
                for (int j = 0; j < KB; ++j) b.t[q][j] = tl[q * LT + i + j];
        };
        auto batch = [&](Batch &b, Batch &next, int i) {
            fetch(next, i + KB);
            double on[KB];  // nodes past the piece count zero
#pragma unroll
            for (int j = 0; j < KB; ++j) {
                on[j] = 1.0;
                if (i + KB > len) {
                    const bool in = i + j < len;
                    on[j] = in ? 1.0 : 0.0;
                    b.S[j] = in ? b.S[j] : d2_t{0.0, 0.0};
                    b.B[j] = in ? b.B[j] : d2_t{0.0, 0.0};
                }
            }
            __builtin_amdgcn_sched_barrier(0);  // the loads stay ahead of the FMAs
#pragma unroll
            for (int g = 0; g < KB; g += R) {
#pragma unroll
                for (int j = 0; j < R; ++j)
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        double t[3];
#pragma unroll
                        for (int q = 0; q < 3; ++q)
                            t[q] = j >= r ? b.t[q][j >= r ? g + j - r : 0] : old[q][j >= r ? 0 : r - j];
                        const d2_t vS = b.S[g + j], vB = b.B[g + j];  // {w D, w sigma}; B with -w
                        aS[r] = fma(t[0], vS[1], aS[r]);
                        aB[r] = fma(t[0], vB[1], aB[r]);
                        s2[r] = fma(t[0], on[g + j], s2[r]);
                        aS[r] = fma(t[2], vB[1], aS[r]);
                        aB[r] = fma(t[2], vS[1], aB[r]);
                        aS[r] = fma(-t[1], vB[0], aS[r]);  // source plane 1 below the surface target
                        aB[r] = fma(t[1], vS[0], aB[r]);   // and 1 above the bottom target
                    }
#pragma unroll
                for (int q = 0; q < 3; ++q)
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
        // the S2 sum's trapezoid weights: half at the ends of the slice
        const double wm = D.dx * D.dy * ((m == 0 || m == M - 1) ? 0.5 : 1.0);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (i0 == 0) s2[r] = fma(-0.5, tl[-r], s2[r]);
            if (i1 == N) s2[r] = fma(-0.5, tl[len - 1 - r], s2[r]);
            a2[r] = fma(wm, s2[r], a2[r]);
        }
        __builtin_amdgcn_wave_barrier();  // the next piece overwrites the window
    }
    // the four waves' sums through the windows' memory (no longer read)
    __syncthreads();
    double(*red)[3 * R][64] = reinterpret_cast<double(*)[3 * R][64]>(lin_lds);
    if (wave > 0) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            red[wave - 1][r][lane] = aS[r];
            red[wave - 1][R + r][lane] = aB[r];
            red[wave - 1][2 * R + r][lane] = a2[r];
        }
    }
    __syncthreads();
    if (wave > 0) return;
    const size_t ntg = (size_t)nk * M;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (k0 + r >= nk) continue;
        auto sum = [&](double v, int at) { return ((v + red[0][at][lane]) + red[1][at][lane]) + red[2][at][lane]; };
        const double s2 = sum(a2[r], 2 * R + r);
        const GlobalPtr<d2_t> o = (GlobalPtr<d2_t>)D.part + (size_t)c * 2 * ntg + (size_t)l * nk + k0 + r;
        o[0] = d2_t{sum(aS[r], r), s2};
        o[ntg] = d2_t{sum(aB[r], R + r), -s2};  // bottom records carry -w
    }
}

// Targets per lane: the R with the least FMAs in flight for the N - 1 targets (7 R per
// node and block of 64 R) and three LDS reads per node.
int conv_targets(int N) {
    int best = 1;
    double cost = 1e30;
    for (int R = 1; R <= 4; ++R) {
        const double c = cdiv(N - 1, 64 * R) * (7.0 * R + 3.0);
        if (c < cost) {
            cost = c;
            best = R;
        }
    }
    return best;
}

}  // namespace

// A wave fills a window of 64 R + N entries for every pair of slices, however short these
// are, where the pairwise form's work goes with nimg N^2: narrow meshes stay with that (whole
// evaluation, pairwise / convolution in us, M = 900: half domain N = 3 60 / 583, 16 822 /
// 898, 20 1308 / 995; full N = 16 438 / 899, 24 938 / 1121; M = 300: full N = 24 134 / 142,
// 31 211 / 173).  So do meshes of few nodes, whose convolution is one chunk of launches and
// latencies (N < 31: 24 x 31 42.6 / 45.1, 24 x 61 44.6 / 35.7; from 31 on the line is lower:
// 66 x 3 20.3 / 23.5, 31 x 11 28.2 / 29.1, 31 x 12 29.3 / 29.4, 129 x 3 31.2 / 30.4, 40 x 12
// 35.4 / 32.9, and the tables' launch, 2 to 3 us of it, is not paid again where they are kept).
bool lin_conv_applies(const Dims &d, bool tables_kept) {
    if ((long)d.nimg * d.N * d.N < 648) return false;
    return d.N < 31 ? d.nnode >= 768 : tables_kept || d.nnode >= 372;
}

size_t lin_table_bytes(const Dims &d) {
    return ((sizeof(double) * 3 * (size_t)(2 * d.M - 1) * (d.N - 1)) + 255) & ~(size_t)255;
}

// Source chunks: about 1024 workgroups (four waves per SIMD), shares of at least 96
// nodes per wave (a wave spends about that many nodes' time on a table window), and no
// more than the partial-sum buffer holds.
int lin_conv_chunks(const Dims &d, int most) {
    const int blocks = d.M * cdiv(d.N - 1, 64 * conv_targets(d.N));
    const int fill = 1024 / blocks, share = std::max(1, d.nnode / (4 * 96));
    return std::max(1, std::min({most, fill, share}));
}

int lin_conv_enqueue(const PairDesc &D, const double *tables, hipStream_t s) {
    const int R = conv_targets(D.N);
    const dim3 grid(D.M * cdiv(D.N - 1, 64 * R) * D.chunks);
    // the windows; at least the reduction's 9 R x 64 values
    const size_t lds = sizeof(double) * std::max(4 * 3 * window(D.N, R), 9 * R * 64);
    switch (R) {
        case 1: hipLaunchKernelGGL(k_lin_conv<1>, grid, dim3(256), lds, s, D, tables, D.chunks); break;
        case 2: hipLaunchKernelGGL(k_lin_conv<2>, grid, dim3(256), lds, s, D, tables, D.chunks); break;
        case 3: hipLaunchKernelGGL(k_lin_conv<3>, grid, dim3(256), lds, s, D, tables, D.chunks); break;
        default: hipLaunchKernelGGL(k_lin_conv<4>, grid, dim3(256), lds, s, D, tables, D.chunks); break;
    }
    return hip_check(hipGetLastError(), "linear convolution launch");
}

}  // namespace bim
