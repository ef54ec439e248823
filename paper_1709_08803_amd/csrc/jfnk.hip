// Jacobian-free Newton-Krylov driver (Section 3.2): damped inexact Newton with a
// backtracking line search on ||F||_2, each step solved by restarted GMRES with
// right preconditioning, the Jacobian action replaced by the first-order
// difference quotient of the residual.  All vectors stay on the device; the
// host reads back one short column of the Hessenberg matrix per GMRES
// iteration and a few norms per Newton step to take its decisions.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <string>
#include <vector>

#include "bim_common.h"
#include "precond.h"
#include "vec.h"

namespace bim {

namespace {

// Largest node elevation of the surface and smallest depth zeta - beta on each
// mesh row of the iterate u: zeta at the nodes is zeta_1 plus the trapezoidal
// x-integral of zeta_x (one wave per row, 64-wide scans).
__global__ __launch_bounds__(64) void k_surface_extent_rows(const double *__restrict__ u,
                                                            const double *__restrict__ beta, int N, int M,
                                                            double dx, double *__restrict__ rows) {
    const int j = blockIdx.x, lane = threadIdx.x;
    const double *s = u + (size_t)j * (N + 1);  // [zeta_1, zeta_x(1..N)]
    const double hdx = 0.5 * dx;
    double run = s[0], zmax = -INFINITY, dmin = INFINITY;
    for (int base = 0; base < N; base += 64) {
        const int i = base + lane;
        double inc = (i > 0 && i < N) ? hdx * (s[i] + s[i + 1]) : 0.0;
        for (int d = 1; d < 64; d <<= 1) {
            const double t = __shfl_up(inc, d, 64);
            if (lane >= d) inc += t;
        }
        if (i < N) {
            const double z = run + inc;
            zmax = fmax(zmax, z);
            dmin = fmin(dmin, z - beta[(size_t)j * N + i]);
        }
        run += __shfl(inc, 63, 64);
    }
    for (int d = 32; d > 0; d >>= 1) {
        zmax = fmax(zmax, __shfl_xor(zmax, d, 64));
        dmin = fmin(dmin, __shfl_xor(dmin, d, 64));
    }
    if (lane == 0) {
        rows[j] = zmax;
        rows[M + j] = dmin;
    }
}

__global__ __launch_bounds__(64) void k_surface_extent_reduce(const double *__restrict__ rows, int M,
                                                              double *__restrict__ out) {
    const int lane = threadIdx.x;
    double zmax = -INFINITY, dmin = INFINITY;
    for (int j = lane; j < M; j += 64) {
        zmax = fmax(zmax, rows[j]);
        dmin = fmin(dmin, rows[M + j]);
    }
    for (int d = 32; d > 0; d >>= 1) {
        zmax = fmax(zmax, __shfl_xor(zmax, d, 64));
        dmin = fmin(dmin, __shfl_xor(dmin, d, 64));
    }
    if (lane == 0) {
        out[0] = zmax;
        out[1] = dmin;
    }
}

}  // namespace

int surface_extent_enqueue(const bim_problem *p, const double *u, double *rows, double *out, hipStream_t s) {
    hipLaunchKernelGGL(k_surface_extent_rows, dim3(p->M), dim3(64), 0, s, u, p->beta, p->N, p->M, p->dx, rows);
    hipLaunchKernelGGL(k_surface_extent_reduce, dim3(1), dim3(64), 0, s, rows, p->M, out);
    return hip_check(hipGetLastError(), "surface extent launch");
}

int physical_status(const bim_problem *p, double max_zeta, double min_depth) {
    // Bernoulli on the surface: zeta / F^2 = 1/2 - |grad Phi|^2 / 2 <= 1/2 without surface
    // tension, so no steady surface rises above F^2 / 2; the fluid depth zeta - beta must
    // stay positive
    const bool crest = p->tau == 0.0 && max_zeta > 0.5 * p->froude * p->froude * (1.0 + 1e-12);
    return (crest || !(min_depth > 0.0)) ? BIM_UNPHYSICAL : BIM_OK;
}

namespace {

inline size_t al256(size_t b) { return (b + 255) & ~(size_t)255; }

struct Workspace {
    void *mem = nullptr;
    hipStream_t s = nullptr;
    ~Workspace() {
        if (mem) (void)hipFreeAsync(mem, s);
    }
};

struct Krylov {
    const bim_problem *p;
    Dims d;
    hipStream_t s;
    const Precond *pc;
    int m;                    // restart length
    PairLaunch pl64, pl32;    // launch shape per precision (workspace sized for the larger chunk count)
    ResidualWork rw;
    double *V, *Z, *w, *ut, *Ft, *r, *part, *hdev, *scal, *ydev;
    double *hhost;            // pinned: h column + norm
    long n;
    int jv_evals = 0, res_evals = 0;
    // Jacobian action of the current Newton point
    const double *u = nullptr, *Fin = nullptr;
    int prec = BIM_FP64, linear = 0;
    const double *lin_tab = nullptr;  // FP64 linear products: the mesh's kernel tables
    double eps = 0;

    int jv(const double *z, double *out) {
        int rc;
        // linear: F_lin is affine, F_lin(u + z) - F_lin(u) = J~ z exactly
        if ((rc = shift_axpy_enqueue(u, z, n, linear ? 1.0 : 0.0, eps, part, scal, ut, s))) return rc;
        if ((rc = residual_enqueue(p, ut, Ft, prec, prec == BIM_FP64 ? pl64 : pl32, rw, s, nullptr, linear,
                                   lin_tab)))
            return rc;
        return quotient_enqueue(Ft, Fin, scal + 2, out, n, s);
    }
    int apply_prec(const double *v, double *z) {
        if (pc) return precond_apply_enqueue(pc, v, z, s);
        return hip_check(hipMemcpyAsync(z, v, sizeof(double) * n, hipMemcpyDeviceToDevice, s), "copy");
    }
    int norm_to_host(const double *v, double *out) {
        int rc;
        if ((rc = dot_enqueue(v, v, n, part, scal + 3, true, s))) return rc;
        if ((rc = hip_check(hipMemcpyAsync(hhost, scal + 3, sizeof(double), hipMemcpyDeviceToHost, s), "copy")))
            return rc;
        if ((rc = hip_check(hipStreamSynchronize(s), "sync"))) return rc;
        *out = hhost[0];
        return BIM_OK;
    }

    // Device work of Arnoldi step j: z_j = P^-1 v_j, w = J z_j, two passes of
    // classical Gram-Schmidt against v_0..v_j, v_{j+1} = w / |w|, and the
    // Hessenberg column copied to the host.
    int arnoldi_enqueue(int j) {
        int rc;
        double *vj = V + (size_t)j * n, *zj = Z + (size_t)j * n, *vn = V + (size_t)(j + 1) * n;
        if ((rc = apply_prec(vj, zj))) return rc;
        if ((rc = jv(zj, w))) return rc;
        if (arnoldi_small_applies(n, j + 1))  // (the column goes straight to the pinned host memory)
            return arnoldi_small_enqueue(V, n, j + 1, w, n, hhost, hhost + m + 1, hhost + 2 * (m + 1), vn, s);
        if ((rc = multidot_enqueue(V, n, j + 1, w, n, part, hdev, false, s))) return rc;
        if ((rc = orth_update_enqueue(V, n, j + 1, hdev, w, n, s))) return rc;
        if ((rc = multidot_enqueue(V, n, j + 1, w, n, part, hdev + m + 1, false, s))) return rc;
        if ((rc = orth_update_enqueue(V, n, j + 1, hdev + m + 1, w, n, s))) return rc;
        if ((rc = dot_enqueue(w, w, n, part, hdev + 2 * (m + 1), true, s))) return rc;
        if ((rc = scale_inv_enqueue(w, hdev + 2 * (m + 1), vn, n, s))) return rc;
        return hip_check(hipMemcpyAsync(hhost, hdev, sizeof(double) * (3 * (m + 1)), hipMemcpyDeviceToHost, s),
                         "copy");
    }
    // Arnoldi step j, replayed from a HIP graph (the buffers of step j do not move
    // during a solve); one set of graphs per inner precision, as a solve may
    // switch from FP32C to FP64.  Captured on the step's fourth use: capturing and
    // instantiating a step costs some 85 us, and replaying it saves the host's share of
    // the launches, which the device mostly hides; Newton converges in two to four steps,
    // and graphs from the first use on cost such solves a tenth of their time (31 x
    // 11 4.3 ms with them, 3.8 without; 121 x 41 22.4 / 20.4).
    static constexpr int kGraphUse = 4;
    std::vector<hipGraphExec_t> graph_sets[2];
    std::vector<int> uses[2];
    bool use_graphs = false;
    int arnoldi(int j) {
        ++jv_evals;
        if (!use_graphs) return arnoldi_enqueue(j);
        const int set = prec == BIM_FP64 ? 0 : 1;
        std::vector<hipGraphExec_t> &graphs = graph_sets[set];
        if (graphs.size() < (size_t)m) {
            graphs.assign(m, nullptr);
            uses[set].assign(m, 0);
        }
        if (!graphs[j] && ++uses[set][j] < kGraphUse) return arnoldi_enqueue(j);
        if (!graphs[j]) {
            int rc = hip_check(hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal), "hipStreamBeginCapture");
            if (rc) return rc;
            const int rc_work = arnoldi_enqueue(j);
            hipGraph_t g = nullptr;
            rc = hip_check(hipStreamEndCapture(s, &g), "hipStreamEndCapture");
            if (rc_work) {
                if (g) (void)hipGraphDestroy(g);
                return rc_work;
            }
            if (rc) return rc;
            hipGraphExec_t ex = nullptr;
            rc = hip_check(hipGraphInstantiate(&ex, g, nullptr, nullptr, 0), "hipGraphInstantiate");
            (void)hipGraphDestroy(g);
            if (rc) return rc;
            graphs[j] = ex;
        }
        return hip_check(hipGraphLaunch(graphs[j], s), "hipGraphLaunch");
    }
    ~Krylov() {
        for (auto &graphs : graph_sets)
            for (auto g : graphs)
                if (g) (void)hipGraphExecDestroy(g);
    }

    // Solves J x = b approximately (x zero-initialised here); returns iterations used.
    int gmres(const double *b, double *x, double rtol, int max_restarts, int *iters, double *relres) {
        int rc;
        *iters = 0;
        if ((rc = hip_check(hipMemsetAsync(x, 0, sizeof(double) * n, s), "memset"))) return rc;
        if ((rc = hip_check(hipMemcpyAsync(r, b, sizeof(double) * n, hipMemcpyDeviceToDevice, s), "copy")))
            return rc;
        double beta;
        if ((rc = norm_to_host(r, &beta))) return rc;
        const double beta0 = beta;
        *relres = 1.0;
        if (!(beta0 > 0.0)) {
            *relres = 0.0;
            return std::isfinite(beta0) ? BIM_OK : fail(BIM_EDOMAIN, "non-finite right-hand side");
        }
        std::vector<double> H((size_t)(m + 1) * m), cs(m), sn(m), g(m + 1), y(m);
        for (int cyc = 0; cyc <= max_restarts; ++cyc) {
            // v0 = r / beta
            hhost[0] = beta;
            if ((rc = hip_check(hipMemcpyAsync(scal + 3, hhost, sizeof(double), hipMemcpyHostToDevice, s), "copy")))
                return rc;
            if ((rc = scale_inv_enqueue(r, scal + 3, V, n, s))) return rc;
            std::fill(g.begin(), g.end(), 0.0);
            g[0] = beta;
            int jend = 0;
            bool done = false;
            for (int j = 0; j < m; ++j) {
                if ((rc = arnoldi(j))) return rc;
                if ((rc = hip_check(hipStreamSynchronize(s), "sync"))) return rc;
                ++*iters;
                double *col = &H[(size_t)j];  // column j: H[i * m + j]
                for (int i = 0; i <= j; ++i) col[(size_t)i * m] = hhost[i] + hhost[m + 1 + i];
                const double hn = hhost[2 * (m + 1)];
                col[(size_t)(j + 1) * m] = hn;
                if (!std::isfinite(hn)) return fail(BIM_EDOMAIN, "non-finite Krylov vector");
                for (int i = 0; i < j; ++i) {  // previous rotations
                    const double a = col[(size_t)i * m], bb = col[(size_t)(i + 1) * m];
                    col[(size_t)i * m] = cs[i] * a + sn[i] * bb;
                    col[(size_t)(i + 1) * m] = -sn[i] * a + cs[i] * bb;
                }
                const double a = col[(size_t)j * m], bb = col[(size_t)(j + 1) * m];
                const double rr = std::hypot(a, bb);
                cs[j] = rr > 0 ? a / rr : 1.0;
                sn[j] = rr > 0 ? bb / rr : 0.0;
                col[(size_t)j * m] = rr;
                col[(size_t)(j + 1) * m] = 0.0;
                g[j + 1] = -sn[j] * g[j];
                g[j] = cs[j] * g[j];
                jend = j + 1;
                *relres = std::fabs(g[j + 1]) / beta0;
                if (*relres <= rtol || hn == 0.0) {
                    done = true;
                    break;
                }
            }
            // y = H^-1 g (upper triangular), x += Z y
            for (int i = jend - 1; i >= 0; --i) {
                double v = g[i];
                for (int k = i + 1; k < jend; ++k) v -= H[(size_t)i * m + k] * y[k];
                y[i] = v / H[(size_t)i * m + i];
            }
            if ((rc = hip_check(hipMemcpyAsync(ydev, y.data(), sizeof(double) * jend, hipMemcpyHostToDevice, s),
                                "copy")))
                return rc;
            if ((rc = combine_enqueue(Z, n, jend, ydev, x, n, s))) return rc;
            if ((rc = hip_check(hipStreamSynchronize(s), "sync"))) return rc;  // y host buffer reuse
            if (done || cyc == max_restarts) break;
            // true residual r = b - J x
            if ((rc = jv(x, w))) return rc;
            ++jv_evals;
            if ((rc = axpby_enqueue(1.0, b, -1.0, w, r, n, s))) return rc;
            if ((rc = norm_to_host(r, &beta))) return rc;
            *relres = beta / beta0;
            if (*relres <= rtol) break;
        }
        return BIM_OK;
    }
};

// Private non-blocking stream for a solve (HIP graphs cannot be captured on the
// null stream): ordered after the caller's stream on entry, and the caller's
// stream is ordered after it on exit.
struct SolveStream {
    hipStream_t caller = nullptr, own = nullptr;
    hipEvent_t ev = nullptr;
    int open(hipStream_t c) {
        caller = c;
        int rc = hip_check(hipStreamCreateWithFlags(&own, hipStreamNonBlocking), "hipStreamCreate");
        if (rc) return rc;
        if ((rc = hip_check(hipEventCreateWithFlags(&ev, hipEventDisableTiming), "hipEventCreate"))) return rc;
        if ((rc = hip_check(hipEventRecord(ev, caller), "hipEventRecord"))) return rc;
        return hip_check(hipStreamWaitEvent(own, ev, 0), "hipStreamWaitEvent");
    }
    ~SolveStream() {
        if (own) {
            if (ev && hipEventRecord(ev, own) == hipSuccess) (void)hipStreamWaitEvent(caller, ev, 0);
            (void)hipStreamSynchronize(own);
            (void)hipStreamDestroy(own);
        }
        if (ev) (void)hipEventDestroy(ev);
    }
};

int solve_impl(const bim_problem *p, const bim_precond *P, double *u_io, const bim_jfnk_opts *o,
               bim_jfnk_report *rep, hipStream_t caller, bool linear_start_only) {
    auto t0 = std::chrono::steady_clock::now();
    SolveStream ss;
    if (int rc0 = ss.open(caller)) return rc0;
    hipStream_t s = ss.own;
    const Dims d(p);
    const long n = d.nvec;
    const int m = std::max(1, o->restart);
    Krylov K{p, d, s};
    K.n = n;
    K.m = m;
    // one workspace sized for the larger chunk count of the two precisions
    const bool lin_conv = linear_start_only && o->inner_prec == BIM_FP64 && lin_conv_applies(d, true);
    const PairLaunch pl64 = o->inner_prec == BIM_FP64 ? pair_launch_for(p, BIM_FP64) : pair_launch_batch(p, BIM_FP64);
    const PairLaunch pl32 = pair_launch_for(p, BIM_FP32C);
    PairLaunch plw = pl64.chunks >= pl32.chunks ? pl64 : pl32;
    size_t bytes = residual_work_bytes(d, plw);
    const size_t vb = al256(sizeof(double) * n);
    bytes += vb * ((size_t)(m + 1) + m + 8);                        // V, Z, w, ut, Ft, r, x, F, Fin, delta
    bytes += al256(sizeof(double) * (size_t)reduce_parts() * (m + 1));  // part
    bytes += al256(sizeof(double) * 3 * (m + 1)) + al256(sizeof(double) * 8) + al256(sizeof(double) * (m + 1));
    if (lin_conv) bytes += lin_table_bytes(d);
    Workspace ws;
    ws.s = s;
    int rc = hip_check(hipMallocAsync(&ws.mem, bytes, s), "hipMallocAsync(jfnk)");
    if (rc) return rc;
    double *hhost = nullptr;
    rc = hip_check(hipHostMalloc((void **)&hhost, sizeof(double) * 3 * (m + 2)), "hipHostMalloc");
    if (rc) return rc;
    struct HostFree {
        double *p;
        ~HostFree() {
            if (p) (void)hipHostFree(p);
        }
    } hf{hhost};
    residual_work_carve(ws.mem, d, plw, &K.rw);
    char *c = (char *)ws.mem + K.rw.bytes;
    auto take = [&](size_t b) {
        char *q = c;
        c += al256(b);
        return (double *)q;
    };
    K.V = take(sizeof(double) * n * (m + 1));
    K.Z = take(sizeof(double) * n * m);
    K.w = take(sizeof(double) * n);
    K.ut = take(sizeof(double) * n);
    K.Ft = take(sizeof(double) * n);
    K.r = take(sizeof(double) * n);
    double *F = take(sizeof(double) * n);
    double *Fin = take(sizeof(double) * n);
    double *delta = take(sizeof(double) * n);
    double *rhs = take(sizeof(double) * n);
    K.part = take(sizeof(double) * (size_t)reduce_parts() * (m + 1));
    K.hdev = take(sizeof(double) * 3 * (m + 1));
    K.scal = take(sizeof(double) * 8);
    K.ydev = take(sizeof(double) * (m + 1));
    K.hhost = hhost;
    K.pl64 = pl64;
    K.pl32 = pl32;
    K.use_graphs = o->use_graphs != 0;

    // preconditioner: caller's, or built here
    bim_precond *own = nullptr;
    double precond_ms = 0.0;
    if (!P && o->use_precond) {
        auto tp = std::chrono::steady_clock::now();
        if ((rc = precond_setup_ex(p, o->band_halfwidth, o->precond_storage, &own, s))) return rc;
        precond_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - tp).count();
        P = own;
    }
    struct OwnFree {
        bim_precond *p;
        ~OwnFree() {
            if (p) precond_destroy(p);
        }
    } of{own};
    K.pc = o->use_precond ? precond_impl(P) : nullptr;

    bim_jfnk_report R{};
    R.precond_ms = precond_ms;
    auto finish = [&](int status) {
        if (!linear_start_only && status >= BIM_OK && (size_t)2 * d.M <= (size_t)reduce_parts() * (m + 1)) {
            // the extent of the last iterate (the caller's u)
            if (surface_extent_enqueue(p, u_io, K.part, K.scal + 6, s) == BIM_OK &&
                hip_check(hipMemcpyAsync(hhost, K.scal + 6, sizeof(double) * 2, hipMemcpyDeviceToHost, s),
                          "copy") == BIM_OK &&
                hip_check(hipStreamSynchronize(s), "sync") == BIM_OK) {
                R.max_zeta = hhost[0];
                R.min_depth = hhost[1];
                if (physical_status(p, R.max_zeta, R.min_depth) != BIM_OK) {
                    status = fail(BIM_UNPHYSICAL, "the iterate rises above the limiting height F^2/2 or "
                                                  "reaches the bottom");
                }
            }
        }
        R.status = status;
        R.jv_evals = K.jv_evals;
        R.time_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
        if (rep) *rep = R;
        return status;
    };

    if (linear_start_only) {
        // u_lin = u0 - J~^-1 F_lin(u0): one linear solve with the exact linear operator
        if ((rc = uniform_stream_enqueue(u_io, d.N, d.M, p->x1, s))) return rc;
        // (with inner_prec BIM_FP32C the operator's products use FP32C sums, the
        // base point included, and the right-hand side stays FP64, summed pair by
        // pair as they are; FP64 products are convolutions with the mesh's tables)
        if (lin_conv) {
            double *tab = take(lin_table_bytes(d));
            if ((rc = kernel_tables_enqueue(tab, d.N, d.M, p->dx, p->dy, s))) return rc;
            K.lin_tab = tab;
        }
        if ((rc = residual_enqueue(p, u_io, F, BIM_FP64, pl64, K.rw, s, nullptr, 1, K.lin_tab))) return rc;
        if ((rc = axpby_enqueue(-1.0, F, 0.0, nullptr, rhs, n, s))) return rc;
        K.u = u_io;
        K.Fin = F;
        if (o->inner_prec == BIM_FP32C) {
            if ((rc = residual_enqueue(p, u_io, Fin, BIM_FP32C, pl32, K.rw, s, nullptr, 1))) return rc;
            K.Fin = Fin;
        }
        K.prec = o->inner_prec;
        K.linear = 1;
        K.eps = std::ldexp(1.0, -52);
        int it = 0;
        double rr = 1.0;
        if ((rc = K.gmres(rhs, delta, o->gmres_rtol, o->max_restarts, &it, &rr))) return rc;
        if ((rc = axpby_enqueue(1.0, u_io, 1.0, delta, u_io, n, s))) return rc;
        if ((rc = hip_check(hipStreamSynchronize(s), "sync"))) return rc;
        R.gmres_iters = it;
        R.gmres_relres_last = rr;
        return finish(rr <= o->gmres_rtol * 10 ? BIM_OK : BIM_NOT_CONVERGED);
    }

    auto norms = [&](const double *v, double *n2, double *ninf) -> int {
        int q;
        if ((q = dot_enqueue(v, v, n, K.part, K.scal + 4, true, s))) return q;
        if ((q = maxabs_enqueue(v, n, K.part, K.scal + 5, s))) return q;
        if ((q = hip_check(hipMemcpyAsync(hhost, K.scal + 4, sizeof(double) * 2, hipMemcpyDeviceToHost, s), "copy")))
            return q;
        if ((q = hip_check(hipStreamSynchronize(s), "sync"))) return q;
        *n2 = hhost[0];
        *ninf = hhost[1];
        return BIM_OK;
    };

    if ((rc = residual_enqueue(p, u_io, F, BIM_FP64, pl64, K.rw, s))) return rc;
    R.residual_evals = 1;
    double fn2, finf;
    if ((rc = norms(F, &fn2, &finf))) return rc;
    R.fnorm0_inf = finf;
    const int maxh = (int)(sizeof(R.history) / sizeof(R.history[0]));
    for (int k = 0;; ++k) {
        if (k < maxh) R.history[k] = finf;
        R.fnorm_inf = finf;
        R.newton_iters = k;
        if (!std::isfinite(fn2)) return finish(fail(BIM_EDOMAIN, "non-finite residual"));
        if (finf <= o->ftol) return finish(BIM_OK);
        if (k >= o->max_newton) return finish(BIM_NOT_CONVERGED);
        if (o->stall_steps > 0 && k >= o->stall_steps && k < maxh && finf > 0.5 * R.history[k - o->stall_steps])
            return finish(BIM_NOT_CONVERGED);
        // inner Jacobian action around u in the requested precision (FP64 once
        // ||F||_inf <= fp64_below when so asked)
        const int prec = (o->inner_prec == BIM_FP32C && !(finf <= o->fp64_below)) ? BIM_FP32C : BIM_FP64;
        K.u = u_io;
        K.prec = prec;
        K.linear = 0;
        K.eps = (o->fd_eps > 0) ? o->fd_eps : (prec == BIM_FP64) ? std::ldexp(1.0, -52) : std::ldexp(1.0, -23);
        if (prec == BIM_FP64) {
            K.Fin = F;
        } else {
            if ((rc = residual_enqueue(p, u_io, Fin, prec, pl32, K.rw, s))) return rc;
            ++R.inner_residual_evals;
            K.Fin = Fin;
        }
        if ((rc = axpby_enqueue(-1.0, F, 0.0, nullptr, rhs, n, s))) return rc;
        int it = 0;
        double rr = 1.0;
        const double rtol = (prec == BIM_FP32C) ? std::max(o->gmres_rtol, o->fp32c_gmres_rtol) : o->gmres_rtol;
        if ((rc = K.gmres(rhs, delta, rtol, o->max_restarts, &it, &rr))) return rc;
        R.gmres_iters += it;
        R.gmres_relres_last = rr;
        // backtracking line search on ||F||_2 (sufficient decrease)
        double mu = 1.0;
        bool ok = false;
        for (int bt = 0; bt <= o->max_backtracks; ++bt) {
            if ((rc = axpby_enqueue(1.0, u_io, mu, delta, K.ut, n, s))) return rc;
            if ((rc = residual_enqueue(p, K.ut, K.Ft, BIM_FP64, pl64, K.rw, s))) return rc;
            ++R.residual_evals;
            double tn2, tinf;
            if ((rc = norms(K.Ft, &tn2, &tinf))) return rc;
            if (std::isfinite(tn2) && tn2 <= (1.0 - 1e-4 * mu) * fn2) {
                ok = true;
                fn2 = tn2;
                finf = tinf;
                break;
            }
            ++R.backtracks;
            mu *= 0.5;
        }
        if (!ok) return finish(BIM_LINESEARCH_FAIL);
        if ((rc = hip_check(hipMemcpyAsync(u_io, K.ut, sizeof(double) * n, hipMemcpyDeviceToDevice, s), "copy")))
            return rc;
        if ((rc = hip_check(hipMemcpyAsync(F, K.Ft, sizeof(double) * n, hipMemcpyDeviceToDevice, s), "copy")))
            return rc;
    }
}

}  // namespace

}  // namespace bim

using namespace bim;

extern "C" {

void jfnk_default_opts(bim_jfnk_opts *o) {
    if (!o) return;
    o->ftol = 1e-10;
    o->gmres_rtol = 1e-8;
    o->restart = 30;
    o->max_restarts = 10;
    o->max_newton = 30;
    o->max_backtracks = 20;
    o->inner_prec = BIM_FP64;
    o->band_halfwidth = -1;
    o->use_precond = 1;
    o->use_graphs = 1;
    o->fd_eps = 0.0;
    o->stall_steps = 0;
    o->fp64_below = 0.0;
    // an inexact-Newton forcing term for the FP32C steps: their Jacobian action
    // resolves ~1e-6 relative, and Newton from it contracts ||F|| by ~1e-2 per
    // step whatever the inner tolerance below that, so GMRES solves to 1e-2
    // (measured at 181 x 61, F = 0.6 ... 1.8: the same or fewer Newton steps as
    // at 1e-4 and 1e-8, the fewest GMRES iterations among 1e-4 ... 1e-1 but at
    // F = 0.9)
    o->fp32c_gmres_rtol = 1e-2;
    o->precond_storage = BIM_STORE_FP64;
}

static int check_opts(const bim_jfnk_opts *o) {
    if (!o) return fail(BIM_EINVAL, "options are NULL");
    if (!(o->ftol > 0) || !(o->gmres_rtol > 0) || o->restart < 1 || o->restart > 200 || o->max_restarts < 0 ||
        o->max_newton < 0 || o->max_backtracks < 0 || !(o->fd_eps < 1.0) || o->stall_steps < 0 ||
        !(o->fp64_below >= 0.0))
        return fail(BIM_EINVAL, "invalid solver options");
    if (o->inner_prec != BIM_FP64 && o->inner_prec != BIM_FP32C) return fail(BIM_EINVAL, "unknown precision");
    if (o->precond_storage != BIM_STORE_FP64 && o->precond_storage != BIM_STORE_FP32)
        return fail(BIM_EINVAL, "unknown preconditioner storage");
    return BIM_OK;
}

int jfnk_solve(const bim_problem *prob, const bim_precond *P, double *u, const bim_jfnk_opts *opts,
               bim_jfnk_report *rep, void *stream) {
    int rc = validate(prob);
    if (rc) return rc;
    bim_jfnk_opts o;
    jfnk_default_opts(&o);
    if (opts) o = *opts;
    if ((rc = check_opts(&o))) return rc;
    if (!u) return fail(BIM_EINVAL, "u must be a device pointer");
    return solve_impl(prob, P, u, &o, rep, (hipStream_t)stream, false);
}

int bim_linear_start(const bim_problem *prob, const bim_precond *P, double *u_out, double rtol, void *stream) {
    return bim_linear_start_ex(prob, P, u_out, rtol, BIM_FP64, stream);
}

int bim_linear_start_ex(const bim_problem *prob, const bim_precond *P, double *u_out, double rtol, int prec,
                        void *stream) {
    int rc = validate(prob);
    if (rc) return rc;
    if (!u_out) return fail(BIM_EINVAL, "u_out must be a device pointer");
    if (prec != BIM_FP64 && prec != BIM_FP32C) return fail(BIM_EINVAL, "unknown precision");
    bim_jfnk_opts o;
    jfnk_default_opts(&o);
    o.inner_prec = prec;
    o.gmres_rtol = rtol > 0 ? rtol : 1e-12;
    o.max_restarts = 20;
    bim_jfnk_report r{};
    return solve_impl(prob, P, u_out, &o, &r, (hipStream_t)stream, true);
}

}  // extern "C"
