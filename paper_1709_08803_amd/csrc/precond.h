// Block-banded preconditioner (internal).
#pragma once

#include <hip/hip_runtime.h>

#include "bim_common.h"

namespace bim {

// The nine arrays the apply reads, in one element type.  S^-1 is kept as
// V^-1 D^-1 L^-1 (S = L D V: L, V unit block-triangular, D the pivot blocks):
// Sinv holds L^-1 below the block diagonal and V^-1 above it (identity blocks
// on it), Uinv the inverse pivot blocks D^-1.
template <typename T>
struct PrecondArrays {
    T *Dinv11, *Dinv22, *E;  // band-0 arrays [M][s][s] (same block on every slice)
    T *B21, *B23, *B31, *G;  // band-h arrays [M][2h+1][s][s]
    T *Sinv;                 // dense [n][n]: L^-1 | I | V^-1 by slice blocks
    T *Uinv;                 // band-0 array [M][s][s]: D^-1
};

// One apply of an FP64-stored preconditioner on its own: sizes, the arrays it
// reads beside the Schur inverse, its scratch, and the vectors (papply.hip).
struct PcDesc {
    int N, M, s, h, half, chunks;  // chunks: source chunks of the banded convolutions
    long n;
    double dx, dy;
    const double *iD11;   // [s][s]      P11^-1 (one slice block)
    const double *iD22;   // [s][s]      P22^-1
    const double *ETs;    // [s + N][s]  E = P11^-1 P12 and the node-value map T
    const double *tab;    // [3][2M - 1][N - 1] kernels K5, K6, K7 by mesh offset
    const double *corr;   // [M][N - 1]  singular subtraction of the K5 sums, halved
    double *a1, *a3, *t2;  // [n] each
    double *q1, *q2;       // [M N] weighted sources of the convolutions (and spare entries read past the end)
    double *p1, *p2;       // [chunks][M][N - 1] their partial sums
    const double *r;
    double *z;
};
constexpr int kPcSourcePad = 64;  // spare entries of q1 and q2

struct Precond {
    int N, M, s, h;
    long n;
    int storage = BIM_STORE_FP64;  // element type of the stored operator
    void *mem = nullptr;           // one device allocation holding the arrays and the scratch
    size_t bytes = 0;
    // FP64 arrays (built first; kept when storage is FP64, else released)
    double *Dinv11, *Dinv22, *E;
    double *B21, *B23, *B31, *G;
    double *Sinv, *Uinv;
    PrecondArrays<float> f32{};   // FP32 copies when storage is FP32
    double *scratch;              // [4 n] apply temporaries
    bool tables = false;          // the single-problem apply convolves with kernel tables
    PcDesc d{};                   // its arrays (r and z set per apply)
    int groups = 1;               // its triangular products: groups of slices (group_start),
    double *bnd = nullptr;        // [groups - 1][(2h + 1) s][(2h + 1) s] factor blocks between them
    long group_start(int k) const { return (long)k * M / groups; }
};

int precond_build(const bim_problem *p, int hb, int storage, Precond **out, hipStream_t st);
int precond_apply_enqueue(const Precond *pc, const double *r, double *z, hipStream_t st);
void precond_free(Precond *pc);
// The array `which` (0..8: Dinv11, Dinv22, E, B21, B23, B31, G, Sinv, Uinv) as stored
// (FP64 or FP32 per pc->storage).
const void *precond_array(const Precond *pc, int which);

// Stages of the apply around the Schur inverse: from r to t2, and from
// z2 = S^-1 t2 (in z) to the rest of z.
int pc_before_schur(const PcDesc &d, hipStream_t st);
int pc_after_schur(const PcDesc &d, hipStream_t st);
int pc_conv_chunks(int N, int M, int h);
// tab[3][2M - 1][N - 1]: K5 = 1/r, K6 = (r^2 + 1)^(-3/2), K7 = (r^2 + 1)^(-1/2) at the
// mesh offsets ((e + 1/2) dx, o dy).
int kernel_tables_enqueue(double *tab, int N, int M, double dx, double dy, hipStream_t st);
// Setup: the halved K5 correction; [A; T].
int pc_corr_enqueue(const double *rowsum, const double *I5, double *corr, int N, int M, hipStream_t st);
int pc_stack_enqueue(const double *A, double *out, int N, double dx, hipStream_t st);

}  // namespace bim

struct bim_precond;
namespace bim {
Precond *precond_impl(const bim_precond *P);
}  // namespace bim
