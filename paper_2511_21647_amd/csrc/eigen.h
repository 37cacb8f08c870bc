// Arguments of the cooperative FP64 Hermitian eigensolvers (eigen.hip; eigen_lds.hip
// for the split-precision form), shared by the clutter filter's driver (svd.hip).
#pragma once

#include "common.h"

namespace ulm {

constexpr int kCoopMaxW = 32;      // work-groups per plane (one barrier flag each)
constexpr int kPlaceWord = kBarStride - 1;  // per-plane word: bit x set by a work-group on XCC x

// Below this |x|^2 a column's rest is zero.  A covariance of FP32 values that is not zero
// has a norm of at least 2e-90, so 1e-135 is far below its rounding; but a covariance of low
// rank (identical frames) leaves a rest that shrinks by 1e-15 a step, and the reciprocals of
// a reflector's squares overflow where it passes 1e-154.
constexpr double kNoReflector = 0x1p-900;

// Inverse iteration for equal eigenvalues (the zeros of a covariance of low rank, frames that
// repeat).  In decoupled parts of T it returns the start vector's share of each part, or only
// that of the part whose eigenvalue is nearest by rounding, and the start vectors are of three
// dimensions: the vectors come out dependent.  So where an eigenvalue equals the one before
// it within its bracket, the start vector has an independent part, and the shift stands off by
// more than the parts differ by.
__device__ inline bool equal_eigenvalues(double a, double b, double tnorm) {
    return fabs(a - b) <= 0x1p-49 * tnorm;
}
__device__ inline double independent_entry(int q, int i) {       // in [-1, 1]
    unsigned h = (unsigned)q * 0x9e3779b9u + (unsigned)(i + 1) * 0x85ebca6bu;
    h = (h ^ (h >> 16)) * 0x7feb352du;
    h = (h ^ (h >> 15)) * 0x846ca68bu;
    return (double)(int)(h ^ (h >> 16)) * 0x1p-31;
}
__device__ inline double start_entry(int q, int i, bool equal) {
    const double x = 1.0 + 0.37 * sin(0.731 * q + 1.3 * i);
    return equal ? x + independent_entry(q, i) : x;
}
__device__ inline double iteration_shift(double lam, double tnorm, bool equal) {
    if (tnorm == 0.0) return 0.0;        // T = 0, whose eigenvalues are the bisection's margin
    return equal ? lam - 0x1p-44 * tnorm : lam;
}
// What stands for a pivot of zero (T = 0 takes any).
__device__ inline double least_pivot(double tnorm, double pivmin) {
    return tnorm > 0.0 ? 0x1p-52 * tnorm + pivmin : 1.0;
}

struct EigArgs {
    const double2 *C;   // [planes][F][F] covariance (full Hermitian)
    double2 *H;         // [planes][F][F] row k: Householder vector v_k (entries k+1..F-1)
    double2 *tau;       // [planes][F]
    double *d, *e;      // [planes][F]
    double *lam;        // [planes][F] eigenvalues, descending
    double *lam_out;    // optional copy of lam
    double2 *V;         // [planes][F][c] clutter eigenvectors
    double *tscr;       // [planes][c][6][F]
    double2 *xscr;      // [planes][c][F]
    double2 *xbuf;      // [planes][2][3][F] published p = tau A v, then columns, by step modulo 3
                        // (eigen_lds.hip: p, [planes][2][F] by step modulo 2)
    double2 *colbuf;    // eigen_lds.hip: published columns, [planes][2][F] (behind p in the same
                        // buffer; strided by plane as above, 480 frames took 1.4% longer)
    int *bar;           // [planes][kBarStride] barrier flags and the XCC mask, zero at launch
    int *flag;          // [planes] non-finite input
    int *status;
    int F, c, W;
    int agent_scope;    // nonzero: the fenced mode even when a plane is on one XCD
    int planes;         // solve planes [plane0, planes)
    int plane0;
};

size_t eigen_coop_lds(int F, int c);
hipError_t launch_eigen_coop(const EigArgs &args, hipStream_t st);
int eigen_lds_width(int F);
size_t eigen_lds_bytes(int F, int c);
hipError_t launch_eigen_lds(const EigArgs &args, hipStream_t st);
hipError_t launch_eigen_clear(int *status, int *bar, int *eflag, double2 *xbuf, int planes, int F,
                              hipStream_t st);

}  // namespace ulm
