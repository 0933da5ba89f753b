// Index maps and weights of the convolution form of the M2L (the algebra is at
// the head of k_conv.hip), shared by its kernels and by host code.
#pragma once
#include "fmm_internal.h"

namespace fmm {

// real vectors of one axis at wave number k
__host__ __device__ inline int nvec(int k, int N) { return k == 0 || 2 * k == N ? 1 : 2; }

// Slot f of one axis for a coefficient whose sign the axis' reflection flips
// or not: wave number, tau, real vector rho, and whether the entry is negated.
struct Axis {
    int k, tau, rho, neg;
};
__host__ __device__ inline Axis axis_of(int f, int n, int flip) {
    const int N = n / 2;
    if (f == 0) return {0, 0, 0, 0};
    if (f == n - 1) return {0, 1, 0, flip};
    const int q = (f + 1) / 2, cosine = f & 1;
    if (2 * q == N) return {q, cosine == !flip ? 0 : 1, 0, flip};
    const int low = 2 * q < N;
    const int rho = ((cosine == low) == !flip) ? 0 : 1;
    return {low ? q : N - q, !low, rho, flip && rho == 0};
}

// Entry (x, y, z slots; coefficient c16 of chunk cc given by its table row t)
// in the column arrays: per triple of wave numbers, chunk, tau, column, 16
// coefficients.  The sign bit is that of a multipole or a local.
struct Entry {
    uint32_t at;
    int neg;
};
__host__ __device__ inline Entry entry_of(Axis ax, Axis ay, Axis az, int pos, const ConvCoef &t, bool local, int N, int NB,
                                 const int32_t *__restrict__ pair) {
    int neg = ax.neg ^ ay.neg ^ az.neg, sw = 0;
    if (ax.k < ay.k) {
        const Axis b = ax;
        ax = ay;
        ay = b;
        pos = t.mir;
        neg ^= local ? t.lneg : t.mneg;
        sw = 1;
    }
    const int rx = nvec(ax.k, N), ry = nvec(ay.k, N), rz = nvec(az.k, N);
    const int rxy = rx * ry * (ax.k != ay.k ? 2 : 1);
    const uint32_t col0 = (uint32_t)pair[ax.k * (ax.k + 1) / 2 + ay.k] + rxy * (az.k == 0 ? 0 : 2 * az.k - 1);
    const int ncol = rxy * rz;
    const int col = ((sw * rx + ax.rho) * ry + ay.rho) * rz + az.rho;
    const int tau = ax.tau * 4 + ay.tau * 2 + az.tau;
    return {(col0 * NB + (pos >> 4) * ncol) * 128u + (uint32_t)(tau * ncol + col) * 16u + (pos & 15), neg};
}

// Weight w_0 of offset d at wave number k for a row and a column whose signs the
// axis' reflection flips (1) or not; w_1 is w_0 with odd d negated.  trig: cos
// then sin of pi j / N, j < 2N.
__host__ __device__ inline double conv_weight(int fr, int fc, int d, int k, int N, const double *trig) {
    const double f = d == 0 || d == 5 ? 1.0 : 2.0;
    const int at = d * k % (2 * N);
    return fr == fc ? f * trig[at] : f * (fc ? -1.0 : 1.0) * trig[2 * N + at];
}
// w_2 of d = 5
__host__ __device__ inline double conv_cross(int fr, int fc, int k, int N, const double *trig) {
    const int at = 5 * k % (2 * N);
    return fr == fc ? trig[2 * N + at] : (fc ? 1.0 : -1.0) * trig[at];
}

}  // namespace fmm
