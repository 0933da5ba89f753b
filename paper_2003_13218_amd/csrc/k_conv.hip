// Stage a6 (M2L, eq. Lcoeffdef) of a whole level as a convolution over the
// periodic grid of cells, products in wave-number space.
//
// A level has n cells and N = n / 2 parents per axis; cell c = 2P + i.  The
// list of a target holds d = 2(P' - P) + (j - i), |P' - P| <= 2, |d| > 2 in some
// axis, so  L_c = sum_d O_d M_{c+d}  couples parents only by their difference:
// a Fourier transform over the parents leaves one 8K x 8K product per wave
// number (8 children), instead of 875 K x K products per cell: 16 K^2 operations
// per cell against 1750 K^2 (or 610 K^2 with the list folded by reflections).
// What reflections do to the operators (O_{sd} = D_s O_d D_s, D_s = +-1 per
// coefficient) makes everything real and removes most of the 8K x 8K matrix:
//
// * Per axis, with phi = pi k / N, k = 0 .. N/2, take the sum (tau = 0) and the
//   difference (tau = 1) of the two children and the real cell transforms
//     C_q = sum_c cos(2 pi q c / n) x_c,   S_q = sum_c sin(2 pi q c / n) x_c.
//   The pair (k, N - k) of frequencies forms one or two real vectors rho over
//   (tau, coefficient); a coefficient that the axis' reflection leaves alone
//   (D = +) and one whose sign it flips (D = -) take
//     rho 0:  tau 0: D+ C_k, D- -S_k;   tau 1: D+ S_{N-k}, D- -C_{N-k}
//     rho 1:  tau 0: D+ S_k, D-  C_k;   tau 1: D+ C_{N-k}, D-  S_{N-k}
//   (k = 0: one vector, tau 0: C_0, tau 1: D+ C_N, D- -C_N;  k = N/2: rho 0).
// * On them the level is a real matrix, the same for every rho.  Its K x K
//   blocks depend, per axis, on the type: 0 (tau 0 to 0), 1 (1 to 1), 2 (0 to 1
//   and 1 to 0, the same block), so 27 blocks per triple of wave numbers:
//     G[r][c] = sum_{d in [0,5]^3} O_d[r][c] prod_axes w_type(d)
//     w_0 = a_d t(d phi),  w_1 = (-1)^d w_0,  a_d = 1 (d = 0, 5) or 2,
//     w_2 = t(5 phi - pi/2) for d = 5, 0 otherwise,
//     t = cos where D_r = D_c, D_c sin where not.
//   (|d| = 5 is in the list of one of the two children only: the other types of
//   block would vanish without it.)
// * The mirror x <-> y is a signed permutation of the coefficients, so (ky, kx,
//   kz) takes the blocks of (kx, ky, kz): up to 16 real vectors (columns) share
//   the 27 blocks, one column block of the matrix cores.
//
// What bounds it: the blocks, read once per evaluation (1M-atom box, level 5,
// p = 12: 405 triples x 27 x 176^2, 1.36 GB in FP32), and the matrix cores (64
// block products per triple on 16 columns).  The transforms are dense n x n per
// line, folded by the symmetries of the cosines to n^2 / 4 multiply-adds, in FP64.
// FP32 levels hold the multipoles and the blocks in FP32; everything after them
// (transforms, columns, products, locals) is FP64 in every mode.
#include "conv_map.h"
#include "fmm_internal.h"
#include "mfma.h"
#include "morton.h"

namespace fmm {

namespace {

// cos(2 pi j / 64), the table of all line transforms (n divides 64): a
// rational-free constexpr series, |error| below one unit in the last place
constexpr double cos_series(double x) {  // |x| <= pi / 4
    double t = 1.0, s = 1.0;
    for (int i = 1; i <= 11; ++i) {
        t *= -x * x / (double)((2 * i - 1) * (2 * i));
        s += t;
    }
    return s;
}
constexpr double sin_series(double x) {
    double t = x, s = x;
    for (int i = 1; i <= 11; ++i) {
        t *= -x * x / (double)((2 * i) * (2 * i + 1));
        s += t;
    }
    return s;
}
constexpr double kPi = 3.14159265358979323846;
constexpr double cos64(int j) {  // cos(2 pi j / 64)
    j = ((j % 64) + 64) % 64;
    if (j > 32) j = 64 - j;             // [0, pi]
    const bool neg = j > 16;
    if (neg) j = 32 - j;                // [0, pi/2]
    const double v = j <= 8 ? cos_series(j * kPi / 32) : sin_series((16 - j) * kPi / 32);
    return neg ? -v : v;
}
struct CosTable {
    double v[64];
};
constexpr CosTable make_cos() {
    CosTable t{};
    for (int j = 0; j < 64; ++j) t.v[j] = cos64(j);
    return t;
}
__device__ constexpr CosTable kCos = make_cos();

constexpr double root(double x) {  // square root by Newton's iteration
    double r = 1.0;
    for (int i = 0; i < 60; ++i) r = 0.5 * (r + x / r);
    return r;
}

template <int n> __device__ inline constexpr double cosn(int j) { return kCos.v[(j * (64 / n)) & 63]; }
template <int n> __device__ inline constexpr double sinn(int j) { return kCos.v[(j * (64 / n) + 48) & 63]; }

// Orthonormal real transform of one line of n values.  Slot 0: C_0, slot
// 2q - 1: C_q, slot 2q: S_q (0 < q < N), slot n - 1: C_N.
template <int n> struct Line {
    static constexpr int N = n / 2, H = n / 4;
    static constexpr double kEnd = 1.0 / root(n), kMid = root(2.0 / n);
    // v -> out[slot]; folded about c = N, then about c = N / 2
    __device__ static inline void forward(double (&v)[n], double (&out)[n]) {
        if constexpr (n == 2) {
            out[0] = (v[0] + v[1]) * kEnd;
            out[1] = (v[0] - v[1]) * kEnd;
        } else {
            double e[H + 1], o[H], g[H + 1], h[H];
            // s_c = v_c + v_{n-c}, d_c = v_c - v_{n-c}
            auto s = [&](int c) { return c == 0 || c == N ? v[c] : v[c] + v[n - c]; };
            auto d = [&](int c) { return v[c] - v[n - c]; };
#pragma unroll
            for (int c = 0; c < H; ++c) {
                e[c] = s(c) + s(N - c);
                o[c] = s(c) - s(N - c);
                if (c > 0) {
                    g[c] = d(c) + d(N - c);
                    h[c] = d(c) - d(N - c);
                }
            }
            e[H] = s(H);
            g[H] = d(H);
#pragma unroll
            for (int q = 0; q <= N; ++q) {
                double a = q % 2 == 0 ? e[0] : o[0];
#pragma unroll
                for (int c = 1; c < H; ++c) a = fma(cosn<n>(q * c), q % 2 == 0 ? e[c] : o[c], a);
                if (q % 2 == 0) a += q % 4 == 0 ? e[H] : -e[H];
                out[q == 0 ? 0 : q == N ? n - 1 : 2 * q - 1] = a * (q == 0 || q == N ? kEnd : kMid);
                if (q > 0 && q < N) {
                    double b = q % 2 == 1 ? (q % 4 == 1 ? g[H] : -g[H]) : 0.0;
#pragma unroll
                    for (int c = 1; c < H; ++c) b = fma(sinn<n>(q * c), q % 2 == 1 ? g[c] : h[c], b);
                    out[2 * q] = b * kMid;
                }
            }
        }
    }
    // the transpose: slots x -> v
    __device__ static inline void inverse(double (&x)[n], double (&v)[n]) {
        if constexpr (n == 2) {
            v[0] = (x[0] + x[1]) * kEnd;
            v[1] = (x[0] - x[1]) * kEnd;
        } else {
            x[0] *= kEnd;
            x[n - 1] *= kEnd;
#pragma unroll
            for (int f = 1; f < n - 1; ++f) x[f] *= kMid;
            auto C = [&](int q) { return q == 0 ? x[0] : q == N ? x[n - 1] : x[2 * q - 1]; };
#pragma unroll
            for (int c = 0; c <= H; ++c) {
                double ce = x[0], co = 0.0, so = 0.0, se = 0.0;
#pragma unroll
                for (int q = 1; q <= N; ++q) {
                    if (q % 2 == 0) ce = fma(cosn<n>(q * c), C(q), ce);
                    else if (c < H) co = fma(cosn<n>(q * c), C(q), co);
                    if (q < N && c > 0) {
                        if (q % 2 == 1) so = fma(sinn<n>(q * c), x[2 * q], so);
                        else if (c < H) se = fma(sinn<n>(q * c), x[2 * q], se);
                    }
                }
                const double a0 = ce + co, a1 = ce - co, b0 = so + se, b1 = so - se;
                v[c] = a0 + b0;
                if (c > 0) v[n - c] = a0 - b0;
                if (c < H) {
                    v[N - c] = a1 + b1;
                    if (c > 0) v[N + c] = a1 - b1;
                }
            }
        }
    }
};

__device__ inline double load_m(const ConvLevel &v, size_t i) {
    return v.fp64 ? reinterpret_cast<const double *>(v.M)[i] : (double)reinterpret_cast<const float *>(v.M)[i];
}
// ---------------------------------------------------------------- levels 1 .. 4
// All three axes of CG coefficients of a level in LDS: a thread takes one line
// at a time in registers, in place.  Rows of a line's y are padded by CG
// doubles so that the lines of z do not meet in one bank.
template <int n, int CG, bool FWD>
__device__ inline void cube(const ConvLevel &v, int part, int NB, int Kp, const ConvCoef *__restrict__ tab,
                            double *lds) {
    constexpr int SY = n * CG + CG, SX = n * SY;
    const int tid = threadIdx.x;
    const bool on = tid < n * n * CG;
    const int c = tid % CG, a = tid / CG % n, b = tid / CG / n;
    const int pos = part * CG + c;
    const ConvCoef t = tab[pos];
    double x[n], o[n];
    if constexpr (FWD) {
        if (on) {  // a = z, b = y
            for (int i = 0; i < n; ++i) x[i] = load_m(v, (size_t)morton3(i, b, a) * Kp + t.sto);
            Line<n>::forward(x, o);
            for (int i = 0; i < n; ++i) lds[i * SX + b * SY + a * CG + c] = o[i];
        }
        __syncthreads();
        if (on) {  // a = z, b = x
            for (int i = 0; i < n; ++i) x[i] = lds[b * SX + i * SY + a * CG + c];
            Line<n>::forward(x, o);
            for (int i = 0; i < n; ++i) lds[b * SX + i * SY + a * CG + c] = o[i];
        }
        __syncthreads();
        if (on) {  // a = y, b = x
            for (int i = 0; i < n; ++i) x[i] = lds[b * SX + a * SY + i * CG + c];
            Line<n>::forward(x, o);
            const Axis ax = axis_of(b, n, t.flips & 1), ay = axis_of(a, n, t.flips >> 1 & 1);
            for (int i = 0; i < n; ++i) {
                const Entry e = entry_of(ax, ay, axis_of(i, n, t.flips >> 2), pos, t, false, n / 2, NB, v.pair);
                v.Q[e.at] = e.neg ? -o[i] : o[i];
            }
        }
    } else {
        if (on) {
            const Axis ax = axis_of(b, n, t.flips & 1), ay = axis_of(a, n, t.flips >> 1 & 1);
            for (int i = 0; i < n; ++i) {
                const Entry e = entry_of(ax, ay, axis_of(i, n, t.flips >> 2), pos, t, true, n / 2, NB, v.pair);
                const double w = v.P[e.at];
                x[i] = e.neg ? -w : w;
            }
            Line<n>::inverse(x, o);
            for (int i = 0; i < n; ++i) lds[b * SX + a * SY + i * CG + c] = o[i];
        }
        __syncthreads();
        if (on) {
            for (int i = 0; i < n; ++i) x[i] = lds[b * SX + i * SY + a * CG + c];
            Line<n>::inverse(x, o);
            for (int i = 0; i < n; ++i) lds[b * SX + i * SY + a * CG + c] = o[i];
        }
        __syncthreads();
        if (on) {
            for (int i = 0; i < n; ++i) x[i] = lds[i * SX + b * SY + a * CG + c];
            Line<n>::inverse(x, o);
            for (int i = 0; i < n; ++i) v.L[(size_t)morton3(i, b, a) * Kp + t.sto] = o[i];
        }
    }
}

struct ConvBatch {
    ConvLevel lv[kConvMaxBatch];
    int nlv;
    int start[kConvMaxBatch + 1];  // first block of each level
};

// DEEP: level 4 among the levels (70 KB of LDS instead of 37).  512 threads: twice the
// blocks of 1024 threads, which are few (p = 10: 66 with level 4), and a workgroup
// that finds room beside the near field's own of 8 wavefronts (leaf M2L of levels 4,
// p = 10: 137 -> 129 us, levels 3, p = 8: 47 -> 43 us; whole call of 125,001 atoms
// 577 -> 551 us).
template <bool FWD, bool DEEP>
__global__ __launch_bounds__(512) void k_conv_cube(ConvBatch bt, int NB, int Kp, const ConvCoef *__restrict__ tab) {
    __shared__ double lds[DEEP ? 16 * 16 * (16 * 2 + 2) : 8 * 8 * (8 * 8 + 8)];
    int w = 0;
    while (w + 1 < bt.nlv && (int)blockIdx.x >= bt.start[w + 1]) ++w;
    const ConvLevel &v = bt.lv[w];
    const int part = blockIdx.x - bt.start[w];
    switch (v.level) {
        case 1: cube<2, 8, FWD>(v, part, NB, Kp, tab, lds); break;
        case 2: cube<4, 8, FWD>(v, part, NB, Kp, tab, lds); break;
        case 3: cube<8, 8, FWD>(v, part, NB, Kp, tab, lds); break;
        case 4:
            if constexpr (DEEP) cube<16, 2, FWD>(v, part, NB, Kp, tab, lds);
            break;
    }
}

// ---------------------------------------------------------------- levels 5, 6
// The x and y lines of one plane of cells (fixed z) for CG coefficients in
// LDS, then the z lines from and to memory.  Between them: [chunk][z][y][x][16].
// S: the type of M.
template <typename S, int n, int CG>
__global__ __launch_bounds__(n *CG) void k_conv_plane_fwd(ConvLevel v, int Kp, const ConvCoef *__restrict__ tab) {
    constexpr int SX = n * CG + CG;
    __shared__ double lds[n * SX];
    constexpr int parts = 16 / CG;
    const int c = threadIdx.x % CG, line = threadIdx.x / CG;
    // the parts of a chunk and the chunks of a plane are 8 blocks apart: one
    // XCD's L2 serves all readers of the plane's multipole rows
    const int per = Kp / CG;  // blocks of a plane
    const int z = blockIdx.x / (8 * per) * 8 + blockIdx.x % 8, part = blockIdx.x / 8 % per;
    const int pos = part * CG + c;
    const int sto = tab[pos].sto;
    double x[n], o[n];
#pragma unroll
    for (int i = 0; i < n; ++i)
        x[i] = reinterpret_cast<const S *>(v.M)[(size_t)morton3(i, line, z) * Kp + sto];
    Line<n>::forward(x, o);
#pragma unroll
    for (int i = 0; i < n; ++i) lds[i * SX + line * CG + c] = o[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < n; ++i) x[i] = lds[line * SX + i * CG + c];
    Line<n>::forward(x, o);
    double *q = v.Q + (size_t)(part / parts * n + z) * n * n * 16 + line * 16 + part % parts * CG + c;
#pragma unroll
    for (int i = 0; i < n; ++i) q[(size_t)i * n * 16] = o[i];
}

template <int n, int CG>
__global__ __launch_bounds__(n *CG) void k_conv_plane_inv(ConvLevel v, int Kp, const ConvCoef *__restrict__ tab) {
    constexpr int SX = n * CG + CG;
    __shared__ double lds[n * SX];
    constexpr int parts = 16 / CG;
    const int c = threadIdx.x % CG, line = threadIdx.x / CG;
    const int per = Kp / CG;
    const int z = blockIdx.x / (8 * per) * 8 + blockIdx.x % 8, part = blockIdx.x / 8 % per;
    const int pos = part * CG + c;
    const int sto = tab[pos].sto;
    double x[n], o[n];
    const double *q = v.P + (size_t)(part / parts * n + z) * n * n * 16 + line * 16 + part % parts * CG + c;
#pragma unroll
    for (int i = 0; i < n; ++i) x[i] = q[(size_t)i * n * 16];
    Line<n>::inverse(x, o);
#pragma unroll
    for (int i = 0; i < n; ++i) lds[line * SX + i * CG + c] = o[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < n; ++i) x[i] = lds[i * SX + line * CG + c];
    Line<n>::inverse(x, o);
#pragma unroll
    for (int i = 0; i < n; ++i) v.L[(size_t)morton3(i, line, z) * Kp + sto] = o[i];
}

// One z line per thread: 16 coefficients x 16 x slots of one y slot per block.
// FWD: Q (planes) -> P (columns); else Q (columns) -> P (planes).
template <int n, bool FWD>
__global__ __launch_bounds__(256) void k_conv_z(ConvLevel v, int NB, const ConvCoef *__restrict__ tab) {
    const int c = threadIdx.x & 15;
    const int fx = blockIdx.x % (n / 16) * 16 + (threadIdx.x >> 4);
    const int fy = blockIdx.x / (n / 16) % n, cc = blockIdx.x / (n / 16) / n;
    const int pos = cc * 16 + c;
    const ConvCoef t = tab[pos];
    const Axis ax = axis_of(fx, n, t.flips & 1), ay = axis_of(fy, n, t.flips >> 1 & 1);
    const size_t plane = ((size_t)cc * n * n + fy) * n * 16 + fx * 16 + c;
    double x[n], o[n];
    if constexpr (FWD) {
#pragma unroll
        for (int i = 0; i < n; ++i) x[i] = v.Q[plane + (size_t)i * n * n * 16];
        Line<n>::forward(x, o);
#pragma unroll
        for (int i = 0; i < n; ++i) {
            const Entry e = entry_of(ax, ay, axis_of(i, n, t.flips >> 2), pos, t, false, n / 2, NB, v.pair);
            v.P[e.at] = e.neg ? -o[i] : o[i];
        }
    } else {
#pragma unroll
        for (int i = 0; i < n; ++i) {
            const Entry e = entry_of(ax, ay, axis_of(i, n, t.flips >> 2), pos, t, true, n / 2, NB, v.pair);
            const double w = v.Q[e.at];
            x[i] = e.neg ? -w : w;
        }
        Line<n>::inverse(x, o);
#pragma unroll
        for (int i = 0; i < n; ++i) v.P[plane + (size_t)i * n * n * 16] = o[i];
    }
}

// ---------------------------------------------------------------- the products
// One workgroup: 16 result rows (all 8 tau) of one triple of wave numbers, its
// waves taking the chunks of 16 columns in turn; their sums meet in LDS in a
// fixed order.  A wave holds the eight 16 x 16 results, the eight column
// fragments of the chunk and the 9 blocks of one x type, each used for one
// (types 0, 1) to eight (type 2 in all axes) of the 64 (tau, tau') products.
// A: type of the blocks.  Columns and products are FP64 for FP32 blocks too.  In FP32
// levels 5 and 6 take 0.1 and 0.4 ms less (whole call, 1M atoms at p = 12 2.98 against
// 3.08 ms, 3M at p = 8 5.77 against 6.14) but round each column and result twice and add
// chains of 128 products: far-field potential error of 4,000 charges in levels 6, p = 3,
// levels 1-4 in FP64, 2.4e-7 against 3.9e-8 (the interaction lists: 2.0e-7), of 20,000 in
// levels 5, p = 6, 1.1e-7 against 2.7e-8 (1.1e-7).
template <typename A>
__device__ inline void conv_product(const ConvLevel &v, int o, int rt, int NB, const double *__restrict__ X,
                                    double *__restrict__ Y, double (*red)[8][4][64]) {
    using AV = typename Mfma<A>::V;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
    const int N = (1 << v.level) / 2, H1 = N / 2 + 1;
    int kx = 0, ky = o / H1;
    const int kz = o % H1, pr = ky;
    while (ky > kx) ky -= ++kx;
    const int rxy = nvec(kx, N) * nvec(ky, N) * (kx != ky ? 2 : 1);
    const uint32_t col0 = (uint32_t)v.pair[pr] + rxy * (kz == 0 ? 0 : 2 * kz - 1);
    const int ncol = rxy * nvec(kz, N);
    const int col = lane & 15;
    // columns past the last read it again; their results are not stored
    const uint32_t xo = col0 * NB * 128u + (uint32_t)(col < ncol ? col : ncol - 1) * 16u + 4u * (lane >> 4);
    const A *ap = reinterpret_cast<const A *>(v.ops) + ((size_t)o * NB + rt) * NB * (kConvTypes * 256) + lane * 4;

    f64x4 acc[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) acc[t] = f64x4{0, 0, 0, 0};
    for (int cc = w; cc < NB; cc += nw) {
        f64x4 b[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) b[t] = *reinterpret_cast<const f64x4 *>(X + xo + (uint32_t)(cc * 8 + t) * ncol * 16u);
        const A *a0 = ap + (size_t)cc * (kConvTypes * 256);
#pragma unroll
        for (int tx = 0; tx < 3; ++tx) {
            AV a[9];
#pragma unroll
            for (int i = 0; i < 9; ++i)
                a[i] = __builtin_nontemporal_load(reinterpret_cast<const AV *>(a0 + (tx * 9 + i) * 256));
#pragma unroll
            for (int i = 0; i < 9; ++i) {
                const int ty = i / 3, tz = i % 3;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const double av = (double)a[i][j];
#pragma unroll
                    for (int t = 0; t < 8; ++t) {
                        // t: tau of the result; the source's tau' follows from the types
                        const int x = t >> 2, y = t >> 1 & 1, z = t & 1;
                        if ((tx < 2 && x != tx) || (ty < 2 && y != ty) || (tz < 2 && z != tz)) continue;
                        const int s = (tx == 2 ? !x : x) << 2 | (ty == 2 ? !y : y) << 1 | (tz == 2 ? !z : z);
                        acc[t] = Mfma<double>::mma(av, b[s][j], acc[t]);
                    }
                }
            }
        }
    }
#pragma unroll
    for (int t = 0; t < 8; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) red[w][t][r][lane] = acc[t][r];
    __syncthreads();
    // lanes along the rows: 16 neighbouring results a column
    const int row = lane & 15;
    const int rr = row >> 2, rl = 16 * (row & 3);  // where the result's layout puts (row, column)
    double *yo = Y + (col0 * NB + rt * ncol) * 128u + row;
    for (int i = w; i < 32; i += nw) {
        const int t = i >> 2, c = 4 * (i & 3) + (lane >> 4);
        if (c >= ncol) continue;
        double s = 0.0;
        for (int k = 0; k < nw; ++k) s += red[k][t][rr][rl + c];
        yo[(uint32_t)(t * ncol + c) * 16u] = s;
    }
}

// The 16-row tiles of one triple are 8 blocks apart (one XCD: they read the
// same columns).  MODE 0: FP32 blocks, 1: FP64 ones, 2: either, by level.
template <int MODE>
__global__ __launch_bounds__(256) void k_conv_product(ConvBatch bt, int NB, int swapPQ) {
    extern __shared__ double red_raw[];  // [wavefronts][8][4][64]
    double(*red)[8][4][64] = reinterpret_cast<double(*)[8][4][64]>(red_raw);
    int w = 0;
    while (w + 1 < bt.nlv && (int)blockIdx.x >= bt.start[w + 1]) ++w;
    const ConvLevel &v = bt.lv[w];
    const int bid = blockIdx.x - bt.start[w];
    const int o = bid / (8 * NB) * 8 + bid % 8, rt = bid / 8 % NB;
    const int H1 = (1 << v.level) / 4 + 1;
    if (o >= H1 * (H1 + 1) / 2 * H1) return;  // whole workgroup
    const double *X = swapPQ ? v.P : v.Q;
    double *Y = swapPQ ? v.Q : v.P;
    if (MODE == 0 || (MODE == 2 && !v.fp64)) conv_product<float>(v, o, rt, NB, X, Y, red);
    else conv_product<double>(v, o, rt, NB, X, Y, red);
}

// ---------------------------------------------------------------- the blocks
// One thread: entry (r, c) of the 27 blocks of the triples (kx >= ky, ky, kz),
// ky and kz of the block; the sums over d are taken axis by axis.
template <typename AT>
__global__ __launch_bounds__(256) void k_conv_build(int N, int Kp, const double *__restrict__ reps,
                                                    const int32_t *__restrict__ index,
                                                    const double *__restrict__ trig, const ConvCoef *__restrict__ tab,
                                                    AT *__restrict__ ops) {
    const int NB = Kp / 16, H = N / 2;
    const int rt = blockIdx.x / NB, cc = blockIdx.x % NB, ky = blockIdx.y, kz = blockIdx.z;
    const int j = threadIdx.x & 3, row = threadIdx.x >> 2 & 15, kq = threadIdx.x >> 6;
    const int r = 16 * rt + row, c = 16 * cc + 4 * kq + j;
    const int fr = tab[r].flips, fc = tab[c].flips;
    auto weight = [&](int a, int k, int d) { return conv_weight(fr >> a & 1, fc >> a & 1, d, k, N, trig); };
    auto cross = [&](int a, int k) { return conv_cross(fr >> a & 1, fc >> a & 1, k, N, trig); };
    // the three types of one axis from the six terms t_d: e / o of even / odd d
    double wz[6], wy[6], xz = cross(2, kz), xy = cross(1, ky);
#pragma unroll
    for (int d = 0; d < 6; ++d) {
        wz[d] = weight(2, kz, d);
        wy[d] = weight(1, ky, d);
    }
    double yv[6][9];
#pragma unroll
    for (int dx = 0; dx < 6; ++dx) {
#pragma unroll
        for (int i = 0; i < 9; ++i) yv[dx][i] = 0.0;
#pragma unroll
        for (int dy = 0; dy < 6; ++dy) {
            double e = 0.0, o = 0.0, f = 0.0;
#pragma unroll
            for (int dz = 0; dz < 6; ++dz) {
                if (dx <= kWS && dy <= kWS && dz <= kWS) continue;
                const double t = reps[((size_t)index[(dx * 6 + dy) * 6 + dz] * Kp + r) * Kp + c];
                if (dz % 2 == 0) e = fma(wz[dz], t, e);
                else o = fma(wz[dz], t, o);
                if (dz == 5) f = xz * t;
            }
            const double z3[3] = {e + o, e - o, f};
#pragma unroll
            for (int tz = 0; tz < 3; ++tz) {
                const double u = wy[dy] * z3[tz];
                yv[dx][0 + tz] += u;
                yv[dx][3 + tz] += dy % 2 == 0 ? u : -u;
                if (dy == 5) yv[dx][6 + tz] = xy * z3[tz];
            }
        }
    }
    for (int kx = ky; kx <= H; ++kx) {
        const size_t orb = (size_t)(kx * (kx + 1) / 2 + ky) * (H + 1) + kz;
        AT *out = ops + ((orb * NB + rt) * NB + cc) * (kConvTypes * 256) + (kq * 16 + row) * 4 + j;
        double wx[6];
#pragma unroll
        for (int d = 0; d < 6; ++d) wx[d] = weight(0, kx, d);
        const double xx = cross(0, kx);
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            const double e = wx[0] * yv[0][i] + wx[2] * yv[2][i] + wx[4] * yv[4][i];
            const double o = wx[1] * yv[1][i] + wx[3] * yv[3][i] + wx[5] * yv[5][i];
            out[(0 * 9 + i) * 256] = (AT)(e + o);
            out[(1 * 9 + i) * 256] = (AT)(e - o);
            out[(2 * 9 + i) * 256] = (AT)(xx * yv[5][i]);
        }
    }
}

}  // namespace

hipError_t launch_conv_build(int level, int p, const double *reps, const int32_t *index, const double *trig,
                             const ConvCoef *tab, void *ops, size_t elem, hipStream_t s) {
    const int N = (1 << level) / 2, Kp = padded_coeffs(p), NB = Kp / 16;
    const dim3 grid(NB * NB, N / 2 + 1, N / 2 + 1);
    if (elem == 4)
        hipLaunchKernelGGL(k_conv_build<float>, grid, dim3(256), 0, s, N, Kp, reps, index, trig, tab, (float *)ops);
    else
        hipLaunchKernelGGL(k_conv_build<double>, grid, dim3(256), 0, s, N, Kp, reps, index, trig, tab, (double *)ops);
    return hipGetLastError();
}

static int product_blocks(int level, int NB) { return (conv_orbits(level) + 7) / 8 * 8 * NB; }

// Wavefronts of a workgroup: they share the chunks of its rows, and the chip takes
// 2048 at a time (two a SIMD); of 4, 2 and 1 the number that needs the fewest
// chunk times in whole rounds (3M-atom box, p = 8, 6 chunks: 2 wavefronts, since 4
// would leave two of them idle in the second turn: far field alone 3.15 -> 2.99 ms;
// 1M atoms, p = 12, 11 chunks: 4 wavefronts 1.20 ms, 2 1.25, 1 1.30).
static int product_waves(const ConvBatch &b, int NB) {
    int64_t tiles = 0, best = 0;
    int nw = 1;
    for (int i = 0; i < b.nlv; ++i) tiles += (int64_t)conv_orbits(b.lv[i].level) * NB;
    for (int k : {4, 2, 1}) {
        if (k > NB) continue;
        const int64_t cost = (tiles * k + 2047) / 2048 * ((NB + k - 1) / k);
        if (best == 0 || cost < best) {
            best = cost;
            nw = k;
        }
    }
    return nw;
}

static hipError_t launch_product(const ConvBatch &b, int blocks, int NB, int swapPQ, hipStream_t s) {
    bool f32 = false, f64 = false;
    for (int i = 0; i < b.nlv; ++i) (b.lv[i].fp64 ? f64 : f32) = true;
    const int nw = product_waves(b, NB);
    const dim3 grid(blocks), block(64 * nw);
    const size_t lds = sizeof(double) * nw * 8 * 4 * 64;
    if (f32 && f64) hipLaunchKernelGGL(k_conv_product<2>, grid, block, lds, s, b, NB, swapPQ);
    else if (f64) hipLaunchKernelGGL(k_conv_product<1>, grid, block, lds, s, b, NB, swapPQ);
    else hipLaunchKernelGGL(k_conv_product<0>, grid, block, lds, s, b, NB, swapPQ);
    return hipGetLastError();
}

template <typename S, int n, int CG>
static hipError_t conv_large(const ConvLevel &v, int Kp, const ConvCoef *tab, hipStream_t s) {
    const int NB = Kp / 16;
    const dim3 planes(n * (Kp / CG)), lines(NB * n * (n / 16));
    ConvBatch b{};
    b.lv[0] = v;
    b.nlv = 1;
    b.start[1] = product_blocks(v.level, NB);
    hipLaunchKernelGGL((k_conv_plane_fwd<S, n, CG>), planes, dim3(n * CG), 0, s, v, Kp, tab);
    hipLaunchKernelGGL((k_conv_z<n, true>), lines, dim3(256), 0, s, v, NB, tab);
    hipError_t e = launch_product(b, b.start[1], NB, 1, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_conv_z<n, false>), lines, dim3(256), 0, s, v, NB, tab);
    hipLaunchKernelGGL((k_conv_plane_inv<n, CG>), planes, dim3(n * CG), 0, s, v, Kp, tab);
    return hipGetLastError();
}

hipError_t launch_conv(const ConvLevel *lv, int nlv, int p, const ConvCoef *tab, hipStream_t s) {
    if (nlv < 1 || nlv > kConvMaxBatch) return hipErrorInvalidValue;
    const int Kp = padded_coeffs(p), NB = Kp / 16;
    if (lv[0].level > 4) {
        if (nlv != 1 || lv[0].level > kConvMaxLevel) return hipErrorInvalidValue;
        if (lv[0].fp64)
            return lv[0].level == 5 ? conv_large<double, 32, 16>(lv[0], Kp, tab, s)
                                    : conv_large<double, 64, 4>(lv[0], Kp, tab, s);
        return lv[0].level == 5 ? conv_large<float, 32, 16>(lv[0], Kp, tab, s)
                                : conv_large<float, 64, 4>(lv[0], Kp, tab, s);
    }
    ConvBatch cube{}, prod{};
    cube.nlv = prod.nlv = nlv;
    bool deep = false;
    for (int i = 0; i < nlv; ++i) {
        const int l = lv[i].level;
        if (l < 1 || l > 4) return hipErrorInvalidValue;
        cube.lv[i] = prod.lv[i] = lv[i];
        deep = deep || l == 4;
        cube.start[i + 1] = cube.start[i] + Kp / (l == 4 ? 2 : 8);
        prod.start[i + 1] = prod.start[i] + product_blocks(l, NB);
    }
    const dim3 grid(cube.start[nlv]);
    if (deep) hipLaunchKernelGGL((k_conv_cube<true, true>), grid, dim3(512), 0, s, cube, NB, Kp, tab);
    else hipLaunchKernelGGL((k_conv_cube<true, false>), grid, dim3(512), 0, s, cube, NB, Kp, tab);
    hipError_t e = launch_product(prod, prod.start[nlv], NB, 0, s);
    if (e != hipSuccess) return e;
    if (deep) hipLaunchKernelGGL((k_conv_cube<false, true>), grid, dim3(512), 0, s, cube, NB, Kp, tab);
    else hipLaunchKernelGGL((k_conv_cube<false, false>), grid, dim3(512), 0, s, cube, NB, Kp, tab);
    return hipGetLastError();
}

}  // namespace fmm
