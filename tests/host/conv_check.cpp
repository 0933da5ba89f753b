// Host check of the convolution form of the M2L, built and run by
// tests/test_conv_host.py: the index maps, weights and tables that the kernels
// use, in plain loops, against the sum over the 875 offsets of every cell.
//   conv_check maps LEVEL P      every array entry is hit exactly once
//   conv_check sum LEVEL P       largest difference over the largest value
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>

#include "conv_map.h"

using namespace fmm;

int main(int argc, char **argv) {
    if (argc != 4) return 2;
    const int level = std::atoi(argv[2]), p = std::atoi(argv[3]);
    const int n = 1 << level, N = n / 2, K = num_coeffs(p), Kp = padded_coeffs(p), NB = Kp / 16;
    std::vector<ConvCoef> tab;
    conv_coef_table(p, tab);
    std::vector<int32_t> pair;
    conv_pair_base(level, pair);
    const size_t total = (size_t)n * n * n * Kp;
    auto entry = [&](int fx, int fy, int fz, int c, bool local) {
        const int f = tab[c].flips;
        return entry_of(axis_of(fx, n, f & 1), axis_of(fy, n, f >> 1 & 1), axis_of(fz, n, f >> 2), c, tab[c], local, N,
                        NB, pair.data());
    };
    if (!std::strcmp(argv[1], "maps")) {
        std::vector<unsigned char> hit(total, 0);
        for (int x = 0; x < n; ++x)
            for (int y = 0; y < n; ++y)
                for (int z = 0; z < n; ++z)
                    for (int c = 0; c < Kp; ++c) {
                        const Entry e = entry(x, y, z, c, false);
                        if (e.at >= total || hit[e.at]) return 1;
                        if (entry(x, y, z, c, true).at != e.at) return 1;
                        hit[e.at] = 1;
                    }
        std::vector<unsigned char> seen(Kp, 0);
        for (const ConvCoef &c : tab) {
            if (c.sto < 0 || c.sto >= Kp || seen[c.sto] || tab[c.mir].mir != &c - tab.data()) return 1;
            seen[c.sto] = 1;
        }
        std::puts("ok");
        return 0;
    }
    // multipoles of every cell, [x][y][z][position in the convolution's order]
    std::mt19937 rng(7);
    std::normal_distribution<double> g;
    std::vector<double> M(total, 0.0), L(total, 0.0), X(total), Y(total, 0.0), W((size_t)n * n);
    auto at = [&](int x, int y, int z) { return (((size_t)x * n + y) * n + z) * Kp; };
    for (size_t i = 0; i < total; ++i)
        if ((int)(i % Kp) < K) M[i] = g(rng);
    for (int c = 0; c < n; ++c)
        for (int q = 0; q <= N; ++q) {
            const double end = std::sqrt(1.0 / n), mid = std::sqrt(2.0 / n), a = 2 * M_PI * q * c / n;
            if (q == 0) W[c] = end;
            else if (q == N) W[(size_t)(n - 1) * n + c] = c % 2 ? -end : end;
            else {
                W[(size_t)(2 * q - 1) * n + c] = mid * std::cos(a);
                W[(size_t)2 * q * n + c] = mid * std::sin(a);
            }
        }
    auto lines = [&](const std::vector<double> &in, bool inverse) {
        std::vector<double> a = in, b(total);
        for (int axis = 0; axis < 3; ++axis) {
            for (int u = 0; u < n; ++u)
                for (int v = 0; v < n; ++v)
                    for (int f = 0; f < n; ++f)
                        for (int c = 0; c < Kp; ++c) {
                            auto cell = [&](int i) {
                                return axis == 0 ? at(i, u, v) : axis == 1 ? at(u, i, v) : at(u, v, i);
                            };
                            double s = 0.0;
                            for (int i = 0; i < n; ++i) s += W[inverse ? (size_t)i * n + f : (size_t)f * n + i] * a[cell(i) + c];
                            b[cell(f) + c] = s;
                        }
            a.swap(b);
        }
        return a;
    };
    const std::vector<double> T = lines(M, false);
    for (int x = 0; x < n; ++x)
        for (int y = 0; y < n; ++y)
            for (int z = 0; z < n; ++z)
                for (int c = 0; c < Kp; ++c) {
                    const Entry e = entry(x, y, z, c, false);
                    X[e.at] = (e.neg ? -1.0 : 1.0) * T[at(x, y, z) + c];
                }
    std::vector<double> reps, trig;
    std::vector<int32_t> index;
    conv_reps(p, tab, reps, index);
    conv_trig(level, trig);
    std::vector<double> G((size_t)27 * Kp * Kp);
    const int H = N / 2;
    for (int kx = 0, pr = 0; kx <= H; ++kx)
        for (int ky = 0; ky <= kx; ++ky, ++pr)
            for (int kz = 0; kz <= H; ++kz) {
                const int k[3] = {kx, ky, kz};
                for (int r = 0; r < Kp; ++r)
                    for (int c = 0; c < Kp; ++c)
                        for (int ty = 0; ty < 27; ++ty) {
                            const int t[3] = {ty / 9, ty / 3 % 3, ty % 3};
                            double s = 0.0;
                            for (int d = 0; d < 216; ++d) {
                                if (index[d] < 0) continue;
                                const int o[3] = {d / 36, d / 6 % 6, d % 6};
                                double w = reps[((size_t)index[d] * Kp + r) * Kp + c];
                                for (int a = 0; a < 3; ++a) {
                                    const int fr = tab[r].flips >> a & 1, fc = tab[c].flips >> a & 1;
                                    if (t[a] == 2) w *= o[a] == 5 ? conv_cross(fr, fc, k[a], N, trig.data()) : 0.0;
                                    else w *= conv_weight(fr, fc, o[a], k[a], N, trig.data()) * (t[a] == 1 && o[a] % 2 ? -1 : 1);
                                }
                                s += w;
                            }
                            G[((size_t)ty * Kp + r) * Kp + c] = s;
                        }
                const int rxy = nvec(kx, N) * nvec(ky, N) * (kx != ky ? 2 : 1), ncol = rxy * nvec(kz, N);
                const size_t base = (size_t)(pair[pr] + rxy * (kz == 0 ? 0 : 2 * kz - 1)) * NB * 128;
                auto el = [&](int tau, int col, int c) { return base + (size_t)(c / 16 * ncol) * 128 + (size_t)(tau * ncol + col) * 16 + c % 16; };
                for (int col = 0; col < ncol; ++col)
                    for (int ta = 0; ta < 8; ++ta)
                        for (int tb = 0; tb < 8; ++tb) {
                            int ty = 0;
                            for (int a = 2; a >= 0; --a) {
                                const int u = ta >> a & 1, v = tb >> a & 1;
                                ty = 3 * ty + (u == v ? u : 2);
                            }
                            for (int r = 0; r < Kp; ++r)
                                for (int c = 0; c < Kp; ++c)
                                    Y[el(ta, col, r)] += G[((size_t)ty * Kp + r) * Kp + c] * X[el(tb, col, c)];
                        }
            }
    std::vector<double> R(total);
    for (int x = 0; x < n; ++x)
        for (int y = 0; y < n; ++y)
            for (int z = 0; z < n; ++z)
                for (int c = 0; c < Kp; ++c) {
                    const Entry e = entry(x, y, z, c, true);
                    R[at(x, y, z) + c] = (e.neg ? -1.0 : 1.0) * Y[e.at];
                }
    const std::vector<double> conv = lines(R, true);
    // the list of every cell, offset by offset
    const Offsets offs = build_offsets();
    std::vector<double> A((size_t)K * K);
    for (int id = 0; id < kNumOffsets; ++id) {
        const int *d = &offs.vec[3 * id];
        const double t[3] = {(double)d[0], (double)d[1], (double)d[2]};
        build_m2l_operator(p, t, A.data());
        for (int par = 0; par < 8; ++par) {
            bool in = false;
            for (int i = 0; i < kILSize; ++i) in = in || offs.il[par * kILSize + i] == id;
            if (!in) continue;
            for (int x = par >> 2 & 1; x < n; x += 2)
                for (int y = par >> 1 & 1; y < n; y += 2)
                    for (int z = par & 1; z < n; z += 2) {
                        auto w = [&](int v) { return ((v % n) + n) % n; };
                        const double *m = &M[at(w(x + d[0]), w(y + d[1]), w(z + d[2]))];
                        for (int r = 0; r < K; ++r)
                            for (int c = 0; c < K; ++c)
                                L[at(x, y, z) + r] += A[(size_t)tab[r].sto * K + tab[c].sto] * m[c];
                    }
        }
    }
    double worst = 0.0, big = 0.0;
    for (size_t i = 0; i < total; ++i) {
        worst = std::fmax(worst, std::fabs(L[i] - conv[i]));
        big = std::fmax(big, std::fabs(L[i]));
    }
    std::printf("%.3e\n", worst / big);
    return 0;
}
