// Host side of the convolution form of the M2L (stage a6): the coefficient
// order of its arrays, the operators of the reflection representatives and the
// tables of one level.  The algebra is at the head of k_conv.hip; plain C++,
// run once per plan.
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <thread>
#include <vector>

#include "fmm_internal.h"

namespace fmm {

// Coefficients grouped by their signs under the three axis reflections (in a
// class by degree and order), so that the lanes of a line transform that
// scatters by class write contiguous runs, and so that the mirror x <-> y maps
// position i of a class to position i of the class with x and y exchanged.
void conv_coef_table(int p, std::vector<ConvCoef> &out) {
    const int K = num_coeffs(p), Kp = padded_coeffs(p);
    struct Item {
        int cls, n, m, im, k;
    };
    std::vector<Item> v;
    for (int n = 0, k = 0; n <= p; ++n)
        for (int r = 0; r < 2 * n + 1; ++r, ++k) {
            const int m = (r + 1) / 2, im = r > 0 && r % 2 == 0;
            const int fx = (m & 1) ^ im, fy = im, fz = (n + m) & 1;  // 1: the reflection flips the sign
            v.push_back({fx | fy << 1 | fz << 2, n, m, im, k});
        }
    std::stable_sort(v.begin(), v.end(), [](const Item &a, const Item &b) { return a.cls < b.cls; });
    std::vector<int> pos(K);
    for (int i = 0; i < K; ++i) pos[v[i].k] = i;
    out.assign(Kp, ConvCoef{});
    for (int i = 0; i < Kp; ++i) {
        ConvCoef &c = out[i];
        if (i >= K) {  // padding: zero operator rows and columns
            c.sto = (int16_t)i;
            c.mir = (int16_t)i;
            continue;
        }
        const Item &t = v[i];
        const int half = (t.m / 2) & 1;  // cos(m pi/2) or sin(m pi/2) is negative
        c.sto = (int16_t)t.k;
        c.flips = (uint8_t)t.cls;
        if (t.m & 1) {
            // the mirror exchanges the real and imaginary parts; multipoles
            // hold conj(R), locals I, hence the opposite signs of the two
            c.mir = (int16_t)pos[t.n * t.n + 2 * t.m - (t.im ? 1 : 0)];
            c.mneg = (uint8_t)!half;
            c.lneg = (uint8_t)half;
        } else {
            c.mir = (int16_t)i;
            c.mneg = c.lneg = (uint8_t)(half ^ t.im);
        }
    }
}

int conv_orbits(int level) {
    const int H = (1 << level) / 4;  // largest wave number of the parents' grid
    return (H + 1) * (H + 2) / 2 * (H + 1);
}

size_t conv_op_bytes(int level, int p, size_t elem) {
    const size_t Kp = (size_t)padded_coeffs(p);
    return (size_t)conv_orbits(level) * kConvTypes * Kp * Kp * elem;
}

// O_d of the 189 offsets with non-negative components, rows and columns in the
// coefficient order above, zero-padded: out[rep][Kp][Kp]; rep of (dx, dy, dz)
// at index[(dx * 6 + dy) * 6 + dz], -1 for the near field.
void conv_reps(int p, const std::vector<ConvCoef> &tab, std::vector<double> &out, std::vector<int32_t> &index) {
    const int K = num_coeffs(p), Kp = padded_coeffs(p);
    index.assign(216, -1);
    std::vector<int> d;
    for (int a = 0; a < 216; ++a) {
        const int x = a / 36, y = a / 6 % 6, z = a % 6;
        if (std::max(x, std::max(y, z)) <= kWS) continue;
        index[a] = (int)d.size();
        d.push_back(a);
    }
    out.assign(d.size() * (size_t)Kp * Kp, 0.0);
    const unsigned nt = std::max(1u, std::min(16u, std::thread::hardware_concurrency()));
    std::vector<std::thread> th;
    for (unsigned w = 0; w < nt; ++w)
        th.emplace_back([&, w] {
            std::vector<double> A((size_t)K * K);
            for (size_t i = w; i < d.size(); i += nt) {
                const double t[3] = {(double)(d[i] / 36), (double)(d[i] / 6 % 6), (double)(d[i] % 6)};
                build_m2l_operator(p, t, A.data());
                double *o = out.data() + i * Kp * Kp;
                for (int r = 0; r < K; ++r)
                    for (int c = 0; c < K; ++c) o[(size_t)r * Kp + c] = A[(size_t)tab[r].sto * K + tab[c].sto];
            }
        });
    for (auto &t : th) t.join();
}

// First column of every pair (kx >= ky) of wave numbers, all kz together:
// the columns of a triple are its real vectors (see k_conv.hip).
void conv_pair_base(int level, std::vector<int32_t> &base) {
    const int N = (1 << level) / 2, H = N / 2;
    auto r = [&](int k) { return k == 0 || 2 * k == N ? 1 : 2; };
    base.clear();
    int32_t at = 0;
    for (int x = 0; x <= H; ++x)
        for (int y = 0; y <= x; ++y) {
            base.push_back(at);
            at += r(x) * r(y) * (x != y ? 2 : 1) * N;
        }
    base.push_back(at);  // N^3, every parent's worth of columns
}

// cos(pi j / N) and sin(pi j / N), j = 0 .. 2N - 1
void conv_trig(int level, std::vector<double> &t) {
    const int N = (1 << level) / 2;
    t.resize(4 * (size_t)N);
    for (int j = 0; j < 2 * N; ++j) {
        // exact at the multiples of pi / 2 (the entries there decide zeros)
        const int q = 2 * j % N == 0 ? 2 * j / N : -1;
        t[j] = q == 0 ? 1.0 : q == 2 ? -1.0 : q >= 0 ? 0.0 : std::cos(M_PI * j / N);
        t[2 * N + j] = q == 1 ? 1.0 : q == 3 ? -1.0 : q >= 0 ? 0.0 : std::sin(M_PI * j / N);
    }
}

}  // namespace fmm
