// Host tables of the direct Poisson solver (fdm.hip): eigenvectors of the
// one-axis second-difference matrix, split by reflection parity.
//
// K (n x n) is the symmetric band matrix -c_|i-j| (|i - j| <= p, zero
// Dirichlet values outside).  It commutes with the reflection j -> n-1-j, so
// its eigenvectors are even or odd; each parity block is diagonalised on its
// own.  Block e (o) has ceil(n/2) (floor(n/2)) modes and as many positions
// j = 0 .. ; the table entry C[k][j] is component j of the normalised
// eigenvector k of the full matrix, so that
//   transform   y_k = sum_j C[k][j] (x_j +- x_{n-1-j})   (centre node once),
//   inverse     x_j = sum_k Ce[k][j] y^e_k + sum_k Co[k][j] y^o_k,
//               x_{n-1-j} = the same with a minus.
#pragma once

#include <cmath>
#include <map>
#include <mutex>
#include <utility>
#include <vector>

namespace fsic {

// 16-row matrix-core tiles of an axis's parity block
inline int fdm_tiles(int n) { return ((n + 1) / 2 + 15) / 16; }
// doubles of an axis table: C[2][16 T][16 T] (parity, mode, position; zero
// padded), lambda[2][16 T] (padded with 1)
inline int fdm_table_doubles(int n) {
    const int L = 16 * fdm_tiles(n);
    return 2 * L * L + 2 * L;
}

// c[0 .. p]: second-difference weights on unit spacing.
inline std::vector<double> fdm_axis_table(int n, int p, const double *c) {
    typedef long double ld;
    const int L = 16 * fdm_tiles(n);
    std::vector<double> tab((size_t)fdm_table_doubles(n), 0.0);
    for (int q = 2 * L * L; q < 2 * L * L + 2 * L; ++q) tab[q] = 1.0;
    auto K = [&](int i, int j) -> ld {
        const int d = i > j ? i - j : j - i;
        return d <= p ? -(ld)c[d] : 0.0L;
    };
    const ld pi = 3.141592653589793238462643383279502884L, r2 = sqrtl(2.0L);
    for (int par = 0; par < 2; ++par) {
        const int h = par == 0 ? (n + 1) / 2 : n / 2;
        const int mid = (par == 0 && (n & 1)) ? h - 1 : -1;
        if (h == 0) continue;
        // parity block in the orthonormal basis (e_j +- e_{n-1-j}) / sqrt 2
        // (e_mid alone), then in the basis of the type-I sines of that parity,
        // which is nearly diagonal already
        std::vector<ld> A((size_t)h * h), V((size_t)h * h), W((size_t)h * h);
        for (int i = 0; i < h; ++i)
            for (int j = 0; j < h; ++j) {
                ld v;
                if (i == mid && j == mid) v = K(i, j);
                else if (i == mid || j == mid) v = r2 * K(i, j);
                else v = par == 0 ? K(i, j) + K(i, n - 1 - j) : K(i, j) - K(i, n - 1 - j);
                A[(size_t)i * h + j] = v;
            }
        const ld sn = sqrtl(2.0L / (n + 1));
        for (int k = 0; k < h; ++k)
            for (int j = 0; j < h; ++j) {
                const long long a = ((long long)(2 * k + par + 1) * (j + 1)) % (2LL * (n + 1));
                V[(size_t)k * h + j] = (j == mid ? sn : sn * r2) * sinl(pi * (ld)a / (ld)(n + 1));
            }
        for (int k = 0; k < h; ++k)  // W = V A
            for (int j = 0; j < h; ++j) {
                ld s = 0;
                for (int i = 0; i < h; ++i) s += V[(size_t)k * h + i] * A[(size_t)i * h + j];
                W[(size_t)k * h + j] = s;
            }
        for (int k = 0; k < h; ++k)  // A = W V^T
            for (int l = 0; l <= k; ++l) {
                ld s = 0;
                for (int i = 0; i < h; ++i) s += W[(size_t)k * h + i] * V[(size_t)l * h + i];
                A[(size_t)k * h + l] = A[(size_t)l * h + k] = s;
            }
        // cyclic Jacobi, rows of V rotated along
        for (int sweep = 0; sweep < 40; ++sweep) {
            bool any = false;
            for (int i = 0; i + 1 < h; ++i)
                for (int j = i + 1; j < h; ++j) {
                    const ld aij = A[(size_t)i * h + j], aii = A[(size_t)i * h + i], ajj = A[(size_t)j * h + j];
                    if (fabsl(aij) <= 1e-19L * sqrtl(fabsl(aii * ajj))) continue;
                    any = true;
                    const ld th = (ajj - aii) / (2 * aij);
                    const ld t = (th >= 0 ? 1 : -1) / (fabsl(th) + sqrtl(1 + th * th));
                    const ld cs = 1 / sqrtl(1 + t * t), ss = t * cs;
                    for (int q = 0; q < h; ++q) {  // rows i, j
                        const ld x = A[(size_t)i * h + q], y = A[(size_t)j * h + q];
                        A[(size_t)i * h + q] = cs * x - ss * y;
                        A[(size_t)j * h + q] = ss * x + cs * y;
                    }
                    for (int q = 0; q < h; ++q) {  // columns i, j
                        const ld x = A[(size_t)q * h + i], y = A[(size_t)q * h + j];
                        A[(size_t)q * h + i] = cs * x - ss * y;
                        A[(size_t)q * h + j] = ss * x + cs * y;
                    }
                    A[(size_t)i * h + j] = A[(size_t)j * h + i] = 0;
                    for (int q = 0; q < h; ++q) {
                        const ld x = V[(size_t)i * h + q], y = V[(size_t)j * h + q];
                        V[(size_t)i * h + q] = cs * x - ss * y;
                        V[(size_t)j * h + q] = ss * x + cs * y;
                    }
                }
            if (!any) break;
        }
        for (int k = 0; k < h; ++k) {
            tab[(size_t)2 * L * L + (size_t)par * L + k] = (double)A[(size_t)k * h + k];
            for (int j = 0; j < h; ++j)
                tab[((size_t)par * L + k) * L + j] = (double)(j == mid ? V[(size_t)k * h + j] : V[(size_t)k * h + j] / r2);
        }
    }
    return tab;
}

// The table of (n, p), made once per process (a 96-node axis takes 12 ms, a
// 192-node one 96 ms) and never dropped: a batch may hold any number of axis
// lengths, and rebuilding those past a limit would cost that time in every
// call.  n <= 192 bounds them to 12 MB per order.
inline const std::vector<double> &fdm_axis(int n, int p, const double *c) {
    static std::mutex mu;
    static std::map<std::pair<int, int>, std::vector<double>> tables;
    std::lock_guard<std::mutex> lk(mu);
    auto f = tables.find({n, p});
    if (f == tables.end()) f = tables.emplace(std::make_pair(n, p), fdm_axis_table(n, p, c)).first;
    return f->second;
}

}  // namespace fsic
