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

#include <algorithm>
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

// The even (par 0) or odd (par 1) half of an axis table; c[0 .. p]:
// second-difference weights on unit spacing.
inline void fdm_axis_parity(int n, int p, const double *c, int par, double *tab) {
    typedef long double ld;
    const int L = 16 * fdm_tiles(n);
    const ld pi = 3.141592653589793238462643383279502884L, r2 = sqrtl(2.0L);
    const int h = par == 0 ? (n + 1) / 2 : n / 2;
    const int mid = (par == 0 && (n & 1)) ? h - 1 : -1;
    if (h == 0) return;
    // the parity block of K in the orthonormal basis (e_j +- e_{n-1-j}) / sqrt 2
    // (e_mid alone), by columns: its few nonzero entries
    auto K = [&](int i, int j) -> ld {
        const int d = i > j ? i - j : j - i;
        return d <= p ? -(ld)c[d] : 0.0L;
    };
    std::vector<std::vector<std::pair<int, ld>>> col(h);
    for (int j = 0; j < h; ++j)
        for (int i = 0; i < h; ++i) {
            ld v;
            if (i == mid && j == mid) v = K(i, j);
            else if (i == mid || j == mid) v = r2 * K(i, j);
            else v = par == 0 ? K(i, j) + K(i, n - 1 - j) : K(i, j) - K(i, n - 1 - j);
            if (v != 0.0L) col[j].push_back({i, v});
        }
    auto dot = [&](const double *f, const double *g) {
        double s = 0.0;
        for (int q = 0; q < h; ++q) s += f[q] * g[q];
        return s;
    };
    // rows of V: the type-I sines of that parity, which make the block nearly
    // diagonal already (A = V K V^T), then eigenvectors by cyclic Jacobi in
    // FP64; A stays symmetric, so a rotation forms rows i and j and stores them
    // as columns too.  (In extended precision the rotations took 12 ms for a
    // 96-node axis and 96 ms for a 192-node one, in a program's first call.)
    std::vector<double> V((size_t)h * h), W((size_t)h * h), A((size_t)h * h);
    const ld sn = sqrtl(2.0L / (n + 1));
    std::vector<ld> sine(2 * (size_t)(n + 1));
    for (int a = 0; a < 2 * (n + 1); ++a) sine[a] = sinl(pi * (ld)a / (ld)(n + 1));
    for (int k = 0; k < h; ++k)
        for (int j = 0; j < h; ++j)
            V[(size_t)k * h + j] = (double)((j == mid ? sn : sn * r2) * sine[((long long)(2 * k + par + 1) * (j + 1)) % (2 * (n + 1))]);
    for (int k = 0; k < h; ++k)
        for (int j = 0; j < h; ++j) {
            double s = 0.0;
            for (const auto &e : col[j]) s += V[(size_t)k * h + e.first] * (double)e.second;
            W[(size_t)k * h + j] = s;
        }
    for (int k = 0; k < h; ++k)
        for (int l = 0; l <= k; ++l) A[(size_t)k * h + l] = A[(size_t)l * h + k] = dot(&W[(size_t)k * h], &V[(size_t)l * h]);
    for (int sweep = 0; sweep < 40; ++sweep) {
        bool any = false;
        for (int i = 0; i + 1 < h; ++i)
            for (int j = i + 1; j < h; ++j) {
                double *const Ai = &A[(size_t)i * h], *const Aj = &A[(size_t)j * h];
                const double aij = Ai[j], aii = Ai[i], ajj = Aj[j];
                if (std::fabs(aij) <= 1e-14 * std::sqrt(std::fabs(aii * ajj))) continue;
                any = true;
                const double th = (ajj - aii) / (2 * aij);
                const double t = (th >= 0 ? 1 : -1) / (std::fabs(th) + std::sqrt(1 + th * th));
                const double cs = 1 / std::sqrt(1 + t * t), ss = t * cs;
                double *const Vi = &V[(size_t)i * h], *const Vj = &V[(size_t)j * h];
                for (int q = 0; q < h; ++q) {
                    const double x = Ai[q], y = Aj[q], u = Vi[q], v = Vj[q];
                    Ai[q] = cs * x - ss * y;
                    Aj[q] = ss * x + cs * y;
                    Vi[q] = cs * u - ss * v;
                    Vj[q] = ss * u + cs * v;
                }
                Ai[i] = aii - t * aij;
                Aj[j] = ajj + t * aij;
                Ai[j] = Aj[i] = 0;
                for (int q = 0; q < h; ++q) {
                    A[(size_t)q * h + i] = Ai[q];
                    A[(size_t)q * h + j] = Aj[q];
                }
            }
        if (!any) break;
    }
    // One step of the refinement of Ogita and Aishima (2018): with the residual
    // r_k = K v_k - lam_k v_k of each FP64 eigenvector formed in extended
    // precision, V += C V, C_kl = r_k . v_l / (lam_k - lam_l),
    // C_kk = (1 - v_k . v_k) / 2, takes the error (1e-14 over the eigenvalues'
    // gaps) to its square.
    std::vector<ld> lam(h), x(h), y(h);
    for (int k = 0; k < h; ++k) {
        ld xy = 0, xx = 0;
        for (int q = 0; q < h; ++q) x[q] = V[(size_t)k * h + q];
        for (int q = 0; q < h; ++q) {
            y[q] = 0;
            for (const auto &e : col[q]) y[q] += x[e.first] * e.second;
            xy += x[q] * y[q];
            xx += x[q] * x[q];
        }
        lam[k] = xy / xx;
        for (int q = 0; q < h; ++q) W[(size_t)k * h + q] = (double)(y[q] - lam[k] * x[q]);
        A[(size_t)k * h + k] = (double)((1 - xx) / 2);
    }
    for (int k = 0; k < h; ++k)
        for (int l = 0; l < h; ++l)
            if (l != k) A[(size_t)k * h + l] = dot(&W[(size_t)k * h], &V[(size_t)l * h]) / (double)(lam[k] - lam[l]);
    std::fill(W.begin(), W.end(), 0.0);
    for (int k = 0; k < h; ++k)
        for (int l = 0; l < h; ++l)
            for (int j = 0; j < h; ++j) W[(size_t)k * h + j] += A[(size_t)k * h + l] * V[(size_t)l * h + j];
    for (int k = 0; k < h; ++k) {
        tab[(size_t)2 * L * L + (size_t)par * L + k] = (double)lam[k];
        for (int j = 0; j < h; ++j) {
            const ld v = (ld)V[(size_t)k * h + j] + (ld)W[(size_t)k * h + j];
            tab[((size_t)par * L + k) * L + j] = (double)(j == mid ? v : v / r2);
        }
    }
}

inline std::vector<double> fdm_axis_table(int n, int p, const double *c) {
    const int L = 16 * fdm_tiles(n);
    std::vector<double> tab((size_t)fdm_table_doubles(n), 0.0);
    for (int q = 2 * L * L; q < 2 * L * L + 2 * L; ++q) tab[q] = 1.0;
    for (int par = 0; par < 2; ++par) fdm_axis_parity(n, p, c, par, tab.data());
    return tab;
}

// The table of (n, p), made once per process (a 96-node axis takes 3 ms, a
// 192-node one 27 ms) and never dropped: a batch may hold any number of axis
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
