// Direct Poisson solver by fast diagonalisation, in FP64 on the matrix cores.
//
// The zero-Dirichlet star operator is the Kronecker sum K = Kx + Ky + Kz of
// one-axis band matrices (Sec. II.A), so with K_d = Q_d Lam_d Q_d^T
//   x = (Qz Qy Qx) [ (Qx^T Qy^T Qz^T b) h^2 / (lam_x + lam_y + lam_z) ]
// solves K x = b exactly, up to FP64 rounding.  Each K_d commutes with the
// reflection of its axis: its eigenvectors are even or odd (fdm_basis.h), so
// a transform is a fold (sums and differences of mirrored nodes) followed by
// two products of half the size, n instead of 2 n flops per value and axis.
//
// What bounds it: the fused form moves 3 x 16 B per node (x-y forward, z with
// the scaling, x-y inverse) and does 2 (nx + ny + nz) flops per node on
// v_mfma_f64_16x16x4_f64; at 96^3 the two are level (16 B at 5.1 TB/s, 192
// flops at 72 TFLOP/s), longer axes are bound by the matrix cores.
//
// Layout of v_mfma_f64_16x16x4_f64 used throughout: with g = lane / 16 and
// c = lane % 16, operand A holds (row c, k g), B holds (k g, column c) and
// accumulator element r holds (row g + 4 r, column c).  Accumulator element
// r of row tile t is therefore already the B operand of k step 4 t + r, so
// a second product that contracts the first one's rows takes its operand
// straight from the accumulators, with no trip through LDS.
#include <algorithm>
#include <mutex>
#include <set>

#include "fdm_basis.h"
#include "kernels.h"

namespace fsic {

namespace {

typedef double dbl4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ dbl4 mfma(double a, double b, dbl4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// LDS row stride of an axis matrix with 16 T columns: operand reads whose
// row runs with c are free of bank conflicts, the others take two passes
template <int T>
constexpr int kStr = 16 * T + 2;

// One axis table (16 Ta x 16 Ta per parity, zero padded) to LDS, padded to
// 16 T: [parity][mode][position], or (TR) [parity][position][mode].
template <int T, bool TR>
__device__ __forceinline__ void load_table(double *dst, const double *tab, int Ta, int nthr) {
    constexpr int L = 16 * T, S = kStr<T>;
    const int La = 16 * Ta;
    for (int i = threadIdx.x; i < 2 * L * L; i += nthr) {
        const int par = i / (L * L), k = (i / L) % L, j = i % L;
        const double v = (k < La && j < La) ? tab[(size_t)(par * La + k) * La + j] : 0.0;
        dst[par * L * S + (TR ? j * S + k : k * S + j)] = v;
    }
}

// bank swizzle of a 16 T wide LDS row: the rows of one operand read (k = 4 s
// + g) alternate halves of the banks
template <int T>
__device__ __forceinline__ int swz(int row, int col) {
    return (T & 1) ? col : (col ^ ((row & 1) << 4));
}

}  // namespace

// ---------------------------------------------------------------------------
// fused in-plane passes (axes up to 128 nodes): one block per z plane, 2 T
// waves; wave (py, kt) or (py, xt) takes one y parity and one 16-column tile
// of the output.  The plane's four parity quadrants pass through LDS one x
// parity at a time, which halves the LDS and lets two blocks share a compute
// unit at T = 3 (axes of 65-96 nodes).
// ---------------------------------------------------------------------------

// waves per SIMD the registers have to leave room for: two blocks of six
// waves share a compute unit at T = 3
template <int T>
constexpr int kXyWaves = T == 3 ? 3 : 2;

// b -> in-plane spectral coefficients, written [z][kx][ky] (ky fastest, even
// modes before odd ones on both axes) so that the inverse pass reads whole
// rows in its operand layout.  SQ: b = scale src^2, else b = src.
template <int T, bool SQ>
__global__ __launch_bounds__(128 * T, kXyWaves<T>) void k_fdm_xy_fwd(const Item *units, const FdmRange *ranges,
                                                         const OrbDesc *orb, const int *done, const double *tab,
                                                         int two, const double *src, double scale, double *out) {
    constexpr int L = 16 * T, S = kStr<T>, NT = 128 * T, NQ = 2 * T;
    extern __shared__ __attribute__((aligned(16))) double fsm[];
    double *const Mx = fsm, *const My = two ? fsm + 2 * L * S : fsm;
    double *const X = fsm + (two ? 4 : 2) * L * S;  // [py][y][x]
    const FdmRange rg = ranges[blockIdx.x];
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, c = lane & 15;
    const int py = w / T, kt = w - py * T;
    {
        const OrbDesc &od = orb[units[rg.u0].orb];
        load_table<T, false>(Mx, tab + od.fd_t[0], od.fd_n[0], NT);
        if (two) load_table<T, false>(My, tab + od.fd_t[1], od.fd_n[1], NT);
    }
    auto next = [&](int u) {
        while (u < rg.u1 && done && done[units[u].orb]) ++u;
        return u;
    };
    const int xq = tid % L, yq0 = tid / L;  // fold quads (yq0 + 8 i, xq)
    double ra[NQ], rb[NQ], rc[NQ], rd[NQ];
    auto issue = [&](int u) {
        const Item it = units[u];
        const OrbDesc &od = orb[it.orb];
        const int nx = od.nx, ny = od.ny, hx = (nx + 1) >> 1, hy = (ny + 1) >> 1;
        const double *p = src + od.off + (long long)it.tile * nx * ny;
        const int x = min(xq, hx - 1), xm = nx - 1 - x;
#pragma unroll
        for (int i = 0; i < NQ; ++i) {
            const int y = min(yq0 + 8 * i, hy - 1), ym = ny - 1 - y;
            ra[i] = p[y * nx + x];
            rb[i] = p[y * nx + xm];
            rc[i] = p[ym * nx + x];
            rd[i] = p[ym * nx + xm];
        }
    };
    int u = next(rg.u0), last = -1;
    if (u < rg.u1) issue(u);
    while (u < rg.u1) {
        const Item it = units[u];
        const OrbDesc &od = orb[it.orb];
        const int nx = od.nx, ny = od.ny, hx = (nx + 1) >> 1, hy = (ny + 1) >> 1;
        const int ox = nx >> 1, oy = ny >> 1;
        const int ksx = (hx + 3) >> 2, ksy = (hy + 3) >> 2;
        if (it.orb != last) {  // nothing of another orbital stays in the padding
            for (int i = tid; i < 2 * L * L; i += NT) X[i] = 0.0;
            last = it.orb;
            __syncthreads();
        }
        // fold: a centre node enters once
        const bool xin = xq < hx, xmid = 2 * xq == nx - 1;
#pragma unroll
        for (int i = 0; i < NQ; ++i) {
            const int y = yq0 + 8 * i;
            const bool ymid = 2 * y == ny - 1;
            double a = ra[i], b = rb[i], cc = rc[i], d = rd[i];
            if (SQ) {
                a = scale * (a * a);
                b = scale * (b * b);
                cc = scale * (cc * cc);
                d = scale * (d * d);
            }
            if (xmid) b = d = 0.0;
            if (ymid) cc = d = 0.0;
            const double s1 = a + b, s2 = cc + d;
            ra[i] = a - b;
            rb[i] = cc - d;
            if (xin && y < hy) {
                const int q = y * L + swz<T>(y, xq);
                X[q] = s1 + s2;
                X[L * L + q] = s1 - s2;
            }
        }
        const int un = next(u + 1);
        double *const o = out + od.off + (long long)it.tile * nx * ny;
#pragma unroll 1
        for (int px = 0; px < 2; ++px) {
            if (px == 1) {
                lds_barrier();  // the even quadrants are read
#pragma unroll
                for (int i = 0; i < NQ; ++i) {
                    const int y = yq0 + 8 * i;
                    if (xin && y < hy) {
                        const int q = y * L + swz<T>(y, xq);
                        X[q] = ra[i] + rb[i];
                        X[L * L + q] = ra[i] - rb[i];
                    }
                }
                if (un < rg.u1) issue(un);
            }
            lds_barrier();
            const double *Xq = X + py * L * L, *By = My + py * L * S, *Ax = Mx + px * L * S;
            dbl4 D[T];
#pragma unroll
            for (int t = 0; t < T; ++t) D[t] = dbl4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int s = 0; s < 4 * T; ++s) {
                if (s >= 4 * (T - 1) && s >= ksy) continue;
                const double b = By[(16 * kt + c) * S + 4 * s + g];
#pragma unroll
                for (int t = 0; t < T; ++t) D[t] = mfma(Xq[(4 * s + g) * L + swz<T>(4 * s + g, 16 * t + c)], b, D[t]);
            }
            dbl4 E[T];
#pragma unroll
            for (int t = 0; t < T; ++t) E[t] = dbl4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int s = 0; s < 4 * T; ++s) {
                if (s >= 4 * (T - 1) && s >= ksx) continue;
#pragma unroll
                for (int t = 0; t < T; ++t) E[t] = mfma(Ax[(16 * t + c) * S + 4 * s + g], D[s >> 2][s & 3], E[t]);
            }
            const int ky = 16 * kt + c, kmax = px ? ox : hx;
            if (ky < (py ? oy : hy)) {
                double *q = o + (py ? hy : 0) + ky + (long long)(px ? hx : 0) * ny;
#pragma unroll
                for (int t = 0; t < T; ++t)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int kx = 16 * t + g + 4 * r;
                        if (kx < kmax) q[kx * ny] = E[t][r];
                    }
            }
        }
        lds_barrier();  // the odd quadrants are read
        u = un;
    }
}

// in-plane spectral coefficients [z][kx][ky] -> x (ACC: x += the result)
template <int T, bool ACC>
__global__ __launch_bounds__(128 * T, kXyWaves<T>) void k_fdm_xy_inv(const Item *units, const FdmRange *ranges,
                                                         const OrbDesc *orb, const int *done, const double *tab,
                                                         int two, const double *in, double *out) {
    constexpr int L = 16 * T, S = kStr<T>, NT = 128 * T, NR = 4 * T;
    extern __shared__ __attribute__((aligned(16))) double fsm[];
    double *const Mx = fsm, *const My = two ? fsm + 2 * L * S : fsm;
    double *const X = fsm + (two ? 4 : 2) * L * S;  // [py][kx][ky]; then the exchange tiles
    const FdmRange rg = ranges[blockIdx.x];
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, c = lane & 15;
    const int py = w / T, xt = w - py * T;
    {
        const OrbDesc &od = orb[units[rg.u0].orb];
        load_table<T, true>(Mx, tab + od.fd_t[0], od.fd_n[0], NT);
        if (two) load_table<T, true>(My, tab + od.fd_t[1], od.fd_n[1], NT);
    }
    auto next = [&](int u) {
        while (u < rg.u1 && done && done[units[u].orb]) ++u;
        return u;
    };
    // staging: two half rows (py) of L modes per row kx, 4 rows per sweep
    const int sj = tid % L, sp = (tid / L) & 1, sr = tid / (2 * L);
    double rv[NR];
    auto issue = [&](int u, int px) {
        const Item it = units[u];
        const OrbDesc &od = orb[it.orb];
        const int nx = od.nx, ny = od.ny, hx = (nx + 1) >> 1, hy = (ny + 1) >> 1;
        const double *p = in + od.off + (long long)it.tile * nx * ny + (long long)(px ? hx : 0) * ny;
        const int rows = px ? nx >> 1 : hx, cols = sp ? ny >> 1 : hy;
        const int col = min(sj, cols - 1) + (sp ? hy : 0);
#pragma unroll
        for (int i = 0; i < NR; ++i) rv[i] = p[min(sr + 4 * i, rows - 1) * ny + col];
    };
    auto stage = [&](const OrbDesc &od, int px) {
        const int hx = (od.nx + 1) >> 1, hy = (od.ny + 1) >> 1;
        const int rows = px ? od.nx >> 1 : hx, cols = sp ? od.ny >> 1 : hy;
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            const int k = sr + 4 * i;
            X[sp * L * L + k * L + swz<T>(k, sj)] = (k < rows && sj < cols) ? rv[i] : 0.0;
        }
    };
    int u = next(rg.u0);
    if (u < rg.u1) issue(u, 0);
    while (u < rg.u1) {
        const Item it = units[u];
        const OrbDesc &od = orb[it.orb];
        const int nx = od.nx, ny = od.ny, hx = (nx + 1) >> 1, hy = (ny + 1) >> 1;
        const int ox = nx >> 1, oy = ny >> 1;
        const int ksx = (hx + 3) >> 2, ksy = (hy + 3) >> 2;
        const int un = next(u + 1);
        dbl4 D[2][T];
#pragma unroll
        for (int px = 0; px < 2; ++px) {
            stage(od, px);
            if (px == 0) issue(u, 1);
            else if (un < rg.u1) issue(un, 0);
            lds_barrier();
            const double *Xq = X + py * L * L, *Bx = Mx + px * L * S;
#pragma unroll
            for (int t = 0; t < T; ++t) D[px][t] = dbl4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int s = 0; s < 4 * T; ++s) {
                if (s >= 4 * (T - 1) && s >= ksx) continue;
                const double b = Bx[(16 * xt + c) * S + 4 * s + g];
#pragma unroll
                for (int t = 0; t < T; ++t)
                    D[px][t] = mfma(Xq[(4 * s + g) * L + swz<T>(4 * s + g, 16 * t + c)], b, D[px][t]);
            }
            lds_barrier();  // X may be overwritten
        }
        // unfold x: columns x and nx-1-x
        dbl4 EL[T], ER[T];
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const dbl4 e = D[0][t], o = D[1][t];
            D[0][t] = e + o;
            D[1][t] = e - o;
            EL[t] = ER[t] = dbl4{0.0, 0.0, 0.0, 0.0};
        }
        const double *Ay = My + py * L * S;
#pragma unroll
        for (int s = 0; s < 4 * T; ++s) {
            if (s >= 4 * (T - 1) && s >= ksy) continue;
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const double a = Ay[(16 * t + c) * S + 4 * s + g];
                EL[t] = mfma(a, D[0][s >> 2][s & 3], EL[t]);
                ER[t] = mfma(a, D[1][s >> 2][s & 3], ER[t]);
            }
        }
        // the even-y wave finishes the left columns, the odd-y wave the right
        // ones: each hands the other half to its partner
        double *const mine = X + (size_t)(2 * xt + py) * T * 256, *const theirs = X + (size_t)(2 * xt + 1 - py) * T * 256;
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) mine[(4 * t + r) * 64 + lane] = py ? EL[t][r] : ER[t][r];
        lds_barrier();
        const int xl = 16 * xt + c;
        const bool xok = xl < (py ? ox : hx);
        double *const o = out + od.off + (long long)it.tile * nx * ny + (py ? nx - 1 - xl : xl);
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const double v = theirs[(4 * t + r) * 64 + lane];
                const double e = py ? v : EL[t][r], d = py ? ER[t][r] : v;
                const int y = 16 * t + g + 4 * r;
                if (xok && y < hy) {
                    const int i1 = y * nx, i2 = (ny - 1 - y) * nx;
                    if (ACC) {
                        o[i1] += e + d;
                        if (y < oy) o[i2] += e - d;
                    } else {
                        o[i1] = e + d;
                        if (y < oy) o[i2] = e - d;
                    }
                }
            }
        lds_barrier();  // the exchange tiles are read
        u = un;
    }
}

// ---------------------------------------------------------------------------
// one-axis passes in registers: a wave takes 16 lines of an axis (a line's
// nodes lie `stride` apart), folds them in registers and multiplies against
// the axis matrices in LDS.  No barrier and no LDS traffic for the data.
// ---------------------------------------------------------------------------

enum { kFdmZ = 0, kFdmYFwd = 1, kFdmYInv = 2, kFdmXFwd = 3, kFdmXInv = 4 };

template <int T>
constexpr int kFdmThreads = T <= 3 ? 256 : 512;

// lines as columns of the B operand (x or y-x neighbours contiguous):
//   kFdmZ: transform, scale by h^2 / (lam_x + lam_y + lam_z), transform back,
//          in place; lines: in-plane points;
//   kFdmYFwd / kFdmYInv: along y, lines (z, x).
template <int T, int MODE>
__global__ __launch_bounds__(kFdmThreads<T>) void k_fdm_col(const Item *units, const FdmRange *ranges,
                                                             const OrbDesc *orb, const int *done,
                                                             const double *tab, const double *in, double *out) {
    constexpr int L = 16 * T, S = kStr<T>, NT = kFdmThreads<T>, NW = NT / 64;
    constexpr int AX = MODE == kFdmZ ? 2 : 1;
    extern __shared__ __attribute__((aligned(16))) double fsm[];
    const FdmRange rg = ranges[blockIdx.x];
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = lane >> 4, c = lane & 15;
    {
        const OrbDesc &od = orb[units[rg.u0].orb];
        load_table<T, MODE != kFdmYFwd>(fsm, tab + od.fd_t[AX], od.fd_n[AX], NT);
    }
    __syncthreads();
    // mode 16 t + c, position 4 s + g (forward A operand); position 16 t + c,
    // mode 4 s + g (inverse A operand)
    auto F = [&](int par, int t, int s) {
        const double *M = fsm + par * L * S;
        return MODE == kFdmYFwd ? M[(16 * t + c) * S + 4 * s + g] : M[(4 * s + g) * S + 16 * t + c];
    };
    auto I = [&](int par, int t, int s) { return fsm[par * L * S + (16 * t + c) * S + 4 * s + g]; };
    const int nsub = 4 * (rg.u1 - rg.u0);
    for (int sub = w; sub < nsub; sub += NW) {
        const Item it = units[rg.u0 + (sub >> 2)];
        if (done && done[it.orb]) continue;  // uniform in the wave
        const OrbDesc &od = orb[it.orb];
        const int n = AX == 2 ? od.nz : od.ny, he = (n + 1) >> 1, ho = n >> 1, ks = (he + 3) >> 2;
        const int M2 = od.nx * od.ny;
        const int lines = AX == 2 ? M2 : od.nx * od.nz;
        const int l0 = it.tile * 64 + (sub & 3) * 16;
        if (l0 >= lines) continue;
        const int ln = min(l0 + c, lines - 1);
        const bool lok = l0 + c < lines;
        const int stride = AX == 2 ? M2 : od.nx;
        const long long base = od.off + (AX == 2 ? (long long)ln : (long long)(ln / od.nx) * M2 + ln % od.nx);
        const double *p = in + base;
        double *q = out + base;
        dbl4 Ce[T], Co[T];
        if (MODE == kFdmZ || MODE == kFdmYFwd) {
            double fe[4 * T], fo[4 * T];
#pragma unroll
            for (int s = 0; s < 4 * T; ++s) {
                const int j = min(4 * s + g, he - 1);
                fe[s] = p[(long long)j * stride];
                fo[s] = p[(long long)(n - 1 - j) * stride];
            }
#pragma unroll
            for (int s = 0; s < 4 * T; ++s) {
                const double a = fe[s], b = 2 * (4 * s + g) == n - 1 ? 0.0 : fo[s];
                fe[s] = a + b;
                fo[s] = a - b;
            }
#pragma unroll
            for (int t = 0; t < T; ++t) Ce[t] = Co[t] = dbl4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int s = 0; s < 4 * T; ++s) {
                if (s >= 4 * (T - 1) && s >= ks) continue;
#pragma unroll
                for (int t = 0; t < T; ++t) Ce[t] = mfma(F(0, t, s), fe[s], Ce[t]);
            }
#pragma unroll
            for (int s = 0; s < 4 * T; ++s) {
                if (s >= 4 * (T - 1) && s >= ks) continue;
#pragma unroll
                for (int t = 0; t < T; ++t) Co[t] = mfma(F(1, t, s), fo[s], Co[t]);
            }
        } else {
#pragma unroll
            for (int t = 0; t < T; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int k = 16 * t + g + 4 * r;
                    const double a = p[(long long)min(k, he - 1) * stride];
                    const double b = p[(long long)(he + max(min(k, ho - 1), 0)) * stride];
                    Ce[t][r] = k < he ? a : 0.0;
                    Co[t][r] = k < ho ? b : 0.0;
                }
        }
        if (MODE == kFdmYFwd) {
            if (lok) {
#pragma unroll
                for (int t = 0; t < T; ++t)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int k = 16 * t + g + 4 * r;
                        if (k < he) q[(long long)k * stride] = Ce[t][r];
                        if (k < ho) q[(long long)(he + k) * stride] = Co[t][r];
                    }
            }
            continue;
        }
        if (MODE == kFdmZ) {
            // spectral position of the line: the fused passes leave [kx][ky],
            // the one-axis passes [ky][kx]
            const int inner = od.fd_fused ? od.ny : od.nx;
            const int a = ln / inner, b = ln - a * inner;
            const int kx = od.fd_fused ? a : b, ky = od.fd_fused ? b : a;
            auto lam = [&](int d, int nd, int k) {
                const int Ld = 16 * od.fd_n[d], hd = (nd + 1) >> 1;
                return tab[od.fd_t[d] + 2 * Ld * Ld + (k < hd ? k : Ld + k - hd)];
            };
            const double lxy = lam(0, od.nx, kx) + lam(1, od.ny, ky);
            const double h2 = od.h * od.h;
            const int Lz = 16 * od.fd_n[2];
            const double *lz = tab + od.fd_t[2] + 2 * Lz * Lz;
#pragma unroll
            for (int t = 0; t < T; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int k = 16 * t + g + 4 * r;
                    Ce[t][r] *= h2 / (lz[k] + lxy);
                    Co[t][r] *= h2 / (lz[Lz + k] + lxy);
                }
        }
        // back to nodes, one 16-position tile at a time
#pragma unroll
        for (int t = 0; t < T; ++t) {
            dbl4 E = {0.0, 0.0, 0.0, 0.0}, O = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int s = 0; s < 4 * T; ++s) {
                if (s >= 4 * (T - 1) && s >= ks) continue;
                E = mfma(I(0, t, s), Ce[s >> 2][s & 3], E);
                O = mfma(I(1, t, s), Co[s >> 2][s & 3], O);
            }
            if (lok) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int j = 16 * t + g + 4 * r;
                    if (j < he) q[(long long)j * stride] = E[r] + O[r];
                    if (j < ho) q[(long long)(n - 1 - j) * stride] = E[r] - O[r];
                }
            }
        }
    }
}

// lines along x (contiguous), as rows of the A operand; lines (z, y)
//   SQ (forward): b = scale src^2;  ACC (inverse): x += the result
template <int T, int MODE, bool SQ, bool ACC>
__global__ __launch_bounds__(kFdmThreads<T>) void k_fdm_row(const Item *units, const FdmRange *ranges,
                                                             const OrbDesc *orb, const int *done,
                                                             const double *tab, const double *in, double scale,
                                                             double *out) {
    constexpr int L = 16 * T, S = kStr<T>, NT = kFdmThreads<T>, NW = NT / 64;
    extern __shared__ __attribute__((aligned(16))) double fsm[];
    const FdmRange rg = ranges[blockIdx.x];
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = lane >> 4, c = lane & 15;
    {
        const OrbDesc &od = orb[units[rg.u0].orb];
        load_table<T, MODE == kFdmXInv>(fsm, tab + od.fd_t[0], od.fd_n[0], NT);
    }
    __syncthreads();
    auto Bop = [&](int par, int t, int s) { return fsm[par * L * S + (16 * t + c) * S + 4 * s + g]; };
    const int nsub = 4 * (rg.u1 - rg.u0);
    for (int sub = w; sub < nsub; sub += NW) {
        const Item it = units[rg.u0 + (sub >> 2)];
        if (done && done[it.orb]) continue;
        const OrbDesc &od = orb[it.orb];
        const int n = od.nx, he = (n + 1) >> 1, ho = n >> 1, ks = (he + 3) >> 2;
        const int lines = od.ny * od.nz;
        const int l0 = it.tile * 64 + (sub & 3) * 16;
        if (l0 >= lines) continue;
        const double *p = in + od.off + (long long)min(l0 + c, lines - 1) * n;
        double *q = out + od.off;
        double fe[4 * T], fo[4 * T];
#pragma unroll
        for (int s = 0; s < 4 * T; ++s) {
            const int k = 4 * s + g;
            if (MODE == kFdmXFwd) {
                const int j = min(k, he - 1);
                fe[s] = p[j];
                fo[s] = p[n - 1 - j];
            } else {
                fe[s] = p[min(k, he - 1)];
                fo[s] = p[he + max(min(k, ho - 1), 0)];
            }
        }
#pragma unroll
        for (int s = 0; s < 4 * T; ++s) {
            const int k = 4 * s + g;
            if (MODE == kFdmXFwd) {
                double a = fe[s], b = fo[s];
                if (SQ) {
                    a = scale * (a * a);
                    b = scale * (b * b);
                }
                if (2 * k == n - 1) b = 0.0;
                fe[s] = a + b;
                fo[s] = a - b;
            } else {
                fe[s] = k < he ? fe[s] : 0.0;
                fo[s] = k < ho ? fo[s] : 0.0;
            }
        }
#pragma unroll
        for (int t = 0; t < T; ++t) {
            dbl4 E = {0.0, 0.0, 0.0, 0.0}, O = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int s = 0; s < 4 * T; ++s) {
                if (s >= 4 * (T - 1) && s >= ks) continue;
                E = mfma(fe[s], Bop(0, t, s), E);
                O = mfma(fo[s], Bop(1, t, s), O);
            }
            const int j = 16 * t + c;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = l0 + g + 4 * r;
                if (row >= lines) continue;
                double *o = q + (long long)row * n;
                if (MODE == kFdmXFwd) {
                    if (j < he) o[j] = E[r];
                    if (j < ho) o[he + j] = O[r];
                } else if (ACC) {
                    if (j < he) o[j] += E[r] + O[r];
                    if (j < ho) o[n - 1 - j] += E[r] - O[r];
                } else {
                    if (j < he) o[j] = E[r] + O[r];
                    if (j < ho) o[n - 1 - j] = E[r] - O[r];
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------
// launches
// ---------------------------------------------------------------------------

namespace {

size_t xy_lds(int T, bool two) {
    const size_t L = 16 * (size_t)T, S = L + 2;
    return ((two ? 4 : 2) * L * S + 2 * L * L) * sizeof(double);
}
size_t line_lds(int T) {
    const size_t L = 16 * (size_t)T, S = L + 2;
    return 2 * L * S * sizeof(double);
}

template <class K>
hipError_t allow_lds(K k, size_t lds) {
    return hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
}

// blocks of a kernel that one compute unit holds
template <class K>
int occ_of(K k, int threads, size_t lds) {
    int n = 0;
    if (allow_lds(k, lds) != hipSuccess) return 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, reinterpret_cast<const void *>(k), threads, lds) != hipSuccess)
        return 0;
    return n;
}

}  // namespace

bool fdm_xy_fits(int nx, int ny, size_t lds_limit) {
    const int T = std::max(fdm_tiles(nx), fdm_tiles(ny));
    return T <= 4 && xy_lds(T, nx != ny) <= lds_limit;
}

int fdm_occupancy(int pass, int T, int two) {
#define XY(TT) case TT: return std::min(occ_of(k_fdm_xy_fwd<TT, true>, 128 * TT, xy_lds(TT, two != 0)), \
                                        occ_of(k_fdm_xy_inv<TT, false>, 128 * TT, xy_lds(TT, two != 0)));
#define Z(TT) case TT: return occ_of(k_fdm_col<TT, kFdmZ>, kFdmThreads<TT>, line_lds(TT));
#define XL(TT) case TT: return occ_of(k_fdm_row<TT, kFdmXFwd, true, false>, kFdmThreads<TT>, line_lds(TT));
#define YL(TT) case TT: return occ_of(k_fdm_col<TT, kFdmYFwd>, kFdmThreads<TT>, line_lds(TT));
    if (pass == kFdmPassXY) {
        switch (T) { XY(1) XY(2) XY(3) XY(4) }
    } else if (pass == kFdmPassZ) {
        switch (T) { Z(1) Z(2) Z(3) Z(4) Z(5) Z(6) }
    } else if (pass == kFdmPassX) {
        switch (T) { XL(1) XL(2) XL(3) XL(4) XL(5) XL(6) }
    } else {
        switch (T) { YL(1) YL(2) YL(3) YL(4) YL(5) YL(6) }
    }
#undef XY
#undef Z
#undef XL
#undef YL
    return 0;
}

hipError_t fdm_setup() {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    static std::mutex mu;
    static std::set<int> ready;
    std::lock_guard<std::mutex> lk(mu);
    if (ready.count(dev)) return hipSuccess;
    auto set = [&](auto k, size_t lds) {
        if (e == hipSuccess) e = allow_lds(k, lds);
    };
#define XY(TT)                                                                  \
    set(k_fdm_xy_fwd<TT, true>, std::min<size_t>(xy_lds(TT, true), 160 * 1024));  \
    set(k_fdm_xy_fwd<TT, false>, std::min<size_t>(xy_lds(TT, true), 160 * 1024)); \
    set(k_fdm_xy_inv<TT, true>, std::min<size_t>(xy_lds(TT, true), 160 * 1024));  \
    set(k_fdm_xy_inv<TT, false>, std::min<size_t>(xy_lds(TT, true), 160 * 1024));
    XY(1) XY(2) XY(3) XY(4)
#undef XY
#define LN(TT)                                                 \
    set(k_fdm_col<TT, kFdmZ>, line_lds(TT));             \
    set(k_fdm_col<TT, kFdmYFwd>, line_lds(TT));          \
    set(k_fdm_col<TT, kFdmYInv>, line_lds(TT));          \
    set(k_fdm_row<TT, kFdmXFwd, true, false>, line_lds(TT));    \
    set(k_fdm_row<TT, kFdmXFwd, false, false>, line_lds(TT));   \
    set(k_fdm_row<TT, kFdmXInv, false, true>, line_lds(TT));    \
    set(k_fdm_row<TT, kFdmXInv, false, false>, line_lds(TT));
    LN(1) LN(2) LN(3) LN(4) LN(5) LN(6)
#undef LN
    if (e == hipSuccess) ready.insert(dev);
    return e;
}

hipError_t launch_fdm(const FdmPlan &p, const OrbDesc *orb, const int *done, const double *tab, const double *src,
                      int square, double scale, double *work, double *out, int accumulate, hipStream_t s) {
    const FdmClass *const cl = p.cls;
    auto each = [&](int pass, auto &&f) -> hipError_t {
        for (int i = 0; i < p.ncls; ++i) {
            if (cl[i].pass != pass || cl[i].blocks <= 0) continue;
            const hipError_t e = f(cl[i]);
            if (e != hipSuccess) return e;
            const hipError_t l = hipGetLastError();
            if (l != hipSuccess) return l;
        }
        return hipSuccess;
    };
#define GO(K, THR, LDS, ...) hipLaunchKernelGGL((K), dim3(q.blocks), dim3(THR), LDS, s, p.units[pass], p.ranges + q.range0, orb, done, tab, __VA_ARGS__)
    int pass = kFdmPassXY;
    hipError_t e = each(pass, [&](const FdmClass &q) -> hipError_t {
#define XY(TT)                                                                                              \
    case TT:                                                                                                \
        if (square) GO((k_fdm_xy_fwd<TT, true>), 128 * TT, xy_lds(TT, q.two), q.two, src, scale, work);       \
        else GO((k_fdm_xy_fwd<TT, false>), 128 * TT, xy_lds(TT, q.two), q.two, src, scale, work);             \
        return hipSuccess;
        switch (q.T) { XY(1) XY(2) XY(3) XY(4) }
#undef XY
        return hipErrorInvalidValue;
    });
    if (e != hipSuccess) return e;
    pass = kFdmPassX;
    e = each(pass, [&](const FdmClass &q) -> hipError_t {
#define LN(TT)                                                                                                        \
    case TT:                                                                                                          \
        if (square) GO((k_fdm_row<TT, kFdmXFwd, true, false>), kFdmThreads<TT>, line_lds(TT), src, scale, work);        \
        else GO((k_fdm_row<TT, kFdmXFwd, false, false>), kFdmThreads<TT>, line_lds(TT), src, scale, work);              \
        return hipSuccess;
        switch (q.T) { LN(1) LN(2) LN(3) LN(4) LN(5) LN(6) }
#undef LN
        return hipErrorInvalidValue;
    });
    if (e != hipSuccess) return e;
#define COL(TT, MODE)                                                                                   \
    case TT:                                                                                            \
        GO((k_fdm_col<TT, MODE>), kFdmThreads<TT>, line_lds(TT), (const double *)work, work);      \
        return hipSuccess;
    pass = kFdmPassY;
    e = each(pass, [&](const FdmClass &q) -> hipError_t {
        switch (q.T) { COL(1, kFdmYFwd) COL(2, kFdmYFwd) COL(3, kFdmYFwd) COL(4, kFdmYFwd) COL(5, kFdmYFwd) COL(6, kFdmYFwd) }
        return hipErrorInvalidValue;
    });
    if (e != hipSuccess) return e;
    pass = kFdmPassZ;
    e = each(pass, [&](const FdmClass &q) -> hipError_t {
        switch (q.T) { COL(1, kFdmZ) COL(2, kFdmZ) COL(3, kFdmZ) COL(4, kFdmZ) COL(5, kFdmZ) COL(6, kFdmZ) }
        return hipErrorInvalidValue;
    });
    if (e != hipSuccess) return e;
    pass = kFdmPassY;
    e = each(pass, [&](const FdmClass &q) -> hipError_t {
        switch (q.T) { COL(1, kFdmYInv) COL(2, kFdmYInv) COL(3, kFdmYInv) COL(4, kFdmYInv) COL(5, kFdmYInv) COL(6, kFdmYInv) }
        return hipErrorInvalidValue;
    });
    if (e != hipSuccess) return e;
#undef COL
    pass = kFdmPassX;
    e = each(pass, [&](const FdmClass &q) -> hipError_t {
#define LN(TT)                                                                                                         \
    case TT:                                                                                                           \
        if (accumulate) GO((k_fdm_row<TT, kFdmXInv, false, true>), kFdmThreads<TT>, line_lds(TT), (const double *)work, 1.0, out); \
        else GO((k_fdm_row<TT, kFdmXInv, false, false>), kFdmThreads<TT>, line_lds(TT), (const double *)work, 1.0, out);           \
        return hipSuccess;
        switch (q.T) { LN(1) LN(2) LN(3) LN(4) LN(5) LN(6) }
#undef LN
        return hipErrorInvalidValue;
    });
    if (e != hipSuccess) return e;
    pass = kFdmPassXY;
    return each(pass, [&](const FdmClass &q) -> hipError_t {
#define XY(TT)                                                                                                     \
    case TT:                                                                                                       \
        if (accumulate) GO((k_fdm_xy_inv<TT, true>), 128 * TT, xy_lds(TT, q.two), q.two, (const double *)work, out); \
        else GO((k_fdm_xy_inv<TT, false>), 128 * TT, xy_lds(TT, q.two), q.two, (const double *)work, out);           \
        return hipSuccess;
        switch (q.T) { XY(1) XY(2) XY(3) XY(4) }
#undef XY
        return hipErrorInvalidValue;
    });
#undef GO
}

}  // namespace fsic
