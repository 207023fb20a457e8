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
// An FP64 matrix product holds a SIMD's vector unit for 64 cycles, so what a
// wave does beside them adds to the time, and memory has to be under way
// during them.  Hence: descriptors through __restrict__ pointers and
// readfirstlane (scalar loads, uniform buffer resources; as vector loads each
// of them waited for all stores before it), raw buffer loads of the next unit
// issued as soon as registers are free, and stores that are never predicated
// (positions outside are dropped by the buffer's bounds).  Against plain
// pointers, 32 orbitals at 96^3: z pass 148 -> 128 us, in-plane pair
// 375 -> 357 us; 64 at 128^3: 765 -> 660 us, 1630 -> 1530 us.
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
#include "lds.h"
#include "buffer.h"

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
// waves share a compute unit at T = 3 (168 registers; the forward pass spills
// 12 B a lane, 20 B where it squares the orbital)
template <int T>
constexpr int kXyWaves = T == 3 ? 3 : 2;

// b -> in-plane spectral coefficients, written [z][kx][ky] (ky fastest, even
// modes before odd ones on both axes) so that the inverse pass reads whole
// rows in its operand layout.  SQ: b = scale src^2, else b = src.
template <int T, bool SQ>
__global__ __launch_bounds__(128 * T, kXyWaves<T>) void k_fdm_xy_fwd(const Item *__restrict__ units, const FdmRange *__restrict__ ranges,
                                                         const OrbDesc *__restrict__ orb, const int *__restrict__ done, const double *__restrict__ tab,
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
        while (u < rg.u1 && done && uni(done[units[u].orb])) ++u;
        return u;
    };
    const int xq = tid % L, yq0 = tid / L;  // fold quads (yq0 + 8 i, xq)
    double ra[NQ], rb[NQ], rc[NQ], rd[NQ];
    // half of a plane's loads: rows y (h 0) or their mirror rows (h 1)
    auto issue = [&](int u, int h) {
        const Item it = units[u];
        const OrbDesc &od = orb[uni(it.orb)];
        const int nx = uni(od.nx), ny = uni(od.ny), hx = (nx + 1) >> 1, hy = (ny + 1) >> 1;
        const Rsrc r = make_rsrc(src + uni(od.off) + (long long)uni(it.tile) * nx * ny, (unsigned)(nx * ny) * 8u);
        const int x = min(xq, hx - 1), xm = nx - 1 - x;
#pragma unroll
        for (int i = 0; i < NQ; ++i) {
            const int y = min(yq0 + 8 * i, hy - 1);
            if (h == 0) {
                ra[i] = bld<double>(r, (unsigned)(y * nx + x), 0);
                rb[i] = bld<double>(r, (unsigned)(y * nx + xm), 0);
            } else {
                rc[i] = bld<double>(r, (unsigned)((ny - 1 - y) * nx + x), 0);
                rd[i] = bld<double>(r, (unsigned)((ny - 1 - y) * nx + xm), 0);
            }
        }
    };
    int u = next(rg.u0), last = -1;
    if (u < rg.u1) {
        issue(u, 1);
        issue(u, 0);
    }
    while (u < rg.u1) {
        const Item it = units[u];
        const int oi = uni(it.orb);
        const OrbDesc &od = orb[oi];
        const int nx = uni(od.nx), ny = uni(od.ny), hx = (nx + 1) >> 1, hy = (ny + 1) >> 1;
        const int ox = nx >> 1, oy = ny >> 1;
        const int ksx = (hx + 3) >> 2, ksy = (hy + 3) >> 2;
        if (oi != last) {  // nothing of another orbital stays in the padding
            for (int i = tid; i < 2 * L * L; i += NT) X[i] = 0.0;
            last = oi;
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
        const Rsrc ro = make_rsrc(out + uni(od.off) + (long long)uni(it.tile) * nx * ny, (unsigned)(nx * ny) * 8u);
        // the next plane's loads go out in halves, as their registers come free:
        // blocks run in step, and one burst a plane would wait for the memory
        if (un < rg.u1) issue(un, 1);
#pragma unroll
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
                if (un < rg.u1) issue(un, 0);
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
            const bool kyok = ky < (py ? oy : hy);
            const int q = (py ? hy : 0) + ky + (px ? hx : 0) * ny;
#pragma unroll
            for (int t = 0; t < T; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int kx = 16 * t + g + 4 * r;
                    bst(ro, kyok && kx < kmax ? (unsigned)(q + kx * ny) : kDrop, 0, E[t][r]);
                }
        }
        lds_barrier();  // the odd quadrants are read
        u = un;
    }
}

// in-plane spectral coefficients [z][kx][ky] -> x
template <int T>
__global__ __launch_bounds__(128 * T, kXyWaves<T>) void k_fdm_xy_inv(const Item *__restrict__ units, const FdmRange *__restrict__ ranges,
                                                         const OrbDesc *__restrict__ orb, const int *__restrict__ done, const double *__restrict__ tab,
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
        while (u < rg.u1 && done && uni(done[units[u].orb])) ++u;
        return u;
    };
    // staging: two half rows (py) of L modes per row kx, 4 rows per sweep
    const int sj = tid % L, sp = (tid / L) & 1, sr = tid / (2 * L);
    double rv[NR];
    auto issue = [&](int u, int px) {
        const Item it = units[u];
        const OrbDesc &od = orb[uni(it.orb)];
        const int nx = uni(od.nx), ny = uni(od.ny), hx = (nx + 1) >> 1, hy = (ny + 1) >> 1;
        const Rsrc r = make_rsrc(in + uni(od.off) + (long long)uni(it.tile) * nx * ny, (unsigned)(nx * ny) * 8u);
        const int rows = px ? nx >> 1 : hx, cols = sp ? ny >> 1 : hy;
        const int col = min(sj, cols - 1) + (sp ? hy : 0), row0 = px ? hx : 0;
#pragma unroll
        for (int i = 0; i < NR; ++i) rv[i] = bld<double>(r, (unsigned)((row0 + min(sr + 4 * i, rows - 1)) * ny + col), 0);
    };
    auto stage = [&](int nx, int ny, int px) {
        const int hx = (nx + 1) >> 1, hy = (ny + 1) >> 1;
        const int rows = px ? nx >> 1 : hx, cols = sp ? ny >> 1 : hy;
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
        const OrbDesc &od = orb[uni(it.orb)];
        const int nx = uni(od.nx), ny = uni(od.ny), hx = (nx + 1) >> 1, hy = (ny + 1) >> 1;
        const int ox = nx >> 1, oy = ny >> 1;
        const int ksx = (hx + 3) >> 2, ksy = (hy + 3) >> 2;
        const int un = next(u + 1);
        dbl4 D[2][T];
#pragma unroll
        for (int px = 0; px < 2; ++px) {
            stage(nx, ny, px);
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
        const Rsrc ro = make_rsrc(out + uni(od.off) + (long long)uni(it.tile) * nx * ny, (unsigned)(nx * ny) * 8u);
        const int xo = py ? nx - 1 - xl : xl;
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const double v = theirs[(4 * t + r) * 64 + lane];
                const double e = py ? v : EL[t][r], d = py ? ER[t][r] : v;
                const int y = 16 * t + g + 4 * r;
                bst(ro, xok && y < hy ? (unsigned)(y * nx + xo) : kDrop, 0, e + d);
                bst(ro, xok && y < oy ? (unsigned)((ny - 1 - y) * nx + xo) : kDrop, 0, e - d);
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

enum { kFdmYFwd, kFdmYInv, kFdmXFwd, kFdmXInv };

template <int T>
constexpr int kFdmThreads = T <= 3 ? 256 : 512;

// lines as columns of the B operand (x or y-x neighbours contiguous):
//   kFdmYFwd / kFdmYInv: along y, lines (z, x).
template <int T, int MODE>
__global__ __launch_bounds__(kFdmThreads<T>) void k_fdm_col(const Item *__restrict__ units, const FdmRange *__restrict__ ranges,
                                                             const OrbDesc *__restrict__ orb, const int *__restrict__ done,
                                                             const double *__restrict__ tab, const double *in, double *out) {
    constexpr int L = 16 * T, S = kStr<T>, NT = kFdmThreads<T>, NW = NT / 64;
    extern __shared__ __attribute__((aligned(16))) double fsm[];
    const FdmRange rg = ranges[blockIdx.x];
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = lane >> 4, c = lane & 15;
    {
        const OrbDesc &od = orb[units[rg.u0].orb];
        load_table<T, MODE != kFdmYFwd>(fsm, tab + od.fd_t[1], od.fd_n[1], NT);
    }
    __syncthreads();
    // A operand: mode 16 t + c, position 4 s + g (forward); position 16 t + c,
    // mode 4 s + g (inverse)
    auto F = [&](int par, int t, int s) { return fsm[par * L * S + (16 * t + c) * S + 4 * s + g]; };
    const int nsub = 4 * (rg.u1 - rg.u0);
    for (int sub = w; sub < nsub; sub += NW) {
        const Item it = units[rg.u0 + (sub >> 2)];
        if (done && done[it.orb]) continue;  // uniform in the wave
        const OrbDesc &od = orb[it.orb];
        const int n = od.ny, he = (n + 1) >> 1, ho = n >> 1, ks = (he + 3) >> 2;
        const int M2 = od.nx * od.ny;
        const int lines = od.nx * od.nz;
        const int l0 = it.tile * 64 + (sub & 3) * 16;
        if (l0 >= lines) continue;
        const int ln = min(l0 + c, lines - 1);
        const bool lok = l0 + c < lines;
        const int stride = od.nx;
        const long long base = od.off + (long long)(ln / od.nx) * M2 + ln % od.nx;
        const double *p = in + base;
        double *q = out + base;
        dbl4 Ce[T], Co[T];
        if (MODE == kFdmYFwd) {
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
        // back to nodes, one 16-position tile at a time
#pragma unroll
        for (int t = 0; t < T; ++t) {
            dbl4 E = {0.0, 0.0, 0.0, 0.0}, O = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int s = 0; s < 4 * T; ++s) {
                if (s >= 4 * (T - 1) && s >= ks) continue;
                E = mfma(F(0, t, s), Ce[s >> 2][s & 3], E);
                O = mfma(F(1, t, s), Co[s >> 2][s & 3], O);
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

// 1 / x for normal x > 0: the hardware seed (about 2^-23) and one third-order
// step, about 1 ulp
__device__ __forceinline__ double rcp2(double x) {
    const double y = __builtin_amdgcn_rcp(x), e = fma(-x, y, 1.0);
    return fma(y, fma(e, e, e), y);
}

// order of the reads and products of a step: kept as written
#define FDM_ORDER() __builtin_amdgcn_sched_barrier(0)

// z: transform, scale by h^2 / (lam_x + lam_y + lam_z), transform back, in
// place; lines: in-plane points, 16 to a wave.  The next lines' loads are
// issued between the two products, the matrix operands read a step ahead.
// KS: k steps taken, 4 T or (half axes that leave the last half tile empty)
// 4 T - 2.
template <int T, int KS>
__device__ __forceinline__ void fdm_z_lines(const Item *__restrict__ units, const FdmRange rg, const OrbDesc *__restrict__ orb, const int *__restrict__ done,
                                            const double *__restrict__ tab, double *fsm, double *data) {
    constexpr int L = 16 * T, S = kStr<T>, NT = kFdmThreads<T>, NW = NT / 64;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = lane >> 4, c = lane & 15;
    const int nsub = 4 * (rg.u1 - rg.u0);
    // base indices of the operand reads, opaque in each iteration: the reads are
    // not to be hoisted out of the loop into registers
    int fb = g * S + c, ib = c * S + g, zb = 2 * L * S + g;
    auto F = [&](int par, int t, int s) { return fsm[fb + par * L * S + 4 * s * S + 16 * t]; };
    auto I = [&](int par, int t, int s) { return fsm[ib + par * L * S + 16 * t * S + 4 * s]; };
    double fe[4 * T], fo[4 * T], la, lb;
    auto find = [&](int sub) {
        for (; sub < nsub; sub += NW) {
            const Item it = units[rg.u0 + (sub >> 2)];
            const int o = uni(it.orb);
            if (uni(!(done && done[o]) && it.tile * 64 + (sub & 3) * 16 < orb[o].nx * orb[o].ny)) break;
        }
        return sub;
    };
    auto issue = [&](int sub) {
        const Item it = units[rg.u0 + (sub >> 2)];
        const OrbDesc *const od = orb + uni(it.orb);
        const int l0 = uni(it.tile) * 64 + (sub & 3) * 16;
        const int n = uni(od->nz), he = (n + 1) >> 1, nx = uni(od->nx), ny = uni(od->ny), M2 = nx * ny;
        const int ln = min(l0 + c, M2 - 1), fused = uni(od->fd_fused);
        const Rsrc r = make_rsrc(data + uni(od->off), (unsigned)(M2 * n) * 8u);
        const unsigned v0 = (unsigned)(ln + g * M2), v1 = (unsigned)(ln + (3 - g) * M2);
#pragma unroll
        for (int s = 0; s < 4 * T; ++s) {
            if (s < 4 * (T - 1)) {
                fe[s] = bld<double>(r, v0, 4 * s * M2);
                fo[s] = bld<double>(r, v1, (n - 4 - 4 * s) * M2);
            } else {
                const int j = min(4 * s + g, he - 1);
                fe[s] = bld<double>(r, (unsigned)(ln + j * M2), 0);
                fo[s] = bld<double>(r, (unsigned)(ln + (n - 1 - j) * M2), 0);
            }
        }
        const int inner = fused ? ny : nx;
        const int a = ln / inner, b = ln - a * inner;
        auto lam = [&](int d, int nd, int k) {
            const int Ld = 16 * uni(od->fd_n[d]), hd = (nd + 1) >> 1;
            return tab[uni(od->fd_t[d]) + 2 * Ld * Ld + (k < hd ? k : Ld + k - hd)];
        };
        la = lam(0, nx, fused ? a : b);
        lb = lam(1, ny, fused ? b : a);
    };
    int sub = find(w);
    if (sub >= nsub) return;
    issue(sub);
    while (true) {
        const Item it = units[rg.u0 + (sub >> 2)];
        const OrbDesc *const od = orb + uni(it.orb);
        const int l0 = uni(it.tile) * 64 + (sub & 3) * 16;
        const int n = uni(od->nz), he = (n + 1) >> 1, ho = n >> 1, M2 = uni(od->nx) * uni(od->ny);
        const double h2 = od->h * od->h;
        const double lxy = la + lb;
        asm volatile("" : "+v"(fb), "+v"(ib), "+v"(zb));
#pragma unroll
        for (int s = 0; s < 4 * T; ++s) {
            // the centre node, in the last tile, enters once
            const double a = fe[s], b = s >= 4 * (T - 1) && 2 * (4 * s + g) == n - 1 ? 0.0 : fo[s];
            fe[s] = a + b;
            fo[s] = a - b;
        }
        dbl4 Ce[T], Co[T];
#pragma unroll
        for (int t = 0; t < T; ++t) Ce[t] = Co[t] = dbl4{0.0, 0.0, 0.0, 0.0};
        double m[2][2 * T];
#pragma unroll
        for (int t = 0; t < T; ++t) {
            m[0][t] = F(0, t, 0);
            m[0][T + t] = F(1, t, 0);
        }
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            if (s + 1 < KS) {
#pragma unroll
                for (int t = 0; t < T; ++t) {
                    m[(s + 1) & 1][t] = F(0, t, s + 1);
                    m[(s + 1) & 1][T + t] = F(1, t, s + 1);
                }
            }
            FDM_ORDER();
#pragma unroll
            for (int t = 0; t < T; ++t) {
                Ce[t] = mfma(m[s & 1][t], fe[s], Ce[t]);
                Co[t] = mfma(m[s & 1][T + t], fo[s], Co[t]);
            }
            FDM_ORDER();
        }
        const int nxt = find(sub + NW);
        if (nxt < nsub) issue(nxt);
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                Ce[t][r] *= h2 * rcp2(fsm[zb + 16 * t + 4 * r] + lxy);
                Co[t][r] *= h2 * rcp2(fsm[zb + L + 16 * t + 4 * r] + lxy);
            }
        const Rsrc r = make_rsrc(data + uni(od->off), (unsigned)(M2 * n) * 8u);
        const bool lok = l0 + c < M2;
        const unsigned v0 = lok ? (unsigned)(l0 + c + g * M2) : kDrop, v1 = lok ? (unsigned)(l0 + c + (3 - g) * M2) : kDrop;
        double p[2][4];
#pragma unroll
        for (int q = 0; q < 4; ++q) p[0][q] = I(q >> 1, 0, q & 1);
#pragma unroll
        for (int t = 0; t < T; ++t) {
            dbl4 E = {0.0, 0.0, 0.0, 0.0}, O = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int u = 0; u < KS / 2; ++u) {
                const int i = t * (KS / 2) + u, nt = (i + 1) / (KS / 2), nu = (i + 1) % (KS / 2);
                if (nt < T) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) p[(i + 1) & 1][q] = I(q >> 1, nt, 2 * nu + (q & 1));
                }
                FDM_ORDER();
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const int s = 2 * u + q;
                    E = mfma(p[i & 1][q], Ce[s >> 2][s & 3], E);
                    O = mfma(p[i & 1][2 + q], Co[s >> 2][s & 3], O);
                }
                FDM_ORDER();
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (t < T - 1) {
                    bst(r, v0, (16 * t + 4 * q) * M2, E[q] + O[q]);
                    bst(r, v1, (n - 4 - 16 * t - 4 * q) * M2, E[q] - O[q]);
                } else {
                    const int j = 16 * t + g + 4 * q;
                    bst(r, lok && j < he ? (unsigned)(l0 + c + j * M2) : kDrop, 0, E[q] + O[q]);
                    bst(r, lok && j < ho ? (unsigned)(l0 + c + (n - 1 - j) * M2) : kDrop, 0, E[q] - O[q]);
                }
            }
        }
        if (nxt >= nsub) break;
        sub = nxt;
    }
}

template <int T>
__global__ __launch_bounds__(kFdmThreads<T>, 2) void k_fdm_z(const Item *__restrict__ units, const FdmRange *__restrict__ ranges,
                                                           const OrbDesc *__restrict__ orb, const int *__restrict__ done, const double *__restrict__ tab,
                                                           double *data) {
    constexpr int L = 16 * T, S = kStr<T>, NT = kFdmThreads<T>;
    extern __shared__ __attribute__((aligned(16))) double fsm[];
    const FdmRange rg = ranges[blockIdx.x];
    const OrbDesc &od = orb[units[rg.u0].orb];
    load_table<T, true>(fsm, tab + od.fd_t[2], od.fd_n[2], NT);
    for (int i = threadIdx.x; i < 2 * L; i += NT) fsm[2 * L * S + i] = tab[od.fd_t[2] + 2 * L * L + i];
    __syncthreads();
    // k steps of the half axis, up to a step of padding (one axis a block)
    if ((od.nz + 1) / 2 > 16 * T - 8) fdm_z_lines<T, 4 * T>(units, rg, orb, done, tab, fsm, data);
    else fdm_z_lines<T, 4 * T - 2>(units, rg, orb, done, tab, fsm, data);
}

// lines along x (contiguous), as rows of the A operand; lines (z, y)
//   SQ (forward): b = scale src^2
template <int T, int MODE, bool SQ>
__global__ __launch_bounds__(kFdmThreads<T>) void k_fdm_row(const Item *__restrict__ units, const FdmRange *__restrict__ ranges,
                                                             const OrbDesc *__restrict__ orb, const int *__restrict__ done,
                                                             const double *__restrict__ tab, const double *in, double scale,
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

size_t z_lds(int T) { return line_lds(T) + 32 * (size_t)T * sizeof(double); }

// blocks of a kernel that one compute unit holds
template <class K>
int occ_of(K k, int threads, size_t lds) {
    int n = 0;
    if (allow_lds(reinterpret_cast<const void *>(k), lds) != hipSuccess) return 0;
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
                                        occ_of(k_fdm_xy_inv<TT>, 128 * TT, xy_lds(TT, two != 0)));
#define Z(TT) case TT: return occ_of(k_fdm_z<TT>, kFdmThreads<TT>, z_lds(TT));
#define XL(TT) case TT: return occ_of(k_fdm_row<TT, kFdmXFwd, true>, kFdmThreads<TT>, line_lds(TT));
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
        if (e == hipSuccess) e = allow_lds(reinterpret_cast<const void *>(k), lds);
    };
#define XY(TT)                                                                  \
    set(k_fdm_xy_fwd<TT, true>, std::min<size_t>(xy_lds(TT, true), 160 * 1024));  \
    set(k_fdm_xy_fwd<TT, false>, std::min<size_t>(xy_lds(TT, true), 160 * 1024)); \
    set(k_fdm_xy_inv<TT>, std::min<size_t>(xy_lds(TT, true), 160 * 1024));
    XY(1) XY(2) XY(3) XY(4)
#undef XY
#define LN(TT)                                                 \
    set(k_fdm_z<TT>, z_lds(TT));             \
    set(k_fdm_col<TT, kFdmYFwd>, line_lds(TT));          \
    set(k_fdm_col<TT, kFdmYInv>, line_lds(TT));          \
    set(k_fdm_row<TT, kFdmXFwd, true>, line_lds(TT));    \
    set(k_fdm_row<TT, kFdmXFwd, false>, line_lds(TT));   \
    set(k_fdm_row<TT, kFdmXInv, false>, line_lds(TT));
    LN(1) LN(2) LN(3) LN(4) LN(5) LN(6)
#undef LN
    if (e == hipSuccess) ready.insert(dev);
    return e;
}

hipError_t launch_fdm(const FdmPlan &p, const OrbDesc *orb, const int *done, const double *tab, const double *src,
                      int square, double scale, double *work, double *out, hipStream_t s) {
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
        if (square) GO((k_fdm_row<TT, kFdmXFwd, true>), kFdmThreads<TT>, line_lds(TT), src, scale, work);        \
        else GO((k_fdm_row<TT, kFdmXFwd, false>), kFdmThreads<TT>, line_lds(TT), src, scale, work);              \
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
#define ZZ(TT) case TT: GO((k_fdm_z<TT>), kFdmThreads<TT>, z_lds(TT), work); return hipSuccess;
    e = each(pass, [&](const FdmClass &q) -> hipError_t {
        switch (q.T) { ZZ(1) ZZ(2) ZZ(3) ZZ(4) ZZ(5) ZZ(6) }
        return hipErrorInvalidValue;
    });
#undef ZZ
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
        GO((k_fdm_row<TT, kFdmXInv, false>), kFdmThreads<TT>, line_lds(TT), (const double *)work, 1.0, out);           \
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
        GO((k_fdm_xy_inv<TT>), 128 * TT, xy_lds(TT, q.two), q.two, (const double *)work, out);           \
        return hipSuccess;
        switch (q.T) { XY(1) XY(2) XY(3) XY(4) }
#undef XY
        return hipErrorInvalidValue;
    });
#undef GO
}

}  // namespace fsic
