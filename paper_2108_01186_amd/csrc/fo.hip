// Fermi orbitals: the cubic interpolation of the KS orbitals at the FODs
// (Sec. II.B) and its derivative for the FOD gradient (Eq. 9-11).  Of the
// orbital-sized work that remains, products.hip does
//   * the Gram matrix G = dV psi psi^T, from which the FO overlap follows
//     exactly as S = dV F F^T = T G T^T (F = T psi), so F is never stored;
//   * the Fermi-Loewdin orbitals phi = Q psi with Q = S^{-1/2} T,
// lowdin.hip everything N x N; the fp32 product of FSIC_FP32_ORBITALS is here.
#include <algorithm>
#include <cstdint>

#include "kernels.h"

namespace fsic {

// ---------------------------------------------------------------------------
// cubic interpolation at the FODs, T = u / |u|
// ---------------------------------------------------------------------------

__device__ __forceinline__ void cubic_weights(double t, double *w, double *dw) {
    // Lagrange basis on the nodes -1, 0, 1, 2 and its derivative in t
    const double tm1 = t - 1.0, tm2 = t - 2.0, tp1 = t + 1.0;
    w[0] = -t * tm1 * tm2 * (1.0 / 6.0);
    w[1] = tp1 * tm1 * tm2 * 0.5;
    w[2] = -tp1 * t * tm2 * 0.5;
    w[3] = tp1 * t * tm1 * (1.0 / 6.0);
    const double t2 = t * t;
    dw[0] = -(3.0 * t2 - 6.0 * t + 2.0) * (1.0 / 6.0);
    dw[1] = (3.0 * t2 - 4.0 * t - 1.0) * 0.5;
    dw[2] = -(3.0 * t2 - 2.0 * t - 2.0) * 0.5;
    dw[3] = (3.0 * t2 - 1.0) * (1.0 / 6.0);
}

// Weights, over the six nodes i0-2 .. i0+3 of one axis, that turn grid
// values into the cubic interpolant (at offset t from node i0) of the
// per-node first differences: central (f[j+1] - f[j-1]) / 2 inside, forward
// at node 0, backward at node n-1 (in units of 1/h).  Sec. II.B builds
// grad psi at an FOD this way.  Entries 0 and 5 stay zero whenever their
// node lies outside the grid (i0 is in [1, n-3]).
__device__ __forceinline__ void fd_interp_weights(const double *w, int i0, int n, double *e) {
#pragma unroll
    for (int k = 0; k < 6; ++k) e[k] = 0.0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int j = i0 - 1 + q;  // node carrying weight w[q]; its slot is q + 1
        if (j == 0) {
            e[q + 2] += w[q];
            e[q + 1] -= w[q];
        } else if (j == n - 1) {
            e[q + 1] += w[q];
            e[q] -= w[q];
        } else {
            e[q + 2] += 0.5 * w[q];
            e[q] -= 0.5 * w[q];
        }
    }
}

// One block per FOD (or query point) i, one thread per orbital a < N (N <=
// 128): u = psi_a(a_i), du = grad psi_a(a_i), and, for the FOD path,
// rho(a_i) and T_i,a = u / sqrt(rho).  FD = false: du is the derivative of
// the cubic interpolant (the exact derivative of the discrete u); FD = true:
// du interpolates the per-node difference gradient.  All channels of a batch
// in one launch, the 16 rows of a cell loaded together: a gather is bound by
// latency (twelve channels of 6 to 40 FODs 12 x 10.6 -> 14 us, two of 16 and
// 15 2 x 10.4 -> 11).
template <bool FD>
__global__ __launch_bounds__(128) void k_interp(InterpBatch ib, double floor, int *status) {
    __shared__ double sred[2];
    int ci = 0;
    while (ci + 1 < ib.n && (int)blockIdx.x >= ib.c[ci + 1].block0) ++ci;
    const InterpChan &ch = ib.c[ci];
    const int N = ch.N, nx = ch.nx, ny = ch.ny, nz = ch.nz;
    const double h = ch.h;
    const double *const psi = ch.psi;
    double *const u = ch.u, *const du = ch.du, *const rhoa = ch.rhoa, *const T = ch.T;
    const int i = blockIdx.x - ch.block0;  // FOD
    const FodCell cl = ch.cells[i];
    double wx[4], wy[4], wz[4], dx[4], dy[4], dz[4];
    cubic_weights(cl.t[0], wx, dx);
    cubic_weights(cl.t[1], wy, dy);
    cubic_weights(cl.t[2], wz, dz);
    const long long M = (long long)nx * ny * nz;
    const int a = threadIdx.x;
    double val = 0.0, gx = 0.0, gy = 0.0, gz = 0.0;
    if (a < N && !FD) {
        const double *f = psi + (long long)a * M;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                const double *row = f + ((long long)(cl.i0[2] - 1 + c) * ny + (cl.i0[1] - 1 + b)) * nx + (cl.i0[0] - 1);
                double sx = 0.0, sdx = 0.0;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    sx += wx[q] * row[q];
                    sdx += dx[q] * row[q];
                }
                val += wz[c] * wy[b] * sx;
                gx += wz[c] * wy[b] * sdx;
                gy += wz[c] * dy[b] * sx;
                gz += dz[c] * wy[b] * sx;
            }
        }
    } else if (a < N) {
        // six-node windows: value weights padded with zeros, difference weights
        double vx6[6] = {0.0, wx[0], wx[1], wx[2], wx[3], 0.0};
        double vy6[6] = {0.0, wy[0], wy[1], wy[2], wy[3], 0.0};
        double vz6[6] = {0.0, wz[0], wz[1], wz[2], wz[3], 0.0};
        double ex[6], ey[6], ez[6];
        fd_interp_weights(wx, cl.i0[0], nx, ex);
        fd_interp_weights(wy, cl.i0[1], ny, ey);
        fd_interp_weights(wz, cl.i0[2], nz, ez);
        int xs[6];
#pragma unroll
        for (int q = 0; q < 6; ++q) xs[q] = min(max(cl.i0[0] - 2 + q, 0), nx - 1);
        const double *f = psi + (long long)a * M;
        for (int c = 0; c < 6; ++c) {
            const int kz = min(max(cl.i0[2] - 2 + c, 0), nz - 1);
            for (int b = 0; b < 6; ++b) {
                const int jy = min(max(cl.i0[1] - 2 + b, 0), ny - 1);
                const double *row = f + ((long long)kz * ny + jy) * nx;
                double sx = 0.0, sdx = 0.0;
#pragma unroll
                for (int q = 0; q < 6; ++q) {
                    const double fv = row[xs[q]];
                    sx += vx6[q] * fv;
                    sdx += ex[q] * fv;
                }
                val += vz6[c] * vy6[b] * sx;
                gx += vz6[c] * vy6[b] * sdx;
                gy += vz6[c] * ey[b] * sx;
                gz += ez[c] * vy6[b] * sx;
            }
        }
    }
    if (a < N) {
        const double ih = 1.0 / h;
        u[(size_t)i * N + a] = val;
        du[((size_t)i * N + a) * 3 + 0] = gx * ih;
        du[((size_t)i * N + a) * 3 + 1] = gy * ih;
        du[((size_t)i * N + a) * 3 + 2] = gz * ih;
    }
    // rho(a_i) = sum_a psi_a(a_i)^2 (occupations 1), fixed-order reduction
    double sq = (a < N) ? val * val : 0.0;
    sq = wave_sum(sq);
    if ((threadIdx.x & 63) == 0) sred[threadIdx.x >> 6] = sq;
    __syncthreads();
    const double rho = sred[0] + sred[1];
    if (a == 0) {
        rhoa[i] = rho;
        if (!(rho > floor)) atomicOr(status, kStVacuum);
        if (!isfinite(rho)) atomicOr(status, kStNonFinite);
    }
    if (a < N) T[(size_t)i * N + a] = (rho > floor) ? val / sqrt(rho) : 0.0;
}

hipError_t launch_interp(const InterpChan *chans, int n, double floor, int *status, bool fd_gradient, hipStream_t s) {
    for (int c0 = 0; c0 < n; c0 += kInterpBatch) {
        InterpBatch ib{};
        ib.n = std::min(kInterpBatch, n - c0);
        int blocks = 0;
        for (int q = 0; q < ib.n; ++q) {
            ib.c[q] = chans[c0 + q];
            if (ib.c[q].K < 1 || ib.c[q].N < 1 || ib.c[q].N > 128) return hipErrorInvalidValue;
            ib.c[q].block0 = blocks;
            blocks += ib.c[q].K;
        }
        if (fd_gradient) hipLaunchKernelGGL(k_interp<true>, dim3(blocks), dim3(128), 0, s, ib, floor, status);
        else hipLaunchKernelGGL(k_interp<false>, dim3(blocks), dim3(128), 0, s, ib, floor, status);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// ---------------------------------------------------------------------------
// out = A psi in fp32 (FSIC_FP32_ORBITALS; the FP64 products: products.hip)
// ---------------------------------------------------------------------------

// A and psi rounded to fp32, products accumulated in fp32 on
// v_mfma_f32_16x16x4f32 (D lane l, item j: row 4 (l/16) + j), out in fp64
typedef float flt4 __attribute__((ext_vector_type(4)));
__global__ __launch_bounds__(256) void k_orb_gemm32(int N, long long M, const double *A,
                                                    const double *psi, double *out) {
    const int Nt = (N + 15) >> 4;
    const int lane = threadIdx.x & 63;
    const int row = lane & 15, kk = lane >> 4;
    const long long nstrip = (M + 15) >> 4;
    const long long wave = ((long long)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const long long nwave = ((long long)gridDim.x * blockDim.x) >> 6;
    for (long long st = wave; st < nstrip; st += nwave) {
        const long long m = st * 16 + row;
        flt4 acc[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) acc[t] = flt4{0.f, 0.f, 0.f, 0.f};
        for (int a0 = 0; a0 < N; a0 += 4) {
            const int a = a0 + kk;
            const float b = (a < N && m < M) ? (float)psi[(long long)a * M + m] : 0.f;
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                if (t < Nt) {
                    const int i = 16 * t + row;
                    const float av = (i < N && a < N) ? (float)A[i * N + a] : 0.f;
                    acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, b, acc[t], 0, 0, 0);
                }
            }
        }
        const long long mo = st * 16 + row;
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            if (t < Nt && mo < M) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int i = 16 * t + 4 * kk + j;
                    if (i < N) out[(long long)i * M + mo] = (double)acc[t][j];
                }
            }
        }
    }
}

hipError_t launch_orb_gemm32(int N, long long M, const double *A, const double *psi, double *out,
                             hipStream_t s) {
    const long long nstrip = (M + 15) / 16;
    long long nblk = (nstrip + 3) / 4;
    if (nblk > 8192) nblk = 8192;
    hipLaunchKernelGGL(k_orb_gemm32, dim3((unsigned)nblk), dim3(256), 0, s, N, M, A, psi, out);
    return hipGetLastError();
}

}  // namespace fsic
