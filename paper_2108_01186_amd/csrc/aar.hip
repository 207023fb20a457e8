// Alternating Anderson-Richardson (AAR) iteration for the per-orbital
// Poisson problems -L v = b, the solver the paper's real-space code uses
// (Sec. II.A).  With f_k = M^{-1} (b + L x_k) (M^{-1}: the sine-transform
// preconditioner) and the last m differences
//   X_k = [x_{i+1} - x_i],  F_k = [f_{i+1} - f_i],  i = k-m .. k-1,
// every p-th iteration is an Anderson extrapolation
//   x_{k+1} = x_k + beta f_k - (X_k + beta F_k) gamma,
//   gamma = argmin || f_k - F_k gamma ||  (normal equations, m x m),
// and the others are Richardson steps x_{k+1} = x_k + omega f_k.
// The history is kept as ring buffers of m columns (column i in slot i % m).
// All orbitals of a batch advance together; converged ones are skipped.
#include "kernels.h"

namespace fsic {

namespace {

// slot of the Gram entry (i, j), i <= j < nh, then nh right-hand sides
__device__ __forceinline__ int gram_slot(int i, int j, int nh) {
    return i * nh - i * (i - 1) / 2 + (j - i);
}

}  // namespace

// History of the newest difference column and, at Anderson steps, the
// per-tile partial sums of F^T F and F^T f.
//   hist: f_k - f_{k-1} goes into slot (k-1) % m (needs k >= 1);
//   fprev := f_k.
// Bound by memory latency unless a thread has many bytes under way: four
// consecutive nodes a step in 16-byte loads, none of them in a branch (15
// orbitals of 64^3, seven columns: 67 -> 38 us against one node a step).  Fields that
// are no multiple of four nodes take them one by one.
template <int VN>
__device__ __forceinline__ void aar_dots_tile(const AarBufs &a, const OrbDesc &od, int tile, int k, int nh, int hist,
                                              int dots, double (&acc)[kAarD]) {
    typedef float VF __attribute__((ext_vector_type(VN)));
    const long long M = (long long)od.nx * od.ny * od.nz;
    const int hs = (k + a.m - 1) % a.m;
#pragma unroll 1
    for (int e = 0; e < kPW / (256 * VN); ++e) {
        const long long i = (long long)tile * kPW + (long long)(e * 256 + threadIdx.x) * VN;
        const bool in = i < M;
        const long long g = od.off + (in ? i : M - VN);
        const VF f = *reinterpret_cast<const VF *>(a.F + g);
        const VF fp = *reinterpret_cast<const VF *>(a.Fprev + g);
        VF col[kAarM];
        if (dots) {
#pragma unroll
            for (int j = 0; j < kAarM; ++j)
                col[j] = *reinterpret_cast<const VF *>(a.Fh + (size_t)min(j, nh - 1) * a.fields + g);
        }
        const VF d = f - fp;
        if (hist && in) {
            *reinterpret_cast<VF *>(a.Fh + (size_t)hs * a.fields + g) = d;
            *reinterpret_cast<VF *>(a.Fprev + g) = f;
        }
        if (dots) {
#pragma unroll
            for (int v = 0; v < VN; ++v) {
                double c[kAarM];
#pragma unroll
                for (int j = 0; j < kAarM; ++j)
                    c[j] = in && j < nh ? (double)(hist && j == hs ? d[v] : col[j][v]) : 0.0;
#pragma unroll
                for (int ii = 0; ii < kAarM; ++ii)
#pragma unroll
                    for (int jj = ii; jj < kAarM; ++jj) acc[gram_slot(ii, jj, kAarM)] += c[ii] * c[jj];
#pragma unroll
                for (int ii = 0; ii < kAarM; ++ii) acc[kAarG + ii] += c[ii] * (in ? (double)f[v] : 0.0);
            }
        }
    }
}

__global__ __launch_bounds__(256) void k_aar_dots(AarBufs a, int k, int nh, int hist, int dots) {
    __shared__ double swave[4][kAarD];
    const Item it = a.items8[blockIdx.x];
    if (it.orb < 0) return;
    if (a.done[it.orb] == 1) return;
    const OrbDesc od = a.orb[it.orb];
    double acc[kAarD];
#pragma unroll
    for (int q = 0; q < kAarD; ++q) acc[q] = 0.0;
    if (((od.off | a.fields | ((long long)od.nx * od.ny * od.nz)) & 3) == 0) aar_dots_tile<4>(a, od, it.tile, k, nh, hist, dots, acc);
    else aar_dots_tile<1>(a, od, it.tile, k, nh, hist, dots, acc);
    if (!dots) return;
    // every accumulator index is a compile-time constant (a runtime index
    // would put the array in scratch memory): wave sums into LDS, one
    // barrier, then thread q adds the four wave sums of entry q in fixed order
    const int w = threadIdx.x >> 6;
#pragma unroll
    for (int q = 0; q < kAarD; ++q) {
        const double t = wave_sum(acc[q]);
        if ((threadIdx.x & 63) == 0) swave[w][q] = t;
    }
    __syncthreads();
    if (threadIdx.x < kAarD) {
        const int q = threadIdx.x;
        a.partD[(size_t)(od.base8 + it.tile) * kAarD + q] = (swave[0][q] + swave[1][q]) + (swave[2][q] + swave[3][q]);
    }
}

// Per orbital: sum the tile partials (fixed order) and solve the nh x nh
// normal equations for gamma by Gaussian elimination with partial pivoting;
// a tiny multiple of the largest diagonal entry is added to the diagonal so
// nearly dependent history columns give a bounded gamma.  A chain of
// latencies: all entries are summed at once, a wave per run of tiles, and
// the matrix is eliminated in the registers of one wave, entry (r, j) in lane
// 8 r + j (15 orbitals of 64^3: 44 -> below 9 us against a reduction per entry
// and one thread with the matrix in memory).
__global__ __launch_bounds__(256) void k_aar_solve(AarBufs a, int nh) {
    static_assert(kAarD <= 64 && kAarM < 8, "lanes of a run, columns of a row");
    __shared__ double run[4][64];
    __shared__ double d[kAarD];
    const int o = blockIdx.x;
    if (a.done[o] == 1) return;
    const OrbDesc od = a.orb[o];
    const int q = threadIdx.x & 63, rn = threadIdx.x >> 6;
    double s = 0.0;
    if (q < kAarD)
#pragma unroll 8
        for (int t = rn; t < od.nt8; t += 4) s += a.partD[(size_t)(od.base8 + t) * kAarD + q];
    run[rn][q] = s;
    __syncthreads();
    if (threadIdx.x < kAarD)
        d[q] = (run[0][q] + run[1][q]) + (run[2][q] + run[3][q]);
    __syncthreads();
    if (threadIdx.x >= 64) return;
    const int r = threadIdx.x >> 3, j = threadIdx.x & 7;
    double v = 0.0, dmax = 0.0;
    for (int i = 0; i < nh; ++i) dmax = fmax(dmax, d[gram_slot(i, i, kAarM)]);
    if (r < nh && j < nh) {
        v = d[gram_slot(min(r, j), max(r, j), kAarM)];
        if (r == j) v += 1e-13 * dmax;
    } else if (r < nh && j == nh) {
        v = d[kAarG + r];
    }
    for (int col = 0; col < nh; ++col) {
        int piv = col;
        double best = fabs(__shfl(v, 9 * col));
        for (int i = col + 1; i < nh; ++i) {
            const double x = fabs(__shfl(v, 8 * i + col));
            if (x > best) {
                best = x;
                piv = i;
            }
        }
        v = __shfl(v, 8 * (r == col ? piv : r == piv ? col : r) + j);
        const double pv = __shfl(v, 9 * col), lead = __shfl(v, 8 * r + col), top = __shfl(v, 8 * col + j);
        const double fct = pv != 0.0 ? lead / pv : 0.0;
        if (r > col && j >= col) v -= fct * top;
    }
    double gam[kAarM];
#pragma unroll
    for (int i = kAarM - 1; i >= 0; --i) {
        double t = __shfl(v, 8 * i + nh);
#pragma unroll
        for (int c = i + 1; c < kAarM; ++c)
            if (c < nh) t -= __shfl(v, 8 * i + c) * gam[c];
        const double p = __shfl(v, 9 * i);
        gam[i] = i < nh && p != 0.0 ? t / p : 0.0;
    }
    if (threadIdx.x == 0)
#pragma unroll
        for (int i = 0; i < kAarM; ++i)
            a.gamma[(size_t)o * kAarM + i] = isfinite(gam[i]) ? gam[i] : 0.0;
}

// The step: Richardson (omega f) or Anderson (beta f - sum_j gamma_j (X_j +
// beta F_j)); x += step and the step becomes history column k (slot k % m).
// hist: 1 also records f_k - f_{k-1} and f_k first, 2 only f_k (the first
// iteration), 0 neither (Anderson steps did both in k_aar_dots).
template <bool AND>
__global__ __launch_bounds__(256) void k_aar_step(AarBufs a, int k, int nh, double omega, double beta,
                                                  int hist) {
    const Item it = a.items8[blockIdx.x];
    if (it.orb < 0) return;
    if (a.done[it.orb] == 1) return;
    const OrbDesc od = a.orb[it.orb];
    const long long M = (long long)od.nx * od.ny * od.nz;
    const long long base = (long long)it.tile * kPW;
    const int hs = (k + a.m - 1) % a.m, xs = k % a.m;
    double gam[kAarM];
#pragma unroll
    for (int j = 0; j < kAarM; ++j) gam[j] = (AND && j < nh) ? a.gamma[(size_t)it.orb * kAarM + j] : 0.0;
    for (int e = 0; e < kPW / 256; ++e) {
        const long long i = base + e * 256 + threadIdx.x;
        if (i >= M) continue;
        const long long g = od.off + i;
        const float f = a.F[g];
        if (hist == 1) a.Fh[(size_t)hs * a.fields + g] = f - a.Fprev[g];
        if (hist) a.Fprev[g] = f;
        double step;
        if (AND) {
            step = beta * (double)f;
#pragma unroll
            for (int j = 0; j < kAarM; ++j)
                if (j < nh)
                    step -= gam[j] * (a.Xh[(size_t)j * a.fields + g] + beta * (double)a.Fh[(size_t)j * a.fields + g]);
        } else {
            step = omega * (double)f;
        }
        a.X[g] += step;
        a.Xh[(size_t)xs * a.fields + g] = step;
    }
}

hipError_t launch_aar_dots(const AarBufs &a, int nitems8, int k, int nh, int hist, int dots,
                           hipStream_t s) {
    if (nitems8 <= 0 || nh > kAarM || a.m != kAarM) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_aar_dots, dim3(nitems8), dim3(256), 0, s, a, k, nh, hist, dots);
    return hipGetLastError();
}

hipError_t launch_aar_solve(const AarBufs &a, int norb, int nh, hipStream_t s) {
    if (norb <= 0 || nh < 1 || nh > kAarM) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_aar_solve, dim3(norb), dim3(256), 0, s, a, nh);
    return hipGetLastError();
}

hipError_t launch_aar_step(const AarBufs &a, int nitems8, int k, int nh, double omega, double beta,
                           bool anderson, int hist, hipStream_t s) {
    if (nitems8 <= 0 || nh > kAarM || a.m != kAarM) return hipErrorInvalidValue;
    if (anderson)
        hipLaunchKernelGGL(k_aar_step<true>, dim3(nitems8), dim3(256), 0, s, a, k, nh, omega, beta, hist);
    else
        hipLaunchKernelGGL(k_aar_step<false>, dim3(nitems8), dim3(256), 0, s, a, k, nh, omega, beta, hist);
    return hipGetLastError();
}

}  // namespace fsic
