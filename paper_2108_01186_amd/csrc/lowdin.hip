// The N x N part of the Fermi-Loewdin orbitals (Eq. 6-8, Sec. I.B): overlap
// S = T G T^T, eigen-decomposition, Z = S^{-1/2}, Q = Z T, and the reverse of
// that chain for the FOD gradient (Eq. 9-11).  One workgroup of 16 waves per
// channel (N <= 128), products on the FP64 matrix cores.
#include <algorithm>
#include <cstdint>

#include "kernels.h"
#include "lds.h"

namespace fsic {

typedef double dbl4 __attribute__((ext_vector_type(4)));

constexpr int kLwThreads = 1024;

// Product of two N x N matrices, a wave per (16 R) x (16 R) block of the
// result: fa(i, k) and fb(k, j) read the factors, fs(i, j, v) takes an entry.
// v_mfma_f64_16x16x4: lane l holds A(l % 16, l / 16), B(l / 16, l % 16) and
// D(l / 16 + 4 r, l % 16).  Eight k-steps of loads are in flight at a time
// (four for R = 2); R = 2 halves the operand reads of the large matrices.
template <int R, class FA, class FB, class FS>
__device__ __forceinline__ void mf_gemm(int N, FA fa, FB fb, FS fs, bool upper = false) {
    constexpr int U = R == 1 ? 8 : 4;
    const int lane = threadIdx.x & 63, c = lane & 15, g = lane >> 4;
    const int nt = (N + 16 * R - 1) / (16 * R);
    for (int t = threadIdx.x >> 6; t < nt * nt; t += kLwThreads / 64) {
        const int ti = t / nt, tj = t - ti * nt;
        if (upper && tj < ti) continue;
        dbl4 acc[R][R];
#pragma unroll
        for (int r = 0; r < R * R; ++r) acc[r / R][r % R] = dbl4{0.0, 0.0, 0.0, 0.0};
        int ri[R], ci[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            ri[r] = min(16 * (R * ti + r) + c, N - 1);  // rows past N: results dropped
            ci[r] = min(16 * (R * tj + r) + c, N - 1);
        }
        for (int k0 = 0; k0 < N; k0 += 4 * U) {
            double av[U][R], bv[U][R];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int k = k0 + 4 * u + g, kc = min(k, N - 1);
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const double a = fa(ri[r], kc), b = fb(kc, ci[r]);
                    av[u][r] = k < N ? a : 0.0;
                    bv[u][r] = k < N ? b : 0.0;
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int r = 0; r < R * R; ++r)
                    acc[r / R][r % R] =
                        __builtin_amdgcn_mfma_f64_16x16x4f64(av[u][r / R], bv[u][r % R], acc[r / R][r % R], 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < R * R; ++r)
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                const int i = 16 * (R * ti + r / R) + g + 4 * d, j = 16 * (R * tj + r % R) + c;
                if (i < N && j < N) fs(i, j, acc[r / R][r % R][d]);
            }
    }
}

// 1/sqrt(x) for x in [2^-2, 2^2] (and 0 -> inf is not reached): the hardware
// seed (about 2^-26) and one third-order step, error about 1 ulp
__device__ __forceinline__ double rsqrt1(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    const double e = fma(-x * y, y, 1.0);
    return fma(y * e, fma(0.375, e, 0.5), y);
}

// value of the lane above / below (wave-wide shifts by one lane)
template <int CTRL>
__device__ __forceinline__ double wave_shift(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp((int)b, (int)b, CTRL, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp((int)(b >> 32), (int)(b >> 32), CTRL, 0xf, 0xf, false);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
constexpr int kWaveShl1 = 0x130;  // lane l reads lane l + 1
constexpr int kWaveShr1 = 0x138;  // lane l reads lane l - 1

// Channel of N orbitals (Ne = N rounded up to even, padded with the
// identity).  Cyclic Jacobi with round-robin pairing: positions 0..Ne-1, pair
// j = positions (j, Ne-1-j); after a round position a moves to a-1 (1 to
// Ne-1, 0 stays), so every thread keeps its positions and with them its LDS
// addresses for the whole run, and after Ne-1 rounds every index is back.
//
// What bounds it: the serial chain of a round (angle, broadcast, rotation),
// N-1 rounds a sweep and 6 to 10 sweeps.  So only the upper triangle of A is
// kept (LDS, odd row stride: the column reads of transposed entries meet no
// bank conflict); waves 0-7 hold the off-diagonal 2 x 2 blocks (K per thread)
// in registers while lanes of wave 0 compute the angles from the diagonal
// ones with two reciprocal square roots and no division; waves 8-15 apply the
// rotations to the eigenvector rows, which stay in registers and move along
// the lanes.  K = 1 for N <= 64, 4 up to 128.  The work of a channel depends on
// N only, so a batch gives the bits of a single call.  Measured against whole
// blocks of a matrix passing through LDS in 256 threads, with divisions and
// scalar products: N = 45, seven sweeps 950 -> 198 us; N = 32 98 -> 52 us;
// N = 128 of a well-localised system 585 -> 146 us.
template <int K>
__device__ __forceinline__ void lowdin_one(int N, const double *T, const double *G, double *S, double *lam,
                                           double *U, double *Z, double *Qm, double *work, double *dsm,
                                           double eig_floor, int *status, double *info) {
    constexpr int R = K == 1 ? 1 : 2;
    constexpr int CL = K == 1 ? 32 : 64;           // lanes along the column pairs
    constexpr int VS = 8 * 64 / CL;                // eigenvector rows per step of waves 8-15
    constexpr int VN = 2 * CL / VS;                // steps
    const int Ne = N + (N & 1), half = Ne >> 1, ld = Ne + 1;
    __shared__ double2 cs[64];
    __shared__ double sred[2][16];
    __shared__ double slam[kMaxOrb];
    __shared__ int sflag;
    double *A = dsm;
    // T G and later Z: LDS where two matrices fit
    double *TG = K == 1 ? dsm + Ne * ld : work;
    const int tl = K == 1 ? ld : N;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    mf_gemm<R>(N, [&](int i, int k) { return T[i * N + k]; }, [&](int k, int j) { return G[k * N + j]; },
               [&](int i, int j, double v) { TG[i * tl + j] = v; });
    if (tid < Ne && Ne > N) A[tid * ld + N] = tid == N ? 1.0 : 0.0;
    __syncthreads();
    // S from its upper triangle, exactly symmetric
    mf_gemm<R>(N, [&](int i, int k) { return TG[i * tl + k]; }, [&](int k, int j) { return T[j * N + k]; },
               [&](int i, int j, double v) {
                   if (i > j) return;
                   S[i * N + j] = v;
                   if (i < j) S[j * N + i] = v;
                   A[i * ld + j] = v;
               }, true);
    __syncthreads();
    // end of the sweeps: off-diagonal against diagonal mass, uniform over the workgroup
    auto converged = [&](double off, double dg) {
        off = wave_sum(2.0 * off);
        dg = wave_sum(dg);
        if (lane == 0) { sred[0][wave] = off; sred[1][wave] = dg; }
        __syncthreads();
        off = dg = 0.0;
        for (int w = 0; w < 8; ++w) { off += sred[0][w]; dg += sred[1][w]; }
        return off <= 1e-30 * dg;
    };
    // eigenvector rows (waves 8-15): lane j of a group holds positions j and Ne-1-j
    const int vj = lane & (CL - 1), vw = (wave - 8) * (64 / CL), vr0 = vw + lane / CL;
    // the two roles run loops of their own (their registers need not fit
    // together) and meet at the same barriers, two a round and one a sweep
    if (wave < 8) {
        // this thread's blocks: address of the entries and where they move to
        auto canon = [&](int a, int b) { return a < b ? a * ld + b : b * ld + a; };
        auto moved = [&](int a) { return a == 0 ? 0 : a == 1 ? Ne - 1 : a - 1; };
        const int nblk = half * (half - 1) / 2;
        int rd[K][4], wr[K][4], ij[K];
        double blk[K][4];
#pragma unroll
        for (int q = 0; q < K; ++q) {
            int e = tid + 512 * q, i = 0;
            ij[q] = -1;
            if (e < nblk) {
                while (e >= half - 1 - i) { e -= half - 1 - i; ++i; }
                const int j = i + 1 + e, I = Ne - 1 - i, J = Ne - 1 - j;
                ij[q] = i | j << 8;
                rd[q][0] = canon(i, j); rd[q][1] = canon(i, J); rd[q][2] = canon(I, j); rd[q][3] = canon(I, J);
                wr[q][0] = canon(moved(i), moved(j)); wr[q][1] = canon(moved(i), moved(J));
                wr[q][2] = canon(moved(I), moved(j)); wr[q][3] = canon(moved(I), moved(J));
            }
        }
        const bool dia = tid < half;
        const int dp = lane, dq = Ne - 1 - lane, mp = moved(dp), mq = moved(dq);
        double app = 0.0, aqq = 0.0, apq = 0.0;
        for (int sweep = 0; sweep < 40; ++sweep) {
            bool done = false;
            for (int r = 0; r < Ne - 1 && !done; ++r) {
#pragma unroll
                for (int q = 0; q < K; ++q)
                    if (ij[q] >= 0)
#pragma unroll
                        for (int d = 0; d < 4; ++d) blk[q][d] = A[rd[q][d]];
                if (dia) {
                    app = A[dp * ld + dp];
                    aqq = A[dq * ld + dq];
                    apq = A[dp * ld + dq];
                }
                if (r == 0) {
                    double off = 0.0, dg = 0.0;
#pragma unroll
                    for (int q = 0; q < K; ++q)
                        if (ij[q] >= 0)
#pragma unroll
                            for (int d = 0; d < 4; ++d) off += blk[q][d] * blk[q][d];
                    if (dia) { off += apq * apq; dg = app * app + aqq * aqq; }
                    done = converged(off, dg);
                }
                if (!done) {
                    if (dia) {
                        // cos 2t = |d| / hypot(d, o), c^2 = (1 + cos 2t) / 2, s = sin 2t / (2 c); the
                        // larger of d and o scaled to [1/2, 1) against overflow
                        const double d0 = aqq - app, o0 = 2.0 * apq;
                        double c = 1.0, s = 0.0, t = 0.0;
                        if (fabs(apq) > 1e-300) {
                            const int ex = __builtin_amdgcn_frexp_exp(fmax(fabs(d0), fabs(o0)));
                            const double d = fabs(ldexp(d0, -ex)), o = ldexp(d0 < 0.0 ? -o0 : o0, -ex);
                            const double h = rsqrt1(fma(d, d, o * o));
                            const double x = fma(0.5 * d, h, 0.5), rc = rsqrt1(x);
                            c = x * rc;
                            s = 0.5 * o * h * rc;
                            t = s * rc;  // s / c: 1 / c = rc
                        }
                        cs[lane] = double2{c, s};
                        app = fma(-t, apq, app);
                        aqq = fma(t, apq, aqq);
                        if (s != 0.0) apq = 0.0;
                    }
                    __syncthreads();
#pragma unroll
                    for (int q = 0; q < K; ++q)
                        if (ij[q] >= 0) {
                            const double2 x = cs[ij[q] & 255], y = cs[ij[q] >> 8];
                            const double r_pp = x.x * blk[q][0] - x.y * blk[q][2];
                            const double r_pq = x.x * blk[q][1] - x.y * blk[q][3];
                            const double r_qp = x.y * blk[q][0] + x.x * blk[q][2];
                            const double r_qq = x.y * blk[q][1] + x.x * blk[q][3];
                            A[wr[q][0]] = y.x * r_pp - y.y * r_pq;
                            A[wr[q][1]] = y.y * r_pp + y.x * r_pq;
                            A[wr[q][2]] = y.x * r_qp - y.y * r_qq;
                            A[wr[q][3]] = y.y * r_qp + y.x * r_qq;
                        }
                    if (dia) {
                        A[mp * ld + mp] = app;
                        A[mq * ld + mq] = aqq;
                        A[canon(mp, mq)] = apq;
                    }
                    __syncthreads();
                }
            }
            if (done) break;
        }
        if (tid < N) lam[tid] = slam[tid] = A[tid * ld + tid];
        __syncthreads();
    } else {
        double vp[VN], vq[VN];
#pragma unroll
        for (int q = 0; q < VN; ++q) {
            const int r = vr0 + VS * q;
            vp[q] = r == vj ? 1.0 : 0.0;
            vq[q] = r == Ne - 1 - vj ? 1.0 : 0.0;
        }
        const bool first = vj == 0, last = vj == half - 1;
        for (int sweep = 0; sweep < 40; ++sweep) {
            if (converged(0.0, 0.0)) break;
            for (int r = 0; r < Ne - 1; ++r) {
                __syncthreads();
                const double2 y = cs[min(vj, half - 1)];
#pragma unroll
                for (int q = 0; q < VN; ++q) {
                    if (vw + VS * q < N) {  // uniform over the wave
                        const double a = y.x * vp[q] - y.y * vq[q], b = y.y * vp[q] + y.x * vq[q];
                        const double up = wave_shift<kWaveShl1>(a), dn = wave_shift<kWaveShr1>(b);
                        vp[q] = first ? a : last ? b : up;
                        vq[q] = first ? (half == 1 ? b : up) : dn;
                    }
                }
                __syncthreads();
            }
        }
        __syncthreads();
        // U over A
        if (vj < half) {
#pragma unroll
            for (int q = 0; q < VN; ++q) {
                const int r = vr0 + VS * q;
                if (r < N) {
                    A[r * ld + vj] = vp[q];
                    A[r * ld + Ne - 1 - vj] = vq[q];
                    U[r * N + vj] = vp[q];
                    if (Ne - 1 - vj < N) U[r * N + Ne - 1 - vj] = vq[q];
                }
            }
        }
    }
    // eigenvalues, condition number, singularity test
    if (wave == 0) {
        double mn = NAN, mx = NAN;  // fmin and fmax pass over NaN
        for (int i = lane; i < N; i += 64) { mn = fmin(mn, slam[i]); mx = fmax(mx, slam[i]); }
        for (int d = 32; d; d >>= 1) {
            mn = fmin(mn, __shfl_xor(mn, d));
            mx = fmax(mx, __shfl_xor(mx, d));
        }
        if (lane == 0) {
            info[0] = mx / mn;
            info[1] = mn;
            sflag = !(mn > eig_floor);
            if (sflag) atomicOr(status, kStSingular);
        }
    }
    __syncthreads();
    if (sflag) return;
    if (tid < N) slam[tid] = 1.0 / sqrt(slam[tid]);
    __syncthreads();
    // Z = U diag(lam^{-1/2}) U^T ; Q = Z T
    mf_gemm<R>(N, [&](int i, int k) { return A[i * ld + k] * slam[k]; }, [&](int k, int j) { return A[j * ld + k]; },
               [&](int i, int j, double v) {
                   TG[i * tl + j] = v;
                   Z[i * N + j] = v;
               });
    __syncthreads();
    mf_gemm<R>(N, [&](int i, int k) { return TG[i * tl + k]; }, [&](int k, int j) { return T[k * N + j]; },
               [&](int i, int j, double v) { Qm[i * N + j] = v; });
}

// channel b's arrays at small + so[b] + the given offsets, its scratch at
// work + b * wstride
__global__ __launch_bounds__(kLwThreads) void k_lowdin_batch(LowdinBatch lb, double *small, LowdinOffsets off,
                                                             double *work, long long wstride, double eig_floor,
                                                             int *status) {
    extern __shared__ double dsm[];
    const int b = blockIdx.x;
    const int N = lb.N[b];
    double *sm = small + lb.so[b];
    if (N <= 64)
        lowdin_one<1>(N, sm + off.T, sm + off.G, sm + off.S, sm + off.lam, sm + off.U, sm + off.Z, sm + off.Q,
                      work + (size_t)b * wstride, dsm, eig_floor, status, sm + off.info);
    else
        lowdin_one<4>(N, sm + off.T, sm + off.G, sm + off.S, sm + off.lam, sm + off.U, sm + off.Z, sm + off.Q,
                      work + (size_t)b * wstride, dsm, eig_floor, status, sm + off.info);
}

__global__ __launch_bounds__(kLwThreads) void k_lowdin(int N, const double *T, const double *G, double *S,
                                                       double *lam, double *U, double *Z, double *Qm, double *work,
                                                       double eig_floor, int *status, double *info) {
    extern __shared__ double dsm[];
    if (N <= 64) lowdin_one<1>(N, T, G, S, lam, U, Z, Qm, work, dsm, eig_floor, status, info);
    else lowdin_one<4>(N, T, G, S, lam, U, Z, Qm, work, dsm, eig_floor, status, info);
}

// one matrix (N > 64) or two in LDS: at most 133 of the CU's 160 KB
static size_t lowdin_lds(int N) {
    const size_t Ne = N + (N & 1);
    return (N <= 64 ? 2 : 1) * Ne * (Ne + 1) * sizeof(double);
}

hipError_t launch_lowdin(int N, const double *T, const double *G, double *S, double *lam,
                         double *U, double *Z, double *Qm, double *work, double eig_floor,
                         int *status, double *info, hipStream_t s) {
    if (N < 1 || N > kMaxOrb) return hipErrorInvalidValue;
    const size_t dyn = lowdin_lds(N);
    const hipError_t e = allow_lds((const void *)k_lowdin, dyn);
    if (e) return e;
    hipLaunchKernelGGL(k_lowdin, dim3(1), dim3(kLwThreads), dyn, s, N, T, G, S, lam, U, Z, Qm, work, eig_floor,
                       status, info);
    return hipGetLastError();
}

hipError_t launch_lowdin_batch(const LowdinBatch &lb, double *small, const LowdinOffsets &off,
                               double *work, long long wstride, double eig_floor, int *status,
                               hipStream_t s) {
    if (lb.n <= 0 || lb.n > kLowdinBatch) return hipErrorInvalidValue;
    size_t dyn = 0;
    for (int b = 0; b < lb.n; ++b) dyn = std::max(dyn, lowdin_lds(lb.N[b]));
    const hipError_t e = allow_lds((const void *)k_lowdin_batch, dyn);
    if (e) return e;
    hipLaunchKernelGGL(k_lowdin_batch, dim3(lb.n), dim3(kLwThreads), dyn, s, lb, small, off, work, wstride,
                       eig_floor, status);
    return hipGetLastError();
}

// Reverse mode through Q = Z T, Z = S^{-1/2}, S = T G T^T, T_i = u_i/|u_i|.
//   Gam_T  = Z^T B + 2 Gam_S T G          (Gam_Q = B)
//   Gam_Z  = B T^T
//   Gam_S  = U [(U^T sym(Gam_Z) U) o K] U^T,
//            K_jk = -1 / (sqrt(l_j) sqrt(l_k) (sqrt(l_j) + sqrt(l_k)))
//   Gam_u_i = (Gam_T_i - (Gam_T_i . T_i) T_i) / |u_i|
//   dE/da_i = sum_a Gam_u_i,a grad psi_a(a_i)
// Bound by the latency of seven dependent products: the intermediate
// matrices are in LDS up to 64 orbitals, symmetrisation, the K factor and the
// sum ride in the products (N = 32 39 -> 15 us, N = 128 261 -> 37 us against
// scalar products in 256 threads).
template <int R>
__device__ __forceinline__ void lowdin_backward_one(int N, const double *B, const double *T, const double *G,
                                                    const double *lam, const double *U, const double *Z,
                                                    const double *rhoa, const double *du, double *work, double *dEda,
                                                    double *packed) {
    extern __shared__ double dsm[];
    __shared__ double sl[kMaxOrb];
    const int ld = R == 1 ? N | 1 : N;
    double *const w = R == 1 ? dsm : work;
    double *const GT = w, *const T1 = w + N * ld, *const T2 = w + 2 * N * ld, *const T3 = w + 3 * N * ld;
    if (threadIdx.x < N) sl[threadIdx.x] = sqrt(lam[threadIdx.x]);
    // T1 = Gam_Z, GT = Z^T B
    mf_gemm<R>(N, [&](int i, int k) { return B[i * N + k]; }, [&](int k, int j) { return T[j * N + k]; },
               [&](int i, int j, double v) { T1[i * ld + j] = v; });
    mf_gemm<R>(N, [&](int i, int k) { return Z[k * N + i]; }, [&](int k, int j) { return B[k * N + j]; },
               [&](int i, int j, double v) { GT[i * ld + j] = v; });
    __syncthreads();
    mf_gemm<R>(N, [&](int i, int k) { return U[k * N + i]; },
               [&](int k, int j) { return 0.5 * (T1[k * ld + j] + T1[j * ld + k]); },
               [&](int i, int j, double v) { T3[i * ld + j] = v; });
    __syncthreads();
    mf_gemm<R>(N, [&](int i, int k) { return T3[i * ld + k]; }, [&](int k, int j) { return U[k * N + j]; },
               [&](int i, int j, double v) { T2[i * ld + j] = -v / (sl[i] * sl[j] * (sl[i] + sl[j])); });
    __syncthreads();
    mf_gemm<R>(N, [&](int i, int k) { return U[i * N + k]; }, [&](int k, int j) { return T2[k * ld + j]; },
               [&](int i, int j, double v) { T1[i * ld + j] = v; });
    __syncthreads();
    mf_gemm<R>(N, [&](int i, int k) { return T1[i * ld + k]; }, [&](int k, int j) { return U[j * N + k]; },
               [&](int i, int j, double v) { T3[i * ld + j] = v; });  // Gam_S
    __syncthreads();
    mf_gemm<R>(N, [&](int i, int k) { return T3[i * ld + k]; }, [&](int k, int j) { return T[k * N + j]; },
               [&](int i, int j, double v) { T1[i * ld + j] = v; });
    __syncthreads();
    mf_gemm<R>(N, [&](int i, int k) { return T1[i * ld + k]; }, [&](int k, int j) { return G[k * N + j]; },
               [&](int i, int j, double v) { GT[i * ld + j] += 2.0 * v; });
    __syncthreads();
    // Gam_u and dE/da: a wave per orbital
    const int lane = threadIdx.x & 63;
    for (int i = threadIdx.x >> 6; i < N; i += kLwThreads / 64) {
        double dot = 0.0;
        for (int a = lane; a < N; a += 64) dot += GT[i * ld + a] * T[i * N + a];
        dot = wave_sum(dot);
        const double inv = 1.0 / sqrt(rhoa[i]);
        double gx = 0.0, gy = 0.0, gz = 0.0;
        for (int a = lane; a < N; a += 64) {
            const double gu = (GT[i * ld + a] - dot * T[i * N + a]) * inv;
            const double *const d = du + ((size_t)i * N + a) * 3;
            gx += gu * d[0];
            gy += gu * d[1];
            gz += gu * d[2];
        }
        gx = wave_sum(gx);
        gy = wave_sum(gy);
        gz = wave_sum(gz);
        if (lane == 0) {
            packed[3 * i] = dEda[3 * i] = gx;
            packed[3 * i + 1] = dEda[3 * i + 1] = gy;
            packed[3 * i + 2] = dEda[3 * i + 2] = gz;
        }
    }
}

// the reverse Loewdin step of up to kLowdinBatch channels in one launch, one
// workgroup each: channel b's B at Bm + b bstride, its small arrays at
// small + so[b], scratch at work + b wstride; dE/da to its small block and to
// packed + go[b] (all channels' gradients in one block for one copy)
__global__ __launch_bounds__(kLwThreads) void k_lowdin_backward_batch(LowdinBwdBatch lb, const double *Bm,
                                                                      long long bstride, double *small,
                                                                      LowdinBwdOffsets off, double *work,
                                                                      long long wstride, double *packed) {
    const int b = blockIdx.x;
    const int N = lb.N[b];
    double *sm = small + lb.so[b];
    const double *const B = Bm + (size_t)b * bstride;
    double *const w = work + (size_t)b * wstride;
    if (N <= 64)
        lowdin_backward_one<1>(N, B, sm + off.T, sm + off.G, sm + off.lam, sm + off.U, sm + off.Z, sm + off.rhoa,
                               sm + off.du, w, sm + off.dEda, packed + lb.go[b]);
    else
        lowdin_backward_one<2>(N, B, sm + off.T, sm + off.G, sm + off.lam, sm + off.U, sm + off.Z, sm + off.rhoa,
                               sm + off.du, w, sm + off.dEda, packed + lb.go[b]);
}

hipError_t launch_lowdin_backward_batch(const LowdinBwdBatch &lb, const double *Bm, long long bstride, double *small,
                                        const LowdinBwdOffsets &off, double *work, long long wstride, double *packed,
                                        hipStream_t s) {
    if (lb.n <= 0 || lb.n > kLowdinBatch) return hipErrorInvalidValue;
    size_t dyn = 0;
    for (int b = 0; b < lb.n; ++b)
        if (lb.N[b] <= 64) dyn = std::max(dyn, (size_t)4 * lb.N[b] * (lb.N[b] | 1) * sizeof(double));
    const hipError_t e = allow_lds((const void *)k_lowdin_backward_batch, dyn);
    if (e) return e;
    hipLaunchKernelGGL(k_lowdin_backward_batch, dim3(lb.n), dim3(kLwThreads), dyn, s, lb, Bm, bstride, small, off,
                       work, wstride, packed);
    return hipGetLastError();
}

}  // namespace fsic
