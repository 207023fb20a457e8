// Plain conjugate gradients for the per-orbital Poisson problems (Sec. II.A):
// the stencil sweep q = -L p with the p.q, r.q, q.q partials, and the pointwise
// update that also forms the next search direction.
#include "zmarch.h"

namespace fsic {

// x += alpha p; r -= alpha q; p = r + beta p (one node)
template <typename T>
__device__ __forceinline__ double upd_elem(T &x, T &r, T &p, T qv, T al, T be, int x_first) {
    x = x_first ? al * p : x + al * p;
    r = r - al * qv;
    p = r + be * p;
    return (double)r * (double)r;
}

// The fields of a block are loaded ahead of the scalars' reduction, and the
// four scalars are reduced together: small problems are bound by this chain
// of latencies (6 x 60x52x71: 14.7 -> 12.6 us a launch against four reductions one
// after the other and the loads behind them).
template <typename T>
__global__ __launch_bounds__(256) void k_cg_update(CGIter<T> a, int k, int cur_ru, int x_first) {
    using V = typename Vec16<T>::V;
    __shared__ double sred[4][4];
    const Item it = a.items8[blockIdx.x];
    if (it.orb < 0) return;
    if (a.done[it.orb]) return;
    const OrbDesc od = a.orb[it.orb];
    const bool restart = a.rs_iter && a.rs_iter[it.orb] == k;
    const bool from_ru = cur_ru || restart;
    const T *Pin = ((k == 0) || restart) ? a.R : a.P;  // p_k = r_k at a (re)start
    const long long M = (long long)od.nx * od.ny * od.nz;
    const long long base = (long long)it.tile * kPW;
    // |r_{k+1}|^2 = |r_k|^2 - 2 alpha r_k.q_k + alpha^2 |q_k|^2, so the next
    // direction is formed here; the direct r.r of this pass (below) decides
    // alpha and convergence of the next iteration
    T al, be;
    auto scalars = [&]() {
        const double *const p0 =
            from_ru ? a.partRU + od.base7 : a.part8 + (size_t)(k & 1) * a.tot8 + od.base8;
        const int n0 = from_ru ? od.nt7 : od.nt8;
        double v[4] = {0.0, 0.0, 0.0, 0.0};  // r.r, p.q, r.q, q.q
        for (int i = threadIdx.x; i < n0; i += 256) v[0] += p0[i];
        for (int i = threadIdx.x; i < od.nt7; i += 256)
#pragma unroll
            for (int d = 0; d < 3; ++d) v[1 + d] += a.part7[(size_t)d * a.tot7 + od.base7 + i];
#pragma unroll
        for (int d = 0; d < 4; ++d) v[d] = wave_sum(v[d]);
        if ((threadIdx.x & 63) == 0)
#pragma unroll
            for (int d = 0; d < 4; ++d) sred[d][threadIdx.x >> 6] = v[d];
        __syncthreads();
#pragma unroll
        for (int d = 0; d < 4; ++d) v[d] = (sred[d][0] + sred[d][1]) + (sred[d][2] + sred[d][3]);
        const double alpha = v[0] / v[1];
        const double rn = v[0] - 2.0 * alpha * v[2] + alpha * alpha * v[3];
        al = (T)alpha;
        be = (T)(rn > 0.0 ? rn / v[0] : 0.0);
    };
    double acc = 0.0;
    auto pass = [&](auto vtag) {
        using W = decltype(vtag);
        constexpr int VN = (int)(sizeof(W) / sizeof(T)), E = kPW / (256 * VN);
        // each thread owns VN consecutive nodes per step; positions past the
        // end read the last ones and are not stored
        W pv[E], qv[E], rv[E], xv[E];
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const long long i = base + (long long)(e * 256 + threadIdx.x) * VN;
            const long long g = od.off + (i < M ? i : M - VN);
            pv[e] = *reinterpret_cast<const W *>(Pin + g);
            qv[e] = *reinterpret_cast<const W *>(a.Q + g);
            rv[e] = *reinterpret_cast<const W *>(a.R + g);
            xv[e] = *reinterpret_cast<const W *>(a.X + g);
        }
        scalars();
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const long long i = base + (long long)(e * 256 + threadIdx.x) * VN;
            T *px = reinterpret_cast<T *>(&xv[e]), *pr = reinterpret_cast<T *>(&rv[e]);
            T *pp = reinterpret_cast<T *>(&pv[e]);
            const T *pq = reinterpret_cast<const T *>(&qv[e]);
            if (i < M) {
                const long long g = od.off + i;
#pragma unroll
                for (int j = 0; j < VN; ++j) acc += upd_elem(px[j], pr[j], pp[j], pq[j], al, be, x_first);
                *reinterpret_cast<W *>(a.X + g) = xv[e];
                *reinterpret_cast<W *>(a.R + g) = rv[e];
                *reinterpret_cast<W *>(a.P + g) = pv[e];
            }
        }
    };
    if (((od.off | M) % Vec16<T>::n) == 0) pass(V{});  // 16-byte vectors
    else pass(T{});
    __syncthreads();
    const double s = block_sum256(acc, &sred[0][0]);
    if (threadIdx.x == 0) {
        a.part8[(size_t)((k + 1) & 1) * a.tot8 + od.base8 + it.tile] = s;
        if (it.tile == 0) {
            a.nact[a.norb + it.orb] += 1;
            if (a.nsamp) a.nsamp[a.norb + it.orb] += 1;
        }
    }
}

template <typename T>
hipError_t launch_cg_stencil(int radius, const Coeffs &c, const CGIter<T> &a, int k,
                             int cur_from_ru, int check, hipStream_t s) {
    if (a.nitems7 <= 0) return hipSuccess;
    PolCG<T> pol{a.items7, a.orb, a, k, cur_from_ru, check, false, false};
#define CALL(P, C, DD) hipLaunchKernelGGL((k_zmarch<T, P, C, DD, PolCG<T>>), dim3(a.nitems7), dim3(256), 0, s, pol, c)
    FSIC_RADIUS_SWITCH(radius, CALL)
#undef CALL
    return hipGetLastError();
}

template <typename T>
hipError_t launch_cg_update(const CGIter<T> &a, int k, int cur_from_ru, int x_first,
                            hipStream_t s) {
    if (a.nitems8 <= 0) return hipSuccess;
    hipLaunchKernelGGL((k_cg_update<T>), dim3(a.nitems8), dim3(256), 0, s, a, k, cur_from_ru,
                       x_first);
    return hipGetLastError();
}

template hipError_t launch_cg_stencil<double>(int, const Coeffs &, const CGIter<double> &, int, int,
                                              int, hipStream_t);
template hipError_t launch_cg_stencil<float>(int, const Coeffs &, const CGIter<float> &, int, int,
                                             int, hipStream_t);
template hipError_t launch_cg_update<double>(const CGIter<double> &, int, int, int, hipStream_t);
template hipError_t launch_cg_update<float>(const CGIter<float> &, int, int, int, hipStream_t);

}  // namespace fsic
