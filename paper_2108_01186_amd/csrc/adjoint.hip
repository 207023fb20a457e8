// Reverse-mode FOD gradient of the discrete SIC energy (the FOD forces of
// Eq. 9-11, in exact form for this discretisation).
//
// With v_i = A rho_i, A = K^{-1} (4 pi I + C E_g P) (K = -L, C: ghost values
// into the right-hand side, E_g: moments to ghost values, P: density to
// moments), U_i = dV/2 rho_i^T A rho_i and dE_xc/drho = dV v_xc:
//   dE/dphi_i = Gam_i = 2 dV phi_i omega_i,
//   omega_i = -( (v_i + A^T rho_i) / 2 + v_xc(rho_i) ),
//   A^T rho = w' + dV sum_lm zt_lm r^l Y_lm,  K w' = 4 pi rho,
//   zt_lm = (1 / 4 pi) sum_ghost 4 pi/(2l+1) Y_lm / r^(l+1) (C^T w')_ghost.
// phi = Q psi gives B = Gam psi^T (products.hip); the rest is N x N
// (lowdin.hip): Q = Z T, Z = S^{-1/2} (Daleckii-Krein form of the derivative
// of the inverse square root), S = T G T^T, T_i = u_i / |u_i|,
// u_i,a = psi_a(a_i) (cubic interpolant).
#include <algorithm>
#include <cstdint>

#include "kernels.h"
#include "lsda.h"

namespace fsic {

// Gam_i(m) = 2 dV phi_i omega_i, omega_i = -((v_i + w_i) / 2 + vxc(phi_i^2)),
// over the channel's N x M values (Gam may be W: each value is read before
// it is written, by the same thread)
__global__ __launch_bounds__(256) void k_gamma(long long count, double dV, const double *PHI,
                                               const double *V, const double *W, double floor,
                                               double *Gam) {
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < count; i += (long long)gridDim.x * 256) {
        const double ph = PHI[i];
        const double om = -(0.5 * (V[i] + W[i]) + vxc_pol(ph * ph, floor));
        Gam[i] = 2.0 * dV * ph * om;
    }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------

hipError_t launch_gamma(long long count, double dV, const double *PHI, const double *V, const double *W, double floor,
                        double *Gam, hipStream_t s) {
    if (count < 1) return hipErrorInvalidValue;
    const long long gblk = std::min((count + 255) / 256, 4096LL);
    hipLaunchKernelGGL(k_gamma, dim3((unsigned)gblk), dim3(256), 0, s, count, dV, PHI, V, W, floor, Gam);
    return hipGetLastError();
}

}  // namespace fsic
