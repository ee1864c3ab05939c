// Parameters and stencil helpers of the CCZ4 right-hand side on the device, and the form in which the
// kernels evaluate the closing relations of App. B of arXiv:2406.11626.
//
// The closing
// relations are evaluated in contracted form: with gt^ml gt_jl = delta^m_j the derivative of
// the physical Christoffel symbols reduces to
//   d_k Gamma^m_ij = d_k Gt^m_ij + 2 (D_kij P^m - gt_ij D_k^ml P_l)/phi
//                    - (delta^m_j dP_(ki) + delta^m_i dP_(kj) - gt_ij gt^ml dP_(kl))/phi
//                    + (delta^m_j P_i P_k + delta^m_i P_j P_k - gt_ij P_k P^m)/phi^2,
// and the two contractions the Ricci tensor needs are formed directly:
//   R_ij = sum_m d_m Gamma^m_ij - d_j (Gamma^m_im) + Gamma^l_ij Gamma^m_lm - Gamma^l_im Gamma^m_lj,
//   d_j Gamma^m_im = -2 D_j^ml D_iml + gt^ml (d_j D_iml + d_i D_jml)/2 - 3 dP_(ij)/phi + 3 P_i P_j/phi^2.
// T is, in the kernels, the type of the nonlinear algebra (double, or float in the mixed-precision mode);
// the inverse metric, its determinant and every factor of 1/phi are formed in double.
#pragma once
#include "ccz4_layout.hpp"

namespace ccz4 {

struct RhsParams {
    double kappa1, kappa2, kappa3, tau, e, c, mu, f, eta, ko_eps;
    int32_t slicing, shift;
    int32_t formulation;  // 0: first order (red terms on), 1: second order (red terms off, aux RHS 0)
    int32_t advection;    // 0: central FD4 advection; 1: lopsided, biased towards +x_k where beta^k > 0;
                          // 2: lopsided with the pairing as printed (towards -x_k where beta^k > 0)
    int32_t transfer;     // coarse-fine halo operators: 0 as printed in App. E; 1 injection + quadratic
};

// The lopsided fourth-order first derivatives of App. D, biased towards +x (points -1..+3) or
// towards -x (points -3..+1), written as the central difference cen plus a fifth difference:
//   right = cen + (-Q-- + 5Q- - 10Q + 10Q+ - 5Q++ + Q+++) / (12 dx),
//   left  = cen + (-Q--- + 5Q-- - 10Q- + 10Q - 5Q+ + Q++) / (12 dx),
// the second being the first mirrored; selecting the operands rather than the two results keeps
// one expression per lane (i12 = 1 / (12 dx)).
__device__ __forceinline__ double lop_from_central(double cen, bool right, double m3, double m2, double m1, double c0,
                                                   double p1, double p2, double p3, double i12)
{
    const double u3 = right ? p3 : -m3, u2 = right ? p2 : -m2, u1 = right ? p1 : -m1, u0 = right ? c0 : -c0;
    const double w1 = right ? m1 : -p1, w2 = right ? m2 : -p2;
    return cen + (u3 - 5.0 * u2 + 10.0 * u1 - 10.0 * u0 + 5.0 * w1 - w2) * i12;
}
// which of the two the advection term takes along an axis with shift component be
__device__ __forceinline__ bool lop_use_right(int32_t mode, double be) { return mode == 1 ? be > 0.0 : !(be > 0.0); }

template <typename T>
__device__ __forceinline__ T cvt(double x) { return static_cast<T>(x); }

}  // namespace ccz4
