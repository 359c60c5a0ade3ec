// rh_adjoint.hpp -- device arithmetic of the hand-written adjoint of L.
//
// With w a field of weights, sum_i w_i . L_i (Eq. (2) of Sikorski et al.,
// arXiv:1604.03360) equals the sum over faces of Fhat(i+1/2) . g(i+1/2) with
// g = (w_{i+1} - w_i) / h; its gradient with respect to the state is therefore
// built face by face: the gradient of each WENO reconstruction (Sec. 1.2) with
// respect to its stencil, scaled by g, is accumulated on the stencil cells, and
// each cell's accumulated split-flux adjoints a+- are mapped through the split
// f+- = (F(u) +- u)/2 and the flux Jacobian of F, whose primitive-recovery part
// comes from the per-cell pack below.
#pragma once
#include "rh_device.hpp"

namespace rh {

// Gradient of weno5 (difference form, see weno5) times gbar, added to out[0..4].
// With omega_k the nonlinear weights, dq_k the candidates minus the centre and
// G_k = 13/3 A_k^2 + B_k^2 + 4 eps:
//   d fhat / d s = e_2 + sum_k omega_k grad(dq_k)
//                  - 2 sum_k omega_k (dq_k - fhat + s2) / G_k grad(G_k),
//   grad(G_k) = 26/3 A_k grad(A_k) + 2 B_k grad(B_k).
template <class T>
__device__ __forceinline__ void weno5_grad_acc(T s0, T s1, T s2, T s3, T s4, T eps4, T gbar,
                                               T& o0, T& o1, T& o2, T& o3, T& o4) {
    const T E1 = s1 - s0, E2 = s2 - s1, E3 = s3 - s2, E4 = s4 - s3;
    const T dq0 = (T)(5.0 / 6.0) * E2 - (T)(1.0 / 3.0) * E1;
    const T dq1 = (T)(1.0 / 6.0) * E2 + (T)(1.0 / 3.0) * E3;
    const T dq2 = (T)(2.0 / 3.0) * E3 - (T)(1.0 / 6.0) * E4;
    const T A0 = E2 - E1, A1 = E3 - E2, A2 = E4 - E3;
    const T B0 = (T)3 * E2 - E1, B1 = E2 + E3, B2 = E4 - (T)3 * E3;
    const T c133 = (T)(13.0 / 3.0);
    const T G0 = (c133 * A0) * A0 + (B0 * B0 + eps4);
    const T G1 = (c133 * A1) * A1 + (B1 * B1 + eps4);
    const T G2 = (c133 * A2) * A2 + (B2 * B2 + eps4);
    const T g0 = G0 * G0, g1 = G1 * G1, g2 = G2 * G2;
    const T w0 = (T)0.1 * (g1 * g2), w1 = (T)0.6 * (g0 * g2), w2 = (T)0.3 * (g0 * g1);
    const T rs = fast_rcp(w0 + w1 + w2);
    const T om0 = w0 * rs, om1 = w1 * rs, om2 = w2 * rs;
    const T fd = om0 * dq0 + om1 * dq1 + om2 * dq2;
    const T c0 = (T)(-2.0) * om0 * (dq0 - fd) * fast_rcp(G0);
    const T c1 = (T)(-2.0) * om1 * (dq1 - fd) * fast_rcp(G1);
    const T c2 = (T)(-2.0) * om2 * (dq2 - fd) * fast_rcp(G2);
    const T pA0 = (T)(26.0 / 3.0) * c0 * A0, pA1 = (T)(26.0 / 3.0) * c1 * A1, pA2 = (T)(26.0 / 3.0) * c2 * A2;
    const T pB0 = (T)2 * c0 * B0, pB1 = (T)2 * c1 * B1, pB2 = (T)2 * c2 * B2;
    // grad(dq): (1/3, -7/6, 5/6, 0, 0), (0, -1/6, -1/6, 1/3, 0), (0, 0, -2/3, 5/6, -1/6)
    // grad(A):  (1, -2, 1, 0, 0), (0, 1, -2, 1, 0), (0, 0, 1, -2, 1)
    // grad(B):  (1, -4, 3, 0, 0), (0, -1, 0, 1, 0), (0, 0, 3, -4, 1)
    const T d0 = (T)(1.0 / 3.0) * om0 + pA0 + pB0;
    const T d1 = (T)(-7.0 / 6.0) * om0 - (T)(1.0 / 6.0) * om1 - (T)2 * pA0 + pA1 - (T)4 * pB0 - pB1;
    const T d2 = (T)1 + (T)(5.0 / 6.0) * om0 - (T)(1.0 / 6.0) * om1 - (T)(2.0 / 3.0) * om2 + pA0
               - (T)2 * pA1 + pA2 + (T)3 * pB0 + (T)3 * pB2;
    const T d3 = (T)(1.0 / 3.0) * om1 + (T)(5.0 / 6.0) * om2 + pA1 - (T)2 * pA2 + pB1 - (T)4 * pB2;
    const T d4 = (T)(-1.0 / 6.0) * om2 + pA2 + pB2;
    o0 += gbar * d0;
    o1 += gbar * d1;
    o2 += gbar * d2;
    o3 += gbar * d3;
    o4 += gbar * d4;
}

// The same gradient written in the first differences E_j and the completed
// squares A_k of the smoothness indicators (see weno5): fewer instructions, more
// live values; used where registers are plentiful.  With omega_k the
// nonlinear weights, dq_k the candidates minus the centre and G_k = h_k + e:
//   d fhat / d E_j = sum_k omega_k d dq_k/d E_j + sum_k c_k d h_k/d E_j,
//   c_k = -2 omega_k (dq_k - sum_m omega_m dq_m) / G_k,
// and d/d s follows from E_j = s_j - s_{j-1} (plus 1 on the centre s2).
template <class T>
__device__ __forceinline__ void weno5_grad_acc_e(T s0, T s1, T s2, T s3, T s4, T eps4, T gbar,
                                                 T& o0, T& o1, T& o2, T& o3, T& o4) {
    const T E1 = s1 - s0, E2 = s2 - s1, E3 = s3 - s2, E4 = s4 - s3;
    const T dq0 = (T)(5.0 / 6.0) * E2 - (T)(1.0 / 3.0) * E1;
    const T dq1 = (T)(1.0 / 6.0) * E2 + (T)(1.0 / 3.0) * E3;
    const T dq2 = (T)(2.0 / 3.0) * E3 - (T)(1.0 / 6.0) * E4;
    const T e = (T)0.1875 * eps4;
    const T A0 = E1 - (T)1.375 * E2, A1 = E2 - (T)0.625 * E3, A2 = E4 - (T)1.375 * E3;
    const T u2 = (T)0.609375 * E2, u3 = (T)0.609375 * E3;
    const T p2 = u2 * E2 + e, p3 = u3 * E3 + e;
    const T G0 = A0 * A0 + p2;
    const T G1 = A1 * A1 + p3;
    const T G2 = A2 * A2 + p3;
    const T g0 = G0 * G0, g1 = G1 * G1, g2 = G2 * G2;
    // 10 w = (g1 g2, 6 g0 g2, 3 g0 g1)
    const T p12 = g1 * g2, p02 = g0 * g2, p01 = g0 * g1;
    const T rs = fast_rcp((T)3 * p01 + ((T)6 * p02 + p12));
    const T om0 = p12 * rs, om1 = p02 * ((T)6 * rs), om2 = p01 * ((T)3 * rs);
    const T fd = om0 * dq0 + om1 * dq1 + om2 * dq2;
    const T gb4 = (T)(-4.0) * gbar;
    // 2 gbar c_k
    const T c0 = (gb4 * om0) * (dq0 - fd) * fast_rcp(G0);
    const T c1 = (gb4 * om1) * (dq1 - fd) * fast_rcp(G1);
    const T c2 = (gb4 * om2) * (dq2 - fd) * fast_rcp(G2);
    const T wb0 = gbar * om0, wb1 = gbar * om1, wb2 = gbar * om2;
    const T m0 = c0 * A0, m1 = c1 * A1, m2 = c2 * A2;
    const T gE1 = m0 - (T)(1.0 / 3.0) * wb0;
    const T gE2 = ((m1 - (T)1.375 * m0) + c0 * u2) + ((T)(5.0 / 6.0) * wb0 + (T)(1.0 / 6.0) * wb1);
    const T gE3 = ((c1 + c2) * u3 - ((T)0.625 * m1 + (T)1.375 * m2)) + ((T)(1.0 / 3.0) * wb1 + (T)(2.0 / 3.0) * wb2);
    const T gE4 = m2 - (T)(1.0 / 6.0) * wb2;
    o0 -= gE1;
    o1 += gE1 - gE2;
    o2 += gbar + (gE2 - gE3);
    o3 += gE3 - gE4;
    o4 += gE4;
}

// Gradient of weno7 times gbar, added to o[0..6], in the first differences D_j
// and the completed squares of the smoothness indicators (see smooth7; G_k is
// their g_k): with omega_k the nonlinear weights and dq_k the candidates minus
// the centre,
//   d fhat / d D_j = sum_k omega_k d dq_k/d D_j + sum_k c_k d G_k/d D_j,
//   c_k = -2 omega_k (dq_k - sum_m omega_m dq_m) / G_k,
// where the shared part q(D3, D2) of G_0 and G_1 takes c_0 + c_1 at once.  The
// weights are 1/G_k^2 with one reciprocal per indicator, which c_k needs as well,
// in FP32 scaled to d_k / (beta_k + eps)^2: their sum overflows where eps is below 1.4e-20
// and the data flat (unscaled already below 1.8e-19; the forward evaluates down to 2.4e-22).
// With tables of the derivatives of every candidate and indicator by every
// stencil value (zeros multiplied too) J^T w took 1099 us at 128^3 FP64 and 636 us
// in FP32, now 809 and 405.
template <class T>
__device__ __forceinline__ void weno7_grad_acc(const T s[7], T eps, T gbar, T o[7]) {
    constexpr double f = 240.0 / 547.0, r = 3167.0 / 2126.0;
    constexpr double c2 = 1063.0 / 1641.0 * f, c3 = 10153.0 / 12756.0 * f;
    const T D1 = s[1] - s[0], D2 = s[2] - s[1], D3 = s[3] - s[2], D4 = s[4] - s[3];
    const T D5 = s[5] - s[4], D6 = s[6] - s[5];
    const Smooth7<T> S = smooth7<T>(D1, D2, D3, D4, D5, D6, eps);
    const T dq0 = (T)0.25 * D1 - (T)(5.0 / 6.0) * D2 + (T)(13.0 / 12.0) * D3;
    const T dq1 = (T)(1.0 / 3.0) * D3 - (T)(1.0 / 12.0) * D2 + (T)0.25 * D4;
    const T dq2 = (T)(1.0 / 12.0) * (D3 - D5) + (T)0.5 * D4;
    const T dq3 = (T)0.75 * D4 - (T)(1.0 / 3.0) * D5 + (T)(1.0 / 12.0) * D6;
    const T r0 = fast_rcp(S.g0), r1 = fast_rcp(S.g1), r2 = fast_rcp(S.g2), r3 = fast_rcp(S.g3);
    constexpr double d = sizeof(T) == 4 ? f * f / 35.0 : 1.0;
    const T a0 = ((T)d * r0) * r0, a1 = ((T)(12.0 * d) * r1) * r1;
    const T a2 = ((T)(18.0 * d) * r2) * r2, a3 = ((T)(4.0 * d) * r3) * r3;
    const T rs = fast_rcp((a0 + a1) + (a2 + a3));
    const T om0 = a0 * rs, om1 = a1 * rs, om2 = a2 * rs, om3 = a3 * rs;
    const T fd = (om0 * dq0 + om1 * dq1) + (om2 * dq2 + om3 * dq3);
    const T w0 = gbar * om0, w1 = gbar * om1, w2 = gbar * om2, w3 = gbar * om3;
    // 2 gbar c_k
    const T b0 = (T)(-4) * w0 * (dq0 - fd) * r0, b1 = (T)(-4) * w1 * (dq1 - fd) * r1;
    const T b2 = (T)(-4) * w2 * (dq2 - fd) * r2, b3 = (T)(-4) * w3 * (dq3 - fd) * r3;
    const T n0 = b0 * S.l0, n1 = b1 * S.l1, n2 = b2 * S.l2, n3 = b3 * S.l3;
    // the shared squares: 2 c2 m_i (c + c') and 2 c3 D (c + c')
    const T bl = b0 + b1, br = b2 + b3;
    const T t1 = bl * ((T)c2 * S.m1), t2 = br * ((T)c2 * S.m2);
    const T g1 = n0 + (T)0.25 * w0;
    const T g2 = (t1 - (T)(1394.0 / 547.0) * n0 + (T)(247.0 / 547.0) * n1) -
                 ((T)(5.0 / 6.0) * w0 + (T)(1.0 / 12.0) * w1);
    const T g3 = (bl * ((T)c3 * D3) - (T)r * t1 + (T)(927.0 / 547.0) * n0 - (T)(714.0 / 547.0) * n1 + n2) +
                 ((T)(13.0 / 12.0) * w0 + (T)(1.0 / 3.0) * w1 + (T)(1.0 / 12.0) * w2);
    const T g4 = (br * ((T)c3 * D4) - (T)r * t2 + (T)(927.0 / 547.0) * n3 - (T)(714.0 / 547.0) * n2 + n1) +
                 ((T)0.25 * w1 + (T)0.5 * w2 + (T)0.75 * w3);
    const T g5 = (t2 - (T)(1394.0 / 547.0) * n3 + (T)(247.0 / 547.0) * n2) -
                 ((T)(1.0 / 12.0) * w2 + (T)(1.0 / 3.0) * w3);
    const T g6 = n3 + (T)(1.0 / 12.0) * w3;
    o[0] -= g1;
    o[1] += g1 - g2;
    o[2] += g2 - g3;
    o[3] += gbar + (g3 - g4);
    o[4] += g4 - g5;
    o[5] += g5 - g6;
    o[6] += g6;
}

// Primitive recovery written as v = kappa(E, M^2) M and p = P(E, M^2), with the
// four partial derivatives of kappa and P (FP64).  This covers the floors: below
// the energy floor kappa = 0 and P = max(E, 0)/3; above the velocity cap M is
// rescaled to |v| = 1 - delta, which makes kappa = K0/|M| and P = E delta/(1 +
// sqrt(1 + 3 delta)) with constants from the closed form.
struct RecoveryPack {
    double kap, p, kap_E, kap_M2, p_E, p_M2;
};

__device__ __forceinline__ RecoveryPack recovery_pack(double E, double Mx, double My, double Mz) {
    RecoveryPack o;
    if (E < kEFloor) {
        o.kap = 0.0;
        o.p = (E > 0.0 ? E : 0.0) / 3.0;
        o.kap_E = o.kap_M2 = o.p_M2 = 0.0;
        o.p_E = E > 0.0 ? 1.0 / 3.0 : 0.0;
        return o;
    }
    const double M2 = Mx * Mx + My * My + Mz * Mz;
    const double cap = (1.0 - kVDelta) * E * E;
    if (M2 > cap) {
        const double q = sqrt(1.0 + 3.0 * kVDelta);
        o.kap = 3.0 * sqrt(1.0 - kVDelta) / ((2.0 + q) * sqrt(M2));
        o.p = E * kVDelta / (1.0 + q);
        o.kap_E = 0.0;
        o.kap_M2 = -0.5 * o.kap / M2;
        o.p_E = kVDelta / (1.0 + q);
        o.p_M2 = 0.0;
        return o;
    }
    const double D = sqrt(4.0 * E * E - 3.0 * M2);
    const double a = 2.0 * E + D, b = E + D;
    const double r = fast_rcp(a * b * D);
    const double ra = b * D * r, rb = a * D * r, rD = a * b * r;
    o.kap = 3.0 * ra;
    o.p = (E * E - M2) * rb;
    o.kap_E = -(o.kap * o.kap / 3.0) * (2.0 + 4.0 * E * rD);
    o.kap_M2 = 0.5 * o.kap * o.kap * rD;
    o.p_E = (2.0 * E - o.p * (1.0 + 4.0 * E * rD)) * rb;
    o.p_M2 = (1.5 * o.p * rD - 1.0) * rb;
    return o;
}

}  // namespace rh
