// rh_device.hpp -- device arithmetic of one WENO sweep for gfx950.
//
// Per cell: FP64 closed-form primitive recovery for the conformal equation of
// state (p = e/3), the physical flux along the sweep axis (Eq. (1) of
// Sikorski et al., arXiv:1604.03360), global Lax-Friedrichs splitting with
// alpha = 1, and finite-difference WENO5 / WENO7 reconstruction with Jiang-Shu
// smoothness indicators (Sec. 1.2).  Templated on the storage/stencil type T
// (float or double); the primitive recovery is always FP64.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace rh {

// Floors of the primitive recovery (they never modify the stored state).
constexpr double kEFloor = 1e-12;   // below this E the cell is treated as at rest
constexpr double kVDelta = 1e-12;   // |M|^2 is capped at (1 - kVDelta) E^2

struct HubbleBC {
    double t;          // stage time
    double t0, e0, n0; // u^mu = x^mu/tau, e = e0 (t0/tau)^4, n = n0 (t0/tau)^3
    double c0[3];      // centre of cell (0,0,0)
    double h[3];       // cell widths
};

// Last SSP-RK3 stage, u^n / 3 + 2/3 (u2 + dt L(u2)) with v = u2 + dt L(u2),
// evaluated in increment form u^n + 2/3 (v - u^n).  The plain form's rounded
// weights sum to 1 + 3e-8 in FP32, which scales every state (and the totals of
// a periodic grid) by that factor each step; in increment form the rounding of
// 2/3 multiplies only the increment and a uniform state stays exactly uniform.
template <class T>
__device__ __forceinline__ T rk3_last(T un, T v) { return un + (T)(2.0 / 3.0) * (v - un); }

// Reciprocals.  FP32: the hardware reciprocal (about 1 ulp).  FP64: the
// hardware estimate (measured within 2^-24.4) with one third-order step,
// e = 1 - x r, r (1 + e + e^2), for the normal-range arguments used here (weight
// sums, (2E + D)(E + D)).  Over 4e6 arguments of 1e-24 .. 1e24 its error is that
// of two Newton steps (largest 1.11e-16, rms 4.9e-17 relative), one operation
// less.
__device__ __forceinline__ float fast_rcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ double fast_rcp(double x) {
    const double r = __builtin_amdgcn_rcp(x);
    const double e = fma(-x, r, 1.0);
    return fma(r, fma(e, e, e), r);
}

// Square root of a positive normal double (no rescaling of tiny or huge
// arguments, no special cases): the hardware reciprocal square root y (measured
// within 2^-24.2) refined by one coupled Goldschmidt step on (g, h) ~ (sqrt(x),
// 1/(2 sqrt(x))) and one Newton correction g <- g + (x - g^2) h.  Over 4e6
// arguments the error is within 1.11e-16, rms 4.6e-17 relative, as with a second
// correction.  Used for 4E^2 - 3M^2 >= E^2 with E above the floor, which is
// always in the normal range.
__device__ __forceinline__ double sqrt_pos(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    double g = x * y, h = 0.5 * y;
    const double r = fma(-g, h, 0.5);
    g = fma(g, r, g);
    h = fma(h, r, h);
    const double d = fma(-g, g, x);
    return fma(d, h, g);
}

// Analytic Hubble-like flow at (x, y, z, t), converted to conserved variables.
// With v = x/t the Lorentz factor is |t|/tau, and only q = 1/tau^2 = 1/(t^2 - r^2) is
// needed: (t0/tau)^2 = t0^2 q, gamma^2 = t^2 q.  The ghost cells of a tile's edge are
// evaluated by a few lanes while their wave waits, so the length of this chain is what
// counts, with its registers where the stage spills: no root and no other division
// (128^3 step with two roots and six divisions 525 us in FP64 and 352 us in FP32, with one
// reciprocal root in their place 511 and 333).  The energy holds q to the third power, so
// the rounding of the last and largest sum in r^2 is taken off tau^2: the error of E is
// 2.8e-16 rms and 1.3e-15 at most for |x|, |y|, |z| <= 5, t = 10 .. 11 (1.5e-15 at most
// without it; the formulas as they are written, with roots and divisions, 3.6e-16 and
// 1.4e-15; from one reciprocal root 4.7e-16 and 1.9e-15, at 458 us per 128^3 step of the
// fused stage in FP64 and 276 us in FP32, now 447 and 273).  Taking off all of the rounding
// spills 8 - 12 more registers there and costs 4 - 9% of the step.
__device__ inline void hubble_conserved(const HubbleBC& hb, double x, double y, double z,
                                        double u[5]) {
    const double t = hb.t;
    const double b = fma(y, y, z * z), r2 = fma(x, x, b);
    const double tau2 = fma(t, t, -r2) - fma(x, x, b - r2);
    // reciprocal from the square of the hardware's reciprocal root (within 2^-23) and one
    // third-order step; not a number outside the light cone, as the flow is there
    const double y0 = __builtin_amdgcn_rsq(tau2), r0 = y0 * y0;
    const double e = fma(-tau2, r0, 1.0);
    const double q = fma(r0, fma(e, e, e), r0);
    const double s2 = (hb.t0 * hb.t0) * q, g = t * q;
    const double p = hb.e0 * (s2 * s2) * (1.0 / 3.0);
    const double k = 4.0 * p * g;   // (e + p) gamma^2 / t
    u[0] = k * t - p;
    u[1] = k * x;
    u[2] = k * y;
    u[3] = k * z;
    u[4] = hb.n0 * s2 * (hb.t0 * fabs(g));
}

// Closed-form primitive recovery for p = e/3 (FP64):
//   M^2 = |M|^2, D = sqrt(4E^2 - 3M^2), v = 3M/(2E + D), p = (E^2 - M^2)/(E + D).
// v = kap M, and both divisions share one (Newton-refined) reciprocal of
// (2E + D)(E + D).
__device__ __forceinline__ void recover_closed(double E, double E2, double M2, double& kap, double& p) {
    const double D = sqrt_pos(4.0 * E2 - 3.0 * M2);
    const double a = 2.0 * E + D;
    const double b = E + D;
    const double r = fast_rcp(a * b);
    kap = 3.0 * b * r;
    p = (E2 - M2) * a * r;
}

// The recovery for all three axes: kap and the (capped) momenta such that
// v_d = kap * Ms_d.  Vacuum and superluminal states are rare, so the closed form is
// evaluated for every lane and one branch then mends the lanes that hold them:
// fewer exec-mask updates than a branch for each kind around the closed form, and the
// same bits.  Per step, branches around -> one branch after, us: MUSTA-FORCE 128^3
// FP64 507 -> 488, FP32 392 -> 372, 24^3 33.4 -> 30.6; WENO5 192^3 FP64 1496 -> 1478.
// TIGHT keeps the branches around it, which hold fewer registers: the fused FP64 stage
// with analytic ghosts spills more otherwise (128^3 WENO5 448 us, 452 with one branch).
template <bool TIGHT = false>
__device__ __forceinline__ void recover_kp3(double E, double Mx, double My, double Mz, double& kap,
                                            double& Mxs, double& Mys, double& Mzs, double& p,
                                            unsigned& clamped) {
    if constexpr (TIGHT) {
        if (E < kEFloor) {
            kap = 0.0;
            Mxs = 0.0;
            Mys = 0.0;
            Mzs = 0.0;
            p = (E > 0.0 ? E : 0.0) / 3.0;
            ++clamped;
            return;
        }
    }
    double M2 = Mx * Mx + My * My + Mz * Mz;
    const double E2 = E * E;
    const double cap = (1.0 - kVDelta) * E * E;
    Mxs = Mx;
    Mys = My;
    Mzs = Mz;
    if constexpr (TIGHT) {
        if (M2 > cap) {
            const double sc = sqrt(cap / M2);
            Mxs *= sc;
            Mys *= sc;
            Mzs *= sc;
            M2 = cap;
            ++clamped;
        }
        recover_closed(E, E2, M2, kap, p);
    } else {
        recover_closed(E, E2, M2, kap, p);
        if (__builtin_expect(E < kEFloor || M2 > cap, 0)) {
            if (E < kEFloor) {
                kap = 0.0;
                Mxs = 0.0;
                Mys = 0.0;
                Mzs = 0.0;
                p = (E > 0.0 ? E : 0.0) / 3.0;
            } else {
                const double sc = sqrt(cap / M2);
                Mxs *= sc;
                Mys *= sc;
                Mzs *= sc;
                recover_closed(E, E2, cap, kap, p);
            }
            ++clamped;
        }
    }
}

// Velocity along one axis and p.
template <int DIR, bool TIGHT = false>
__device__ __forceinline__ void recover_vp(double E, double Mx, double My, double Mz,
                                           double& vd, double& p, unsigned& clamped) {
    double kap, Mxs, Mys, Mzs;
    recover_kp3<TIGHT>(E, Mx, My, Mz, kap, Mxs, Mys, Mzs, p, clamped);
    vd = kap * (DIR == 0 ? Mxs : (DIR == 1 ? Mys : Mzs));
}

// Two sweep axes at once (each v_d is bitwise the value recover_vp<d> returns).
template <bool TIGHT = false>
__device__ __forceinline__ void recover_kp(double E, double Mx, double My, double Mz, double& kap,
                                           double& Mxs, double& Mys, double& p, unsigned& clamped) {
    double Mzs;
    recover_kp3<TIGHT>(E, Mx, My, Mz, kap, Mxs, Mys, Mzs, p, clamped);
}

// Ideal-gas equation of state (unit rest mass per unit charge):
// p = (gamma - 1)(e - n), cut off at zero pressure; c_s^2 = gamma p / (e + p).
__device__ __forceinline__ double ideal_p(double gm1, double e, double n) {
    const double p = gm1 * (e - n);
    return p > 0.0 ? p : 0.0;
}

// Ideal-gas primitive recovery (FP64), in the form of recover_kp3: v_d =
// kap * Ms_d, with e and p.  The speed v along M solves
//   g(v) = v (E + p(E - |M| v, N sqrt(1 - v^2))) - |M| = 0,
// g increasing on [0, 1) (dg/dv >= E - (gamma - 1)|M| > 0 for gamma <= 2), with
// the root inside [|M| / (gamma E), |M| / E] because 0 <= p <= (gamma - 1) E.
// Newton steps, kept inside the shrinking bracket (a step leaving it is
// replaced by bisection), stop at a relative step of at most 1e-15.  They start from
// the root for the same fluid without rest mass (n = 0, p = (gamma - 1) e), the
// smaller root of (gamma - 1)|M| v^2 - gamma E v + |M| = 0, which lies in the
// bracket and is exact when N = 0.
// Floors as the closed form: E below the floor -> at rest; |M|^2 capped.
__device__ inline void recover_ideal(double E, double Mx, double My, double Mz, double N, double gm1,
                                     double& kap, double& Mxs, double& Mys, double& Mzs, double& p,
                                     double& e, unsigned& clamped) {
    if (E < kEFloor) {
        kap = 0.0;
        Mxs = Mys = Mzs = 0.0;
        e = E > 0.0 ? E : 0.0;
        p = ideal_p(gm1, e, N);
        ++clamped;
        return;
    }
    double M2 = Mx * Mx + My * My + Mz * Mz;
    const double cap = (1.0 - kVDelta) * E * E;
    Mxs = Mx;
    Mys = My;
    Mzs = Mz;
    if (M2 > cap) {
        const double sc = sqrt(cap / M2);
        Mxs *= sc;
        Mys *= sc;
        Mzs *= sc;
        M2 = cap;
        ++clamped;
    }
    if (!(M2 > 0.0)) {
        kap = 0.0;
        e = E;
        p = ideal_p(gm1, E, N);
        return;
    }
    const double M = sqrt(M2);
    const double ge = (gm1 + 1.0) * E;
    double lo = M / ge, hi = M / E;
    // 2|M| / (gamma E + sqrt(gamma^2 E^2 - 4 (gamma - 1) M^2)); the radicand is at
    // least (2 - gamma)^2 E^2 >= 0
    const double rad = ge * ge - 4.0 * gm1 * M2;
    double v = 2.0 * M / (ge + sqrt(rad > 0.0 ? rad : 0.0));
    v = v < lo ? lo : (v > hi ? hi : v);
#pragma unroll 1
    for (int it = 0; it < 80; ++it) {
        const double w = sqrt_pos(1.0 - v * v);
        const double pr = gm1 * ((E - M * v) - N * w);
        double g, dg;
        if (pr > 0.0) {
            g = v * (E + pr) - M;
            dg = (E + pr) + v * gm1 * (N * v * fast_rcp(w) - M);
        } else {
            g = v * E - M;
            dg = E;
        }
        if (g == 0.0) break;
        if (g > 0.0) hi = v;
        else lo = v;
        const double vn = v - g * fast_rcp(dg);
        // converged: tested before the bracket, since a step below the rounding
        // of v lands on v itself, the end of the bracket just moved there
        if (fabs(vn - v) <= 1e-15 * v) {
            v = vn;
            break;
        }
        v = vn > lo && vn < hi ? vn : 0.5 * (lo + hi);
    }
    kap = v / M;
    e = E - M * v;
    p = ideal_p(gm1, e, N * sqrt(1.0 - v * v));
}

// Largest characteristic speed along an axis, from the velocity along it, v^2
// and c_s^2: the acoustic eigenvalues
//   (v_d (1 - c^2) +- c sqrt((1 - v^2)(1 - v^2 c^2 - v_d^2 (1 - c^2)))) / (1 - v^2 c^2)
// bracket v_d, so the larger magnitude of the two bounds every wave.
__device__ __forceinline__ double max_char_speed(double vd, double v2, double cs2) {
    const double disc = cs2 * (1.0 - v2) * (1.0 - v2 * cs2 - vd * vd * (1.0 - cs2));
    const double root = sqrt(disc > 0.0 ? disc : 0.0);
    const double a = vd * (1.0 - cs2);
    return (fabs(a) + root) / (1.0 - v2 * cs2);
}

// Split fluxes f+- = (F_d(u) +- u) / 2 of one cell along axis DIR, given the
// velocity along DIR and the pressure, returned doubled (F_d +- u).
//
// The forward sweeps work with twice the split fluxes, F +- u: the WENO
// reconstruction is homogeneous of degree one when eps scales with the square
// of the data, so reconstructing F +- u with 4 eps gives exactly (all scalings
// are powers of two) twice the face flux, and the factor 1/2 is folded into
// the flux difference.
template <class T, int DIR>
__device__ __forceinline__ void split_flux_vp(const T u[5], T v, T P, T fp[5], T fm[5]) {
    T f[5];
    f[0] = u[1 + DIR];
    f[1] = u[1] * v + (DIR == 0 ? P : (T)0);
    f[2] = u[2] * v + (DIR == 1 ? P : (T)0);
    f[3] = u[3] * v + (DIR == 2 ? P : (T)0);
    f[4] = u[4] * v;
#pragma unroll
    for (int c = 0; c < 5; ++c) {
        fp[c] = f[c] + u[c];
        fm[c] = f[c] - u[c];
    }
}

template <class T, int DIR>
__device__ __forceinline__ void split_flux(const T u[5], T fp[5], T fm[5], unsigned& clamped) {
    double vd, p;
    recover_vp<DIR>((double)u[0], (double)u[1], (double)u[2], (double)u[3], vd, p, clamped);
    split_flux_vp<T, DIR>(u, (T)vd, (T)p, fp, fm);
}

// WENO5: s0..s4 = f_{i-2..i+2}; left-biased value at i+1/2 (Jiang-Shu).
// Written in the differences E_j = s_j - s_{j-1} about the centre c = s2:
//   q_k - c:  (-E1/3 + 5 E2/6), (E2/6 + E3/3), (2 E3/3 - E4/6)
//   beta_k = 13/12 A_k^2 + 1/4 B_k^2 with A = (E2-E1, E3-E2, E4-E3),
//            B = (3E2-E1, E2+E3, E4-3E3).
// Completing the square in the outer difference, 4 beta_k = 16/3 h_k with
//   h0 = (E1 - 11/8 E2)^2 + c E2^2,  h1 = (E2 - 5/8 E3)^2 + c E3^2,
//   h2 = (E4 - 11/8 E3)^2 + c E3^2,  c = 39/64
// (the remainder is the least energy given the difference that two
// neighbouring candidates share, so h1 and h2 have it in common, and c is the same
// for all).  FP64 evaluates these; FP32 keeps the expanded forms
//   h0 = E1^2 - 11/4 E1 E2 + 5/2 E2^2,  h1 = E2^2 - 5/4 E2 E3 + E3^2,
//   h2 = E4^2 - 11/4 E3 E4 + 5/2 E3^2,
// one operation more (256^3 step 1870 against 1815 us), so that single-precision
// runs keep their bits.  Then
// g_k = (h_k + 3/16 (4 eps))^2 is (3/16)^2 (4 eps + 4 beta_k)^2 and the common
// factor cancels in the weights
// alpha_k = d_k / (eps + beta_k)^2, d = (1, 6, 3)/10, which are evaluated with
// one reciprocal and carried as 10 w = (g1 g2, 6 g0 g2, 3 g0 g1), the factors 6
// and 3 folded into the candidates of the numerator:
//   num = g2 (g1 dq0 + g0 (6 dq1)) + g0 g1 (3 dq2),  den = g2 (g1 + 6 g0) + 3 g0 g1.
template <class T>
__device__ __forceinline__ T weno5(T s0, T s1, T s2, T s3, T s4, T eps4) {
    const T E1 = s1 - s0, E2 = s2 - s1, E3 = s3 - s2, E4 = s4 - s3;
    const T dq0 = (T)(5.0 / 6.0) * E2 - (T)(1.0 / 3.0) * E1;   // q0 - c
    const T dq1s = E2 + (T)2 * E3;                              // 6 (q1 - c)
    const T dq2s = (T)2 * E3 - (T)0.5 * E4;                     // 3 (q2 - c)
    const T e = (T)0.1875 * eps4;
    T g0, g1, g2;
    if constexpr (sizeof(T) == 4) {
        g0 = E1 * (E1 - (T)2.75 * E2) + ((T)2.5 * E2 * E2 + e);
        g1 = E2 * (E2 - (T)1.25 * E3) + (E3 * E3 + e);
        g2 = E4 * (E4 - (T)2.75 * E3) + ((T)2.5 * E3 * E3 + e);
    } else {
        const T p2 = ((T)0.609375 * E2) * E2 + e, p3 = ((T)0.609375 * E3) * E3 + e;
        const T a0 = E1 - (T)1.375 * E2, a1 = E2 - (T)0.625 * E3, a2 = E4 - (T)1.375 * E3;
        g0 = a0 * a0 + p2;
        g1 = a1 * a1 + p3;
        g2 = a2 * a2 + p3;
    }
    g0 *= g0;
    g1 *= g1;
    g2 *= g2;
    const T a = g0 * g1;
    const T num = g2 * (g1 * dq0 + g0 * dq1s) + a * dq2s;
    const T den = g2 * ((T)6 * g0 + g1) + (T)3 * a;
    return s2 + num * fast_rcp(den);
}

// Smoothness of the four WENO7 candidates in the differences D1..D6 of the
// stencil.  beta_k is the sum of the cell integrals of the squared first three
// derivatives of the cubic on its four cells, a quadratic form in its three
// differences.  Completing the square in the outermost one leaves the least value over the
// cubics through the other three cells, which two neighbouring candidates share:
//   240/547 beta_0 = l0^2 + q(D3, D2),  240/547 beta_1 = l1^2 + q(D3, D2),
//   240/547 beta_2 = l2^2 + q(D4, D5),  240/547 beta_3 = l3^2 + q(D4, D5),
//   l0 = D1 + (927 D3 - 1394 D2)/547,  l1 = D4 + (247 D2 - 714 D3)/547 and
//   mirrored, q(a, b) = c2 (b - r a)^2 + c3 a^2, r = 3167/2126,
//   c2 = 1063/1641 * 240/547, c3 = 10153/12756 * 240/547.
// The factor 240/547 (on eps too) cancels in the weights.  22 operations for all
// four, no cancellation; the derivative coefficients squared took 46 and the
// expanded forms 36.
template <class T>
struct Smooth7 {
    T l0, l1, l2, l3;   // the completed squares
    T m1, m2;           // D2 - r D3 and D5 - r D4
    T g0, g1, g2, g3;   // 240/547 (beta_k + eps)
};
template <class T>
__device__ __forceinline__ Smooth7<T> smooth7(T D1, T D2, T D3, T D4, T D5, T D6, T eps) {
    constexpr double f = 240.0 / 547.0, r = 3167.0 / 2126.0;
    constexpr double c2 = 1063.0 / 1641.0 * f, c3 = 10153.0 / 12756.0 * f;
    const T e = (T)f * eps;
    Smooth7<T> o;
    o.m1 = D2 - (T)r * D3;
    o.m2 = D5 - (T)r * D4;
    const T q1 = ((T)c2 * o.m1) * o.m1 + (((T)c3 * D3) * D3 + e);
    const T q2 = ((T)c2 * o.m2) * o.m2 + (((T)c3 * D4) * D4 + e);
    o.l0 = (D1 + (T)(927.0 / 547.0) * D3) - (T)(1394.0 / 547.0) * D2;
    o.l1 = (D4 + (T)(247.0 / 547.0) * D2) - (T)(714.0 / 547.0) * D3;
    o.l2 = (D3 + (T)(247.0 / 547.0) * D5) - (T)(714.0 / 547.0) * D4;
    o.l3 = (D6 + (T)(927.0 / 547.0) * D4) - (T)(1394.0 / 547.0) * D5;
    o.g0 = o.l0 * o.l0 + q1;
    o.g1 = o.l1 * o.l1 + q1;
    o.g2 = o.l2 * o.l2 + q2;
    o.g3 = o.l3 * o.l3 + q2;
    return o;
}

// WENO7: s0..s6 = f_{i-3..i+3}; linear weights d = (1, 12, 18, 4)/35.  With
// D_j = s_j - s_{j-1} and c = s3, the candidates are c + dq_k; 35 d is folded
// into the candidates, q_k = 35 d_k dq_k, and the weight sum.
template <class T>
__device__ __forceinline__ T weno7(T s0, T s1, T s2, T s3, T s4, T s5, T s6, T eps) {
    const T D1 = s1 - s0, D2 = s2 - s1, D3 = s3 - s2, D4 = s4 - s3, D5 = s5 - s4, D6 = s6 - s5;
    const T q0 = (T)0.25 * D1 - (T)(5.0 / 6.0) * D2 + (T)(13.0 / 12.0) * D3;
    const T q1 = ((T)4 * D3 - D2) + (T)3 * D4;
    const T q2 = (T)1.5 * (D3 - D5) + (T)9 * D4;
    const T q3 = ((T)3 * D4 - (T)(4.0 / 3.0) * D5) + (T)(1.0 / 3.0) * D6;
    if constexpr (sizeof(T) == 8) {
        // FP64: one reciprocal, the weights multiplied through by g0 g1 g2 g3
        const Smooth7<T> S = smooth7<T>(D1, D2, D3, D4, D5, D6, eps);
        const T g0 = S.g0 * S.g0, g1 = S.g1 * S.g1, g2 = S.g2 * S.g2, g3 = S.g3 * S.g3;
        const T g01 = g0 * g1, g23 = g2 * g3;
        const T num = g23 * (g1 * q0 + g0 * q1) + g01 * (g3 * q2 + g2 * q3);
        const T den = g23 * (g1 + (T)12 * g0) + g01 * ((T)18 * g3 + (T)4 * g2);
        return s3 + num * fast_rcp(den);
    } else {
        // FP32: 240 beta_k as quadratic forms in its three differences
        // (x, y, z) = (D_{k+1}, D_{k+2}, D_{k+3}); the factor 240 (on eps too)
        // cancels in the weights.  Rounding in the terms grows by at most the ratio
        // of the summed absolute coefficients to 240 (68 for the outer stencils): a
        // few 1e-6 relative in beta, far below the parity bar.  The completed
        // squares take 12 operations less; the expanded forms stay so that
        // single-precision runs keep their bits.
        const T e = (T)240 * eps;
        auto q = [e](T x, T y, T z, T cxx, T cxy, T cxz, T cyy, T cyz, T czz) {
            return x * (cxx * x + cxy * y + cxz * z) + (y * (cyy * y + cyz * z) + (czz * z * z + e));
        };
        T g0 = q(D1, D2, D3, (T)547, (T)-2788, (T)1854, (T)3708, (T)-5188, (T)2107);
        T g1 = q(D2, D3, D4, (T)267, (T)-1108, (T)494, (T)1468, (T)-1428, (T)547);
        T g2 = q(D3, D4, D5, (T)547, (T)-1428, (T)494, (T)1468, (T)-1108, (T)267);
        T g3 = q(D4, D5, D6, (T)2107, (T)-5188, (T)1854, (T)3708, (T)-2788, (T)547);
        g0 *= g0;
        g1 *= g1;
        g2 *= g2;
        g3 *= g3;
        // products of three squared terms can overflow, so one reciprocal per weight
        const T r0 = fast_rcp(g0), r1 = fast_rcp(g1), r2 = fast_rcp(g2), r3 = fast_rcp(g3);
        const T num = (r0 * q0 + r1 * q1) + (r2 * q2 + r3 * q3);
        const T den = (r0 + (T)12 * r1) + ((T)18 * r2 + (T)4 * r3);
        return s3 + num * fast_rcp(den);
    }
}

}  // namespace rh
