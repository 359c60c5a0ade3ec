// rh_face.hpp -- the numerical flux of one face: WENO reconstructions of split
// fluxes (Sec. 1.2 of Sikorski et al., arXiv:1604.03360), with alpha per face for
// local splitting, and the MUSCL + MUSTA-FORCE flux (Sec. 1.1).
#pragma once
#include "rh_device.hpp"
#include "../../include/rh.h"

namespace rh {

// Equations of state of the kernels (the values of RH_EOS_*).
enum { EOS_CONFORMAL = 0, EOS_IDEAL = 1 };

// One reconstruction from a window of 2R doubled split fluxes of cells
// i - R + 1 .. i + R (interface i + 1/2): plus = left-biased on f+, minus =
// mirrored on f-.  eps2 is the epsilon of the doubled data (4 eps); WENO5
// carries its smoothness indicators as 4 beta and takes 4 eps2.
template <class T, int ORDER>
__device__ __forceinline__ T stage_recon_plus(const T* w, T eps2) {
    if constexpr (ORDER == 5) return weno5<T>(w[0], w[1], w[2], w[3], w[4], (T)4 * eps2);
    else return weno7<T>(w[0], w[1], w[2], w[3], w[4], w[5], w[6], eps2);
}
template <class T, int ORDER>
__device__ __forceinline__ T stage_recon_minus(const T* w, T eps2) {
    if constexpr (ORDER == 5) return weno5<T>(w[5], w[4], w[3], w[2], w[1], (T)4 * eps2);
    else return weno7<T>(w[7], w[6], w[5], w[4], w[3], w[2], w[1], eps2);
}

// One face from the staged pairs of its 2R stencil cells: global splitting
// stages (F + u, F - u) and reconstructs them directly; local splitting stages
// (F, u) and reconstructs F +- alpha u with alpha the largest speed of the 2R
// cells.
template <class T, int ORDER>
__device__ __forceinline__ T recon_local(const T* wa, const T* wb, T alpha, T eps2) {
    constexpr int W = ORDER + 1;
    T wp[W], wm[W];
#pragma unroll
    for (int j = 0; j < W; ++j) {
        wp[j] = wa[j] + alpha * wb[j];
        wm[j] = wa[j] - alpha * wb[j];
    }
    return stage_recon_plus<T, ORDER>(wp, eps2) + stage_recon_minus<T, ORDER>(wm, eps2);
}

// Limiter and stage count of a kernel instance: fixed at compile time for the
// default scheme (minmod, two stages: straight-line face code), read from the
// grid entry otherwise.
constexpr int kAnyLimiter = -1, kAnyStages = 0, kAnyAxis = -1;

// What a face needs of its grid.
template <class T>
struct MustaFace {
    T lam;          // dt/dx of the local predictor-corrector
    double gm1;     // ideal gas: gamma - 1
    int limiter, mk;
};

// Limited MUSCL slope from the one-sided differences a, b (zero where they
// differ in sign or one is NaN): minmod, MC, van Leer, superbee, or none.  Minmod, the
// default, is selects only: ten slopes a face were a quarter of its
// instructions as branches (MUSTA-FORCE step, FP64: 128^3 559 us, now 511; 192^3
// 1805, now 1653).
template <class T, int LIM>
__device__ __forceinline__ T limited_slope(int rt_lim, T a, T b) {
    const int lim = LIM == kAnyLimiter ? rt_lim : LIM;
    if (lim == RH_LIMITER_NONE) return (T)0;
    if constexpr (LIM == RH_LIMITER_MINMOD) {
        const T m = max(min(a, b), (T)0) + min(max(a, b), (T)0);   // one term is zero
        return __builtin_isunordered(a, b) ? (T)0 : m;
    }
    if (!((a > (T)0 && b > (T)0) || (a < (T)0 && b < (T)0))) return (T)0;
    const T aa = fabs(a), ab = fabs(b);
    T m;
    if (lim == RH_LIMITER_MINMOD) m = min(aa, ab);
    else if (lim == RH_LIMITER_MC) m = min(min((T)2 * aa, (T)2 * ab), (T)0.5 * (aa + ab));
    else if (lim == RH_LIMITER_VANLEER) return (T)2 * a * b / (a + b);
    else m = max(min((T)2 * aa, ab), min(aa, (T)2 * ab));
    return a > (T)0 ? m : -m;
}

// Physical flux along DIR of a state (FP64 recovery for the fluid of EOS).
// DIR is the axis, or kAnyAxis to take it from rt_dir.
template <class T, int DIR, int EOS>
__device__ __forceinline__ void phys_flux(const T u[5], double gm1, T f[5], unsigned& cl, int rt_dir = 0) {
    const int dir = DIR == kAnyAxis ? rt_dir : DIR;
    double vd, p;
    if constexpr (EOS == EOS_CONFORMAL && DIR == kAnyAxis) {
        double kap, Mxs, Mys, Mzs;
        recover_kp3((double)u[0], (double)u[1], (double)u[2], (double)u[3], kap, Mxs, Mys, Mzs, p, cl);
        vd = kap * (dir == 0 ? Mxs : (dir == 1 ? Mys : Mzs));
    } else if constexpr (EOS == EOS_CONFORMAL) {
        recover_vp<DIR>((double)u[0], (double)u[1], (double)u[2], (double)u[3], vd, p, cl);
    } else {
        double kap, Mxs, Mys, Mzs, e;
        recover_ideal((double)u[0], (double)u[1], (double)u[2], (double)u[3], (double)u[4], gm1, kap,
                      Mxs, Mys, Mzs, p, e, cl);
        vd = kap * (dir == 0 ? Mxs : (dir == 1 ? Mys : Mzs));
    }
    const T v = (T)vd, P = (T)p;
    f[0] = dir == 0 ? u[1] : (dir == 1 ? u[2] : u[3]);
    f[1] = u[1] * v + (dir == 0 ? P : (T)0);
    f[2] = u[2] * v + (dir == 1 ? P : (T)0);
    f[3] = u[3] * v + (dir == 2 ? P : (T)0);
    f[4] = u[4] * v;
}

// MUSTA flux of the states uL, uR on both sides of a face.
template <class T, int DIR, int EOS, int MK>
__device__ __forceinline__ void musta_flux(T uL[5], T uR[5], const MustaFace<T>& Gr, T F[5], unsigned& cl,
                                           int rt_dir = 0) {
    const T lam = Gr.lam, hlam = (T)0.5 * Gr.lam, q4 = (T)1 / ((T)4 * Gr.lam);
    const int mk = MK == kAnyStages ? Gr.mk : MK;
    constexpr int kUnroll = MK == kAnyStages ? 1 : MK;
#pragma unroll kUnroll
    for (int st = 1; st <= mk; ++st) {
        T fL[5], fR[5], uM[5], fM[5];
        phys_flux<T, DIR, EOS>(uL, Gr.gm1, fL, cl, rt_dir);
        phys_flux<T, DIR, EOS>(uR, Gr.gm1, fR, cl, rt_dir);
#pragma unroll
        for (int q = 0; q < 5; ++q) uM[q] = (T)0.5 * (uL[q] + uR[q]) - hlam * (fR[q] - fL[q]);
        phys_flux<T, DIR, EOS>(uM, Gr.gm1, fM, cl, rt_dir);
#pragma unroll
        for (int q = 0; q < 5; ++q) F[q] = (T)0.25 * (fL[q] + (T)2 * fM[q] + fR[q]) - (uR[q] - uL[q]) * q4;
        if (st < mk) {
#pragma unroll
            for (int q = 0; q < 5; ++q) {
                uL[q] = uL[q] - lam * (F[q] - fL[q]);
                uR[q] = uR[q] - lam * (fR[q] - F[q]);
            }
        }
    }
}

// MUSCL + MUSTA flux of face i+1/2 from the cells i-1 .. i+2 (a, b, c, d).
template <class T, int DIR, int EOS, int LIM, int MK>
__device__ __forceinline__ void musta_face(const T a[5], const T b[5], const T c[5], const T d[5],
                                           const MustaFace<T>& Gr, T F[5], unsigned& cl, int rt_dir = 0) {
    T uL[5], uR[5];
#pragma unroll
    for (int q = 0; q < 5; ++q) {
        const T si = limited_slope<T, LIM>(Gr.limiter, b[q] - a[q], c[q] - b[q]);
        const T sj = limited_slope<T, LIM>(Gr.limiter, c[q] - b[q], d[q] - c[q]);
        uL[q] = b[q] + (T)0.5 * si;
        uR[q] = c[q] - (T)0.5 * sj;
    }
    musta_flux<T, DIR, EOS, MK>(uL, uR, Gr, F, cl, rt_dir);
}

}  // namespace rh
