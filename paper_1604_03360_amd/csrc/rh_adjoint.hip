// rh_adjoint.hip -- gfx950 kernels of the adjoint of L and of the SSP-RK3 step.
//
// One adjoint sweep per axis, from the primitive recovery of each cell and its
// derivatives (FP64 arithmetic, in a per-cell pack).  The x sweep stages
// contiguous cells in LDS, differentiates each face once and gathers the face
// partials per cell; it writes the output from the caller's linear combination
// plus its part.  On periodic rows of 32..256 cells it takes whole rows
// (adj_xrow) and also computes and stores the pack; otherwise it takes short tiles
// that recover for themselves (adj_small) or, in FP32 WENO5 on large grids, longer
// ones that read the pack (adj_x).  Along y and z small grids take adj_small as well
// (adjoint_small), large ones and short axes a rolling sweep that reads the pack
// (adj_roll); where a sweep reads it and no row kernel has, a launch of its own fills it
// (adj_pack).  adj_roll gives each lane a segment [k0, k1) of one grid line; the lane rolls
// along it over every face whose stencil reaches an owned position (the segment plus R
// faces on each side), keeping a register window of 2R cells of split fluxes
// and of split-flux adjoints; for each face it adds the face weight
// g = (w_{i+1} - w_i)/h times the WENO gradients to the window, and a position
// leaving the window is complete and, if the lane owns it, is mapped through
// the flux Jacobian and added to the adjoint field.  Every cell (and every
// ghost position that copies it under outflow boundaries) is owned by exactly
// one lane per sweep, so the read-modify-write needs no atomics.
#include "rh_internal.hpp"
#include "rh_adjoint.hpp"
#include "../../include/rh.h"

namespace rh {

namespace {

// A field's base pointer made opaque once per lane-line: loads through it then
// keep the scalar-base + 32-bit-offset form instead of being re-associated by
// the compiler into per-lane 64-bit address arithmetic (one 64-bit add per
// access).
template <class T>
using gptr = __attribute__((address_space(1))) T*;

template <class T>
__device__ __forceinline__ gptr<T> opaque_base(T* p) {
    gptr<T> g = (gptr<T>)p;
    asm("" : "+s"(g));
    return g;
}
template <class T>
__device__ __forceinline__ T ld_off(gptr<const T> base, uint32_t off) {
    return *(gptr<const T>)((gptr<const char>)base + off);
}
template <class T>
__device__ __forceinline__ void st_off(gptr<T> base, uint32_t off, T v) {
    *(gptr<T>)((gptr<char>)base + off) = v;
}

template <class T, int DIR>
struct Column {
    gptr<const T> u[5];    // field base pointers (uniform)
    gptr<const T> w[5];
    gptr<const T> pk[6];
    gptr<T> ub[5];
    // lane -> line: plane axes are (y, z) for DIR 0, (x, z) for DIR 1, (x, y) for DIR 2;
    // byte offsets of the line's first cell and between consecutive cells
    uint32_t cb;
    uint32_t sb;
    int ia, ib;   // the two transverse indices
};

template <class T, int DIR>
__device__ __forceinline__ bool column_of(const AdjArgs<T>& A, unsigned p, Column<T, DIR>& C) {
    const int nx = A.n[0], ny = A.n[1], nz = A.n[2];
#pragma unroll
    for (int f = 0; f < 5; ++f) {
        C.u[f] = opaque_base(A.u + f * A.fstride);
        C.w[f] = opaque_base(A.w + f * A.fstride);
        C.ub[f] = opaque_base(A.ub + f * A.fstride);
    }
#pragma unroll
    for (int f = 0; f < 6; ++f) C.pk[f] = opaque_base(A.pk + f * A.fstride);
    if (DIR == 0) {
        const int y = (int)(p % (unsigned)ny), z = (int)(p / (unsigned)ny);
        if (z >= nz) return false;
        C.ia = y;
        C.ib = z;
        C.cb = (uint32_t)sizeof(T) * ((uint32_t)nx * ((uint32_t)y + (uint32_t)ny * (uint32_t)z));
        C.sb = (uint32_t)sizeof(T);
    } else if (DIR == 1) {
        const int x = (int)(p % (unsigned)nx), z = (int)(p / (unsigned)nx);
        if (z >= nz) return false;
        C.ia = x;
        C.ib = z;
        C.cb = (uint32_t)sizeof(T) * ((uint32_t)x + (uint32_t)nx * (uint32_t)ny * (uint32_t)z);
        C.sb = (uint32_t)sizeof(T) * (uint32_t)nx;
    } else {
        const int x = (int)(p % (unsigned)nx), y = (int)(p / (unsigned)nx);
        if (y >= ny) return false;
        C.ia = x;
        C.ib = y;
        C.cb = (uint32_t)sizeof(T) * ((uint32_t)x + (uint32_t)nx * (uint32_t)y);
        C.sb = (uint32_t)sizeof(T) * ((uint32_t)nx * (uint32_t)ny);
    }
    return true;
}

template <class T, int DIR>
__device__ __forceinline__ void cell_xyz(const Column<T, DIR>& C, int m, int c[3]) {
    if (DIR == 0) { c[0] = m; c[1] = C.ia; c[2] = C.ib; }
    else if (DIR == 1) { c[0] = C.ia; c[1] = m; c[2] = C.ib; }
    else { c[0] = C.ia; c[1] = C.ib; c[2] = m; }
}

// state at line position m (ghosts by the boundary condition of the axis)
template <class T, int DIR>
__device__ __forceinline__ void adj_load(const AdjArgs<T>& A, const Column<T, DIR>& C, int m, T u[5]) {
    const int nd = A.n[DIR];
    int mm = m;
    if (m < 0 || m >= nd) {
        if (A.bc == RH_BC_PERIODIC) {
            mm = m % nd;
            if (mm < 0) mm += nd;
        } else if (A.bc == RH_BC_OUTFLOW) {
            mm = m < 0 ? 0 : nd - 1;
        } else {
            int c[3];
            cell_xyz(C, m, c);
            double uh[5];
            hubble_conserved(A.hb, A.hb.c0[0] + c[0] * A.hb.h[0], A.hb.c0[1] + c[1] * A.hb.h[1],
                             A.hb.c0[2] + c[2] * A.hb.h[2], uh);
#pragma unroll
            for (int f = 0; f < 5; ++f) u[f] = (T)uh[f];
            return;
        }
    }
    const uint32_t off = C.cb + (uint32_t)mm * C.sb;
#pragma unroll
    for (int f = 0; f < 5; ++f) u[f] = ld_off(C.u[f], off);
}

// State at line position m with its velocity along the sweep axis and pressure,
// taken from the recovery pack (interior, periodic and outflow positions) or,
// for analytic ghosts, evaluated and recovered here in FP64.  HUB = false
// compiles the analytic branch out (its FP64 registers would otherwise count
// against the whole rolling window).
template <class T, int DIR, bool HUB>
__device__ __forceinline__ void adj_state(const AdjArgs<T>& A, const Column<T, DIR>& C, int m, T u[5], T& v,
                                          T& P) {
    const int nd = A.n[DIR];
    int mm = m;
    if (m < 0 || m >= nd) {
        if (A.bc == RH_BC_PERIODIC) {
            mm = m % nd;
            if (mm < 0) mm += nd;
        } else if (!HUB || A.bc == RH_BC_OUTFLOW) {
            mm = m < 0 ? 0 : nd - 1;
        } else {
            adj_load<T, DIR>(A, C, m, u);
            double vd, pd;
            unsigned dummy = 0;
            recover_vp<DIR>((double)u[0], (double)u[1], (double)u[2], (double)u[3], vd, pd, dummy);
            v = (T)vd;
            P = (T)pd;
            return;
        }
    }
    const uint32_t off = C.cb + (uint32_t)mm * C.sb;
#pragma unroll
    for (int f = 0; f < 5; ++f) u[f] = ld_off(C.u[f], off);
    v = ld_off(C.pk[0], off) * u[1 + DIR];
    P = ld_off(C.pk[1], off);
}

// weights at line position m: zero outside the grid unless periodic
template <class T, int DIR>
__device__ __forceinline__ void adj_weight(const AdjArgs<T>& A, const Column<T, DIR>& C, int m, T w[5]) {
    const int nd = A.n[DIR];
    int mm = m;
    if (m < 0 || m >= nd) {
        if (A.bc != RH_BC_PERIODIC) {
#pragma unroll
            for (int f = 0; f < 5; ++f) w[f] = (T)0;
            return;
        }
        mm = m % nd;
        if (mm < 0) mm += nd;
    }
    const uint32_t off = C.cb + (uint32_t)mm * C.sb;
#pragma unroll
    for (int f = 0; f < 5; ++f) w[f] = ld_off(C.w[f], off);
}

}  // namespace

// The WENO reconstruction is component-wise, so the face gradients of each
// conserved component need only that component's window; the components are
// therefore processed in groups, one pass per group over the lane's segment,
// each pass carrying only its group's window (which keeps the register file
// small enough for several waves per SIMD).  A pass adds its group's part of
// (d f+/du)^T a+ + (d f-/du)^T a- to every field of the owned cells.
//
// Components per pass: FP32 WENO5 3 (passes {0,1,2}, {3,4}); otherwise 2.
template <class T, int ORDER>
struct AdjGroup {
    static constexpr int value = (sizeof(T) == 4 && ORDER == 5) ? 3 : 2;
};

template <class T, int ORDER, int DIR, int CLO, int CHI, bool HUB>
__device__ __forceinline__ void adj_pass(const AdjArgs<T>& A, const Column<T, DIR>& C, int k0, int k1) {
    constexpr int R = (ORDER + 1) / 2, W = 2 * R, NC = CHI - CLO;
    // WENO5 gradient in the first differences (fewer instructions, more live
    // values) except where the analytic-ghost branch leaves too few registers
    // for it at three FP32 waves per SIMD
    constexpr bool EFORM = !(sizeof(T) == 4 && HUB);
    const int nd = A.n[DIR];
    const bool periodic = A.bc == RH_BC_PERIODIC;
    int i_lo = k0 - R, i_hi = k1 + R - 2;
    if (!periodic) {
        i_lo = max(i_lo, -1);
        i_hi = min(i_hi, nd - 1);
    }
    // owned positions [own_lo, own_hi): outflow edges also own the ghost positions
    const int own_lo = (!periodic && k0 == 0 && A.bc == RH_BC_OUTFLOW) ? -(1 << 30) : k0;
    const int own_hi = (!periodic && k1 == nd && A.bc == RH_BC_OUTFLOW) ? (1 << 30) : k1;
    const T eps = A.eps;
    const T half = (T)0.5;
    // adjoint fields this group changes: its own components, and with any
    // momentum or charge component the energy and the momenta (through the
    // velocity and pressure); the others are neither loaded nor stored
    auto touched = [](int f) {
        return (f >= CLO && f < CHI) || (CHI > 1 && f < 4) || (CLO == 0 && f == 1 + DIR);
    };

    // doubled split fluxes F +- u of the group's components from a cell state:
    // the reconstruction is homogeneous of degree one in (f, sqrt(eps)), so its
    // gradient at (2 f, 4 eps) equals the gradient at (f, eps), bit for bit
    // (all scalings are powers of two); the 1/2 of the split stays in finish
    auto group_flux = [&](const T u[5], T v, T P, T fp[NC], T fm[NC]) {
#pragma unroll
        for (int q = 0; q < NC; ++q) {
            const int c = CLO + q;
            T f;
            if (c == 0) f = u[1 + DIR];
            else if (c == 4) f = u[4] * v;
            else f = u[c] * v + (c == 1 + DIR ? P : (T)0);
            fp[q] = f + u[c];
            fm[q] = f - u[c];
        }
    };
    // Owned position pos -> the cell whose adjoint it updates (outflow ghost
    // positions fold onto the edge cell; analytic ghosts are constants).
    auto target = [&](int pos, int& tgt) -> bool {
        if (pos < own_lo || pos >= own_hi) return false;
        tgt = pos;
        if (pos < 0 || pos >= nd) {
            if (A.bc != RH_BC_OUTFLOW) return false;
            tgt = pos < 0 ? 0 : nd - 1;
        }
        return true;
    };
    // state and running adjoint of the cell updated next; consecutive updates
    // of one cell (outflow edges) continue from registers
    int last_tgt = -1;
    T ubo[5], uf[5], pkf[5];
    auto fetch_cell = [&](int tgt) {
        const uint32_t off = C.cb + (uint32_t)tgt * C.sb;
#pragma unroll
        for (int f = 0; f < 5; ++f) uf[f] = ld_off(C.u[f], off);
        if constexpr (CHI > 1) {
            pkf[0] = ld_off(C.pk[0], off);
#pragma unroll
            for (int q = 1; q < 5; ++q) pkf[q] = ld_off(C.pk[q + 1], off);
        }
        if (tgt == last_tgt) return;
#pragma unroll
        for (int f = 0; f < 5; ++f)
            if (touched(f)) ubo[f] = ld_off(C.ub[f], off);
    };
    // ub += scale * sum over the group of (d f+_c/du)^T a+_c + (d f-_c/du)^T a-_c
    auto finish = [&](int tgt, const T apj[NC], const T amj[NC]) {
        // pkf = (kappa, dkappa/dE, dkappa/dM2, dP/dE, dP/dM2); v_d = kappa M_d
        T lam[5] = {(T)0, (T)0, (T)0, (T)0, (T)0}, g[5] = {(T)0, (T)0, (T)0, (T)0, (T)0};
#pragma unroll
        for (int q = 0; q < NC; ++q) {
            lam[CLO + q] = half * (apj[q] + amj[q]);
            g[CLO + q] = half * (apj[q] - amj[q]);
        }
        g[1 + DIR] += lam[0];
        if constexpr (CHI > 1) {
            const T Md = uf[1 + DIR], vd = pkf[0] * Md;
            T S = (T)0;
#pragma unroll
            for (int c = (CLO > 1 ? CLO : 1); c < CHI; ++c) {
                S += lam[c] * uf[c];
                g[c] += lam[c] * vd;
            }
            const T lp = lam[1 + DIR];
            // dv_d/dE = M_d kappa_E, dv_d/dM_m = kappa delta_dm + 2 M_d M_m kappa_M2,
            // dP/dE = P_E, dP/dM_m = 2 M_m P_M2
            g[0] += S * (Md * pkf[1]) + lp * pkf[3];
            const T sk = (T)2 * S * Md * pkf[2], sp = (T)2 * lp * pkf[4];
#pragma unroll
            for (int m = 0; m < 3; ++m) g[1 + m] += (sk + sp) * uf[1 + m];
            g[1 + DIR] += S * pkf[0];
        }
        const uint32_t off = C.cb + (uint32_t)tgt * C.sb;
#pragma unroll
        for (int f = 0; f < 5; ++f) {
            if (!touched(f)) continue;
            ubo[f] = ubo[f] + A.scale * g[f];
            st_off(C.ub[f], off, ubo[f]);
        }
        last_tgt = tgt;
    };
    T wp[NC][W], wm[NC][W], ap[NC][W], am[NC][W];
#pragma unroll
    for (int j = 0; j < W; ++j) {
        T u[5], v, P, fp[NC], fm[NC];
        adj_state<T, DIR, HUB>(A, C, i_lo - R + 1 + j, u, v, P);
        group_flux(u, v, P, fp, fm);
#pragma unroll
        for (int q = 0; q < NC; ++q) {
            wp[q][j] = fp[q];
            wm[q][j] = fm[q];
            ap[q][j] = (T)0;
            am[q][j] = (T)0;
        }
    }
    // loads run one face ahead: the weights of the next face's right cell and
    // the state of the next cell to enter the window are in flight while this
    // face is differentiated (positions past the segment stay in bounds)
    T wl[NC], wn[NC], un[5], vn, Pn;
    {
        T w5[5];
        adj_weight<T, DIR>(A, C, i_lo, w5);
#pragma unroll
        for (int q = 0; q < NC; ++q) wl[q] = w5[CLO + q];
        adj_weight<T, DIR>(A, C, i_lo + 1, w5);
#pragma unroll
        for (int q = 0; q < NC; ++q) wn[q] = w5[CLO + q];
    }
    adj_state<T, DIR, HUB>(A, C, i_lo + R + 1, un, vn, Pn);
    // two faces per trip: the second face's window is the first one's renamed,
    // so the register moves of the shift are paid once per two faces
#pragma unroll 2
    for (int i = i_lo; i <= i_hi; ++i) {
        T wr[NC], unew[5];
#pragma unroll
        for (int q = 0; q < NC; ++q) wr[q] = wn[q];
#pragma unroll
        for (int f = 0; f < 5; ++f) unew[f] = un[f];
        const T vnew = vn, Pnew = Pn;
        {
            T w5[5];
            adj_weight<T, DIR>(A, C, i + 2, w5);
#pragma unroll
            for (int q = 0; q < NC; ++q) wn[q] = w5[CLO + q];
        }
        adj_state<T, DIR, HUB>(A, C, i + R + 2, un, vn, Pn);
        int tgt = 0;
        const bool own = target(i - R + 1, tgt);
        if (own) fetch_cell(tgt);
#pragma unroll
        for (int q = 0; q < NC; ++q) {
            const T g = (wr[q] - wl[q]) * A.inv_h;
            wl[q] = wr[q];
            if constexpr (ORDER == 5) {
                if constexpr (EFORM) {
                    weno5_grad_acc_e<T>(wp[q][0], wp[q][1], wp[q][2], wp[q][3], wp[q][4], (T)16 * eps, g,
                                        ap[q][0], ap[q][1], ap[q][2], ap[q][3], ap[q][4]);
                    weno5_grad_acc_e<T>(wm[q][5], wm[q][4], wm[q][3], wm[q][2], wm[q][1], (T)16 * eps, g,
                                        am[q][5], am[q][4], am[q][3], am[q][2], am[q][1]);
                } else {
                    weno5_grad_acc<T>(wp[q][0], wp[q][1], wp[q][2], wp[q][3], wp[q][4], (T)16 * eps, g,
                                      ap[q][0], ap[q][1], ap[q][2], ap[q][3], ap[q][4]);
                    weno5_grad_acc<T>(wm[q][5], wm[q][4], wm[q][3], wm[q][2], wm[q][1], (T)16 * eps, g,
                                      am[q][5], am[q][4], am[q][3], am[q][2], am[q][1]);
                }
            } else {
                T sv[7], o[7];
#pragma unroll
                for (int j = 0; j < 7; ++j) { sv[j] = wp[q][j]; o[j] = (T)0; }
                weno7_grad_acc<T>(sv, (T)4 * eps, g, o);
#pragma unroll
                for (int j = 0; j < 7; ++j) ap[q][j] += o[j];
#pragma unroll
                for (int j = 0; j < 7; ++j) { sv[j] = wm[q][7 - j]; o[j] = (T)0; }
                weno7_grad_acc<T>(sv, (T)4 * eps, g, o);
#pragma unroll
                for (int j = 0; j < 7; ++j) am[q][7 - j] += o[j];
            }
        }
        if (own) {
            T a0p[NC], a0m[NC];
#pragma unroll
            for (int q = 0; q < NC; ++q) {
                a0p[q] = ap[q][0];
                a0m[q] = am[q][0];
            }
            finish(tgt, a0p, a0m);
        }
        if (i < i_hi) {
            T fp[NC], fm[NC];
            group_flux(unew, vnew, Pnew, fp, fm);
#pragma unroll
            for (int q = 0; q < NC; ++q) {
#pragma unroll
                for (int j = 0; j < W - 1; ++j) {
                    wp[q][j] = wp[q][j + 1];
                    wm[q][j] = wm[q][j + 1];
                    ap[q][j] = ap[q][j + 1];
                    am[q][j] = am[q][j + 1];
                }
                wp[q][W - 1] = fp[q];
                wm[q][W - 1] = fm[q];
                ap[q][W - 1] = (T)0;
                am[q][W - 1] = (T)0;
            }
        }
    }
    // positions still in the window after the last face
#pragma unroll
    for (int j = 1; j < W; ++j) {
        int tgt = 0;
        if (!target(i_hi - R + 1 + j, tgt)) continue;
        fetch_cell(tgt);
        T ajp[NC], ajm[NC];
#pragma unroll
        for (int q = 0; q < NC; ++q) {
            ajp[q] = ap[q][j];
            ajm[q] = am[q][j];
        }
        finish(tgt, ajp, ajm);
    }
}

template <class T, int ORDER, int DIR, int CLO, bool HUB>
__device__ __forceinline__ void adj_passes(const AdjArgs<T>& A, const Column<T, DIR>& C, int k0, int k1) {
    if constexpr (CLO < 5) {
        constexpr int GS = AdjGroup<T, ORDER>::value;
        constexpr int CHI = CLO + GS < 5 ? CLO + GS : 5;
        adj_pass<T, ORDER, DIR, CLO, CHI, HUB>(A, C, k0, k1);
        adj_passes<T, ORDER, DIR, CHI, HUB>(A, C, k0, k1);
    }
}

// Three waves per SIMD for FP32 (the register window fits in 168 VGPRs); FP64
// takes what the window needs.
template <class T>
struct AdjMinBlocks {
    static constexpr int value = sizeof(T) == 4 ? 3 : 1;
};

template <class T, int ORDER, int DIR, bool HUB>
__global__ void __launch_bounds__(256, (AdjMinBlocks<T>::value)) adj_roll(AdjArgs<T> A) {
    Column<T, DIR> C;
    if (!column_of<T, DIR>(A, blockIdx.x * 256u + threadIdx.x, C)) return;
    const int k0 = blockIdx.y * A.seg;
    const int k1 = min(k0 + A.seg, A.n[DIR]);
    adj_passes<T, ORDER, DIR, 0, HUB>(A, C, k0, k1);
}

template <class T>
__global__ void adj_pack(const T* __restrict__ u, T* __restrict__ pk, long long n) {
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x) {
        const RecoveryPack o = recovery_pack((double)u[i], (double)u[n + i], (double)u[2 * n + i],
                                             (double)u[3 * n + i]);
        pk[i] = (T)o.kap;
        pk[n + i] = (T)o.p;
        pk[2 * n + i] = (T)o.kap_E;
        pk[3 * n + i] = (T)o.kap_M2;
        pk[4 * n + i] = (T)o.p_E;
        pk[5 * n + i] = (T)o.p_M2;
    }
}

// ---------------------------------------------------------------------------
// x axis of large grids, FP32 WENO5: x is contiguous, so a block takes a tile of TX cells x TY rows plus
// ghosts in LDS, as the forward x sweep does.  Per component, each lane
// differentiates one face (the tile's faces are spread over the lanes) and
// writes the face's stencil partials to LDS; after a barrier each lane sums
// the partials of the faces that reach its cell in a fixed order.  With all
// five split-flux adjoints of its cell in registers the lane applies the flux
// Jacobian once and writes out = (linear combination of init terms) + scale g.
// Outflow ghost positions fold onto the edge cells (same state, so their
// split-flux adjoints add before the Jacobian); analytic ghosts are constants.
// ---------------------------------------------------------------------------
template <class T>
__device__ __forceinline__ void x_state(const AdjArgs<T>& A, int gx, int row, T u[5], T& v, T& P) {
    const int nx = A.n[0];
    int mx = gx;
    if (gx < 0 || gx >= nx) {
        if (A.bc == RH_BC_PERIODIC) {
            mx = gx % nx;
            if (mx < 0) mx += nx;
        } else if (A.bc == RH_BC_OUTFLOW) {
            mx = gx < 0 ? 0 : nx - 1;
        } else {
            const int y = row % A.n[1], z = row / A.n[1];
            double uh[5];
            hubble_conserved(A.hb, A.hb.c0[0] + gx * A.hb.h[0], A.hb.c0[1] + y * A.hb.h[1],
                             A.hb.c0[2] + z * A.hb.h[2], uh);
#pragma unroll
            for (int f = 0; f < 5; ++f) u[f] = (T)uh[f];
            double vd, pd;
            unsigned dummy = 0;
            recover_vp<0>(uh[0], uh[1], uh[2], uh[3], vd, pd, dummy);
            v = (T)vd;
            P = (T)pd;
            return;
        }
    }
    const long long id = mx + (long long)nx * row;
#pragma unroll
    for (int f = 0; f < 5; ++f) u[f] = A.u[f * A.fstride + id];
    v = A.pk[id] * u[1];
    P = A.pk[A.fstride + id];
}

template <class T, int TX, int TY>
__global__ void __launch_bounds__(256) adj_x(AdjArgs<T> A, Lin3<T> init) {
    constexpr int R = 3, K = 2 * R - 1;
    constexpr int CPL = TX * TY / 256;   // cells per lane
    constexpr int NF = TX + 2 * R - 1;   // faces x0-R .. x0+TX+R-2 (face i: between cells i and i+1)
    constexpr int NC = TX + 4 * R - 2;   // cells x0-2R+1 .. x0+TX+2R-2
    constexpr int NW = TX + 2 * R;       // weights x0-R .. x0+TX+R-1
    static_assert(TX * TY % 256 == 0, "whole cells per lane");
    __shared__ T sfp[5][TY][NC];
    __shared__ T sfm[5][TY][NC];
    __shared__ T sw[5][TY][NW];
    __shared__ T sp[TY][NF][K];          // plus partials of face fl for cells fl .. fl+K-1 (local)
    __shared__ T sm[TY][NF][K];          // minus partials of face fl for cells fl+1 .. fl+K
    const int nx = A.n[0];
    const int nrows = A.n[1] * A.n[2];
    const int ntx = (nx + TX - 1) / TX;
    const int bx = blockIdx.x % ntx, by = blockIdx.x / ntx;
    const int x0 = bx * TX, r0 = by * TY;
    const int tid = threadIdx.x;
    const bool periodic = A.bc == RH_BC_PERIODIC;
    const T half = (T)0.5;

    for (int idx = tid; idx < TY * NC; idx += 256) {
        const int ly = idx / NC, lx = idx - ly * NC;
        const int row = r0 + ly;
        T fp[5] = {(T)0, (T)0, (T)0, (T)0, (T)0}, fm[5] = {(T)0, (T)0, (T)0, (T)0, (T)0};
        if (row < nrows) {
            T u[5], v, P;
            x_state<T>(A, x0 - 2 * R + 1 + lx, row, u, v, P);
            T f[5];
            f[0] = u[1];
            f[1] = u[1] * v + P;
            f[2] = u[2] * v;
            f[3] = u[3] * v;
            f[4] = u[4] * v;
#pragma unroll
            for (int c = 0; c < 5; ++c) {
                fp[c] = f[c] + u[c];   // doubled split fluxes (eps scaled by 4 below)
                fm[c] = f[c] - u[c];
            }
        }
#pragma unroll
        for (int c = 0; c < 5; ++c) {
            sfp[c][ly][lx] = fp[c];
            sfm[c][ly][lx] = fm[c];
        }
    }
    for (int idx = tid; idx < TY * NW; idx += 256) {
        const int ly = idx / NW, lx = idx - ly * NW;
        const int row = r0 + ly;
        int gx = x0 - R + lx;
        bool inside = row < nrows;
        if (inside && (gx < 0 || gx >= nx)) {
            if (periodic) {
                gx %= nx;
                if (gx < 0) gx += nx;
            } else {
                inside = false;   // weights vanish outside a non-periodic grid
            }
        }
        const long long id = gx + (long long)nx * row;
#pragma unroll
        for (int c = 0; c < 5; ++c) sw[c][ly][lx] = inside ? A.w[c * A.fstride + id] : (T)0;
    }
    __syncthreads();

    T ap[CPL][5], am[CPL][5];
#pragma unroll 1
    for (int c = 0; c < 5; ++c) {
        for (int f = tid; f < TY * NF; f += 256) {
            const int fy = f / NF, fl = f - fy * NF;
            const int i = x0 - R + fl;
            T op[K], om[K];
#pragma unroll
            for (int k = 0; k < K; ++k) op[k] = om[k] = (T)0;
            if ((periodic || (i >= -1 && i <= nx - 1)) && r0 + fy < nrows) {
                const T g = (sw[c][fy][fl + 1] - sw[c][fy][fl]) * A.inv_h;
                weno5_grad_acc_e<T>(sfp[c][fy][fl], sfp[c][fy][fl + 1], sfp[c][fy][fl + 2], sfp[c][fy][fl + 3],
                                    sfp[c][fy][fl + 4], (T)16 * A.eps, g, op[0], op[1], op[2], op[3], op[4]);
                weno5_grad_acc_e<T>(sfm[c][fy][fl + 5], sfm[c][fy][fl + 4], sfm[c][fy][fl + 3], sfm[c][fy][fl + 2],
                                    sfm[c][fy][fl + 1], (T)16 * A.eps, g, om[4], om[3], om[2], om[1], om[0]);
            }
#pragma unroll
            for (int k = 0; k < K; ++k) {
                sp[fy][fl][k] = op[k];
                sm[fy][fl][k] = om[k];
            }
        }
        __syncthreads();
        // partials reaching staged cell q: plus from faces q-k, minus from faces q-1-k
#pragma unroll
        for (int j = 0; j < CPL; ++j) {
            const int cell = tid + 256 * j, lx = cell % TX, ly = cell / TX;
            const int q = lx + 2 * R - 1;   // every face reaching an owned cell is in the tile
            T a_p = (T)0, a_m = (T)0;
#pragma unroll
            for (int k = 0; k < K; ++k) {
                a_p += sp[ly][q - k][k];
                a_m += sm[ly][q - 1 - k][k];
            }
            const int gx = x0 + lx;
            if (A.bc == RH_BC_OUTFLOW && (gx == 0 || gx == nx - 1) && r0 + ly < nrows) {
                // ghost positions beyond the edge fold onto the edge cell
                for (int e = 1; e < 2 * R; ++e) {
                    const int qe = gx == 0 ? q - e : q + e;
                    for (int k = 0; k < K; ++k) {
                        const int fp_ = qe - k, fm_ = qe - 1 - k;
                        if (fp_ >= 0 && fp_ < NF) a_p += sp[ly][fp_][k];
                        if (fm_ >= 0 && fm_ < NF) a_m += sm[ly][fm_][k];
                    }
                }
            }
            ap[j][c] = a_p;
            am[j][c] = a_m;
        }
        __syncthreads();
    }
#pragma unroll
    for (int j = 0; j < CPL; ++j) {
        const int cell = tid + 256 * j, lx = cell % TX, ly = cell / TX;
        const int gx = x0 + lx, row = r0 + ly;
        if (gx >= nx || row >= nrows) continue;
        const long long id = gx + (long long)nx * row;
        T uf[5];
#pragma unroll
        for (int f = 0; f < 5; ++f) uf[f] = A.u[f * A.fstride + id];
        const T kap = A.pk[id], kE = A.pk[2 * A.fstride + id], kM2 = A.pk[3 * A.fstride + id];
        const T pE = A.pk[4 * A.fstride + id], pM2 = A.pk[5 * A.fstride + id];
        T lam[5], g[5];
#pragma unroll
        for (int c = 0; c < 5; ++c) {
            lam[c] = half * (ap[j][c] + am[j][c]);
            g[c] = half * (ap[j][c] - am[j][c]);
        }
        // F = (Mx, Mx v + p, My v, Mz v, N v) with v = kappa Mx
        const T Mx = uf[1], vd = kap * Mx;
        g[1] += lam[0];
        T S = (T)0;
#pragma unroll
        for (int c = 1; c < 5; ++c) {
            S += lam[c] * uf[c];
            g[c] += lam[c] * vd;
        }
        const T lp = lam[1];
        g[0] += S * (Mx * kE) + lp * pE;
        const T sk = (T)2 * S * Mx * kM2, spp = (T)2 * lp * pM2;
#pragma unroll
        for (int m = 0; m < 3; ++m) g[1 + m] += (sk + spp) * uf[1 + m];
        g[1] += S * kap;
#pragma unroll
        for (int f = 0; f < 5; ++f) {
            const long long o = f * A.fstride + id;
            T acc = (T)0;
            if (init.X1) acc += init.a1 * init.X1[o];
            if (init.X2) acc += init.a2 * init.X2[o];
            if (init.X3) acc += init.a3 * init.X3[o];
            A.ub[o] = acc + A.scale * g[f];
        }
    }
}

// ---------------------------------------------------------------------------
// Small grids along any axis, and x wherever whole rows do not fit: what bounds a
// tile is the length of its chain of dependent work and its barriers (an FP64
// recovery, two WENO gradients per lane), not its throughput.  A block takes 16 positions
// along the axis x 4 lines and differentiates the faces of all five components
// at once, one (component, face) per lane; the partials go to LDS, are gathered
// one (component, cell) per lane, and the lane that owns the cell applies the
// flux Jacobian: three barriers in all, five with HALF (a component at a time as in adj_x:
// eleven).
// Each block recovers the primitives of the cells it stages (FP64, as adj_pack):
// reading them from a pack measured no faster (130x128x128 FP64 868 us against
// 877) and costs small grids a launch.  J^T w at 33x20x17 FP64 WENO7: 168 us with
// rolling lanes, 58 with tiles that take a component at a time, 21 with these.  x
// writes out = (linear combination of init terms) +
// scale g; y and z add scale g to out.  The order of every sum is that of adj_x.
//
// Lines are numbered so that consecutive ones are neighbours in memory along y
// and z; along x a line is a row.
// ---------------------------------------------------------------------------
// Position m of line `line` of the axis DIR.
template <int DIR>
__device__ __forceinline__ long long line_cell(const int n[3], int line, int m) {
    if constexpr (DIR == 0) return m + (long long)n[0] * line;
    else if constexpr (DIR == 1) return line % n[0] + (long long)n[0] * (m + (long long)n[1] * (line / n[0]));
    else return line + (long long)n[0] * n[1] * m;
}

// State, velocity along the axis and pressure at position m of a line (ghost
// cells by the boundary condition of the axis), recovered here.
template <class T, int DIR>
__device__ __forceinline__ void line_state(const AdjArgs<T>& A, int m, int line, T u[5], T& v, T& P) {
    const int nd = A.n[DIR];
    if (m < 0 || m >= nd) {
        if (A.bc == RH_BC_PERIODIC) {
            m %= nd;
            if (m < 0) m += nd;
        } else if (A.bc == RH_BC_OUTFLOW) {
            m = m < 0 ? 0 : nd - 1;
        } else {
            int c[3];
            if (DIR == 0) { c[0] = m; c[1] = line % A.n[1]; c[2] = line / A.n[1]; }
            else if (DIR == 1) { c[0] = line % A.n[0]; c[1] = m; c[2] = line / A.n[0]; }
            else { c[0] = line % A.n[0]; c[1] = line / A.n[0]; c[2] = m; }
            double uh[5];
            hubble_conserved(A.hb, A.hb.c0[0] + c[0] * A.hb.h[0], A.hb.c0[1] + c[1] * A.hb.h[1],
                             A.hb.c0[2] + c[2] * A.hb.h[2], uh);
#pragma unroll
            for (int f = 0; f < 5; ++f) u[f] = (T)uh[f];
            double vd, pd;
            unsigned dummy = 0;
            recover_vp<DIR>(uh[0], uh[1], uh[2], uh[3], vd, pd, dummy);
            v = (T)vd;
            P = (T)pd;
            return;
        }
    }
    const long long id = line_cell<DIR>(A.n, line, m);
#pragma unroll
    for (int f = 0; f < 5; ++f) u[f] = A.u[f * A.fstride + id];
    const RecoveryPack o = recovery_pack((double)u[0], (double)u[1], (double)u[2], (double)u[3]);
    v = (T)o.kap * u[1 + DIR];
    P = (T)o.p;
}

constexpr int kSmallTX = 16, kSmallTY = 4, kSmallLanes = 512;

// Three blocks a CU in FP64 (six waves per SIMD): what the owners hold from the
// recovery to the end (WENO7: their state as well) is parked in LDS, which saves
// the registers, and WENO7 with HALF takes the plus and the minus partials
// through the same LDS one after the other, two barriers more.  J^T w at two
// blocks a CU and at three, FP64, us: 64^3 WENO5 101 -> 91, WENO7 124 -> 116; 72^3 181 -> 155
// and 223 -> 198; but WENO7 at 33x20x17, where every block has its place at
// once, 20.1 -> 21.0, so HALF begins where two blocks a CU are not enough.
template <class T, int ORDER, bool HALF>
struct AdjSmall {
    static constexpr bool three = sizeof(T) == 8 && (ORDER == 5 || HALF);
    static constexpr int waves = sizeof(T) == 4 ? 8 : three ? 6 : 4;
    static constexpr int park = !three ? 0 : ORDER == 5 ? 5 : 10;
};

template <class T, int ORDER, int DIR, bool HALF>
__global__ void __launch_bounds__(kSmallLanes, (AdjSmall<T, ORDER, HALF>::waves)) adj_small(AdjArgs<T> A, Lin3<T> init) {
    constexpr int R = (ORDER + 1) / 2, K = 2 * R - 1;
    constexpr int TX = kSmallTX, TY = kSmallTY, CELLS = TX * TY;
    constexpr int NF = TX + 2 * R - 1;   // faces x0-R .. x0+TX+R-2 (face i: between cells i and i+1)
    constexpr int NC = TX + 4 * R - 2;   // cells x0-2R+1 .. x0+TX+2R-2
    constexpr int NW = TX + 2 * R;       // weights x0-R .. x0+TX+R-1
    constexpr int W0 = 128, OWN0 = 256;  // first lanes staging weights and owning cells
    static_assert(NC * TY <= W0 && W0 + NW * TY <= OWN0 && OWN0 + CELLS <= kSmallLanes, "lanes for every role");
    static_assert(5 * NF * TY <= kSmallLanes, "one face and component per lane");
    __shared__ T sfp[5][NC * TY], sfm[5][NC * TY];   // split fluxes, [position][line]
    __shared__ T sw[5][NW * TY];                     // weights
    __shared__ T spm[HALF ? 1 : 2][5][K][NF * TY];   // partials of face f for cells f + k (minus: f + 1 + k)
    T (*sp)[K][NF * TY] = spm[0], (*sm)[K][NF * TY] = spm[HALF ? 0 : 1];
    __shared__ T sa[10][CELLS];                      // split-flux adjoints of the tile's cells
    constexpr int PARK = AdjSmall<T, ORDER, HALF>::park;
    __shared__ T sr[PARK ? PARK : 1][PARK ? CELLS : 1];   // what their owners keep until the end
    const int nd = A.n[DIR];
    const int nlines = DIR == 0 ? A.n[1] * A.n[2] : DIR == 1 ? A.n[0] * A.n[2] : A.n[0] * A.n[1];
    const int ntx = (nd + TX - 1) / TX;
    const unsigned blk = blockIdx.x + (unsigned)A.seg * blockIdx.y;
    const int bx = (int)(blk % ntx), by = (int)(blk / ntx);
    const int x0 = bx * TX, r0 = by * TY;
    const int tid = threadIdx.x;
    const bool periodic = A.bc == RH_BC_PERIODIC;
    const T half = (T)0.5;

    // this lane's own cell (lanes OWN0 ..): along x lanes run along the line
    const int own = tid - OWN0;
    const int ox = DIR == 0 ? own & (TX - 1) : own / TY, oy = DIR == 0 ? own / TX : own & (TY - 1);
    const bool owner = own >= 0 && own < CELLS && x0 + ox < nd && r0 + oy < nlines;
    T uf[5] = {(T)0, (T)0, (T)0, (T)0, (T)0}, base[5];
    T kap = (T)0, kE = (T)0, kM2 = (T)0, pE = (T)0, pM2 = (T)0;
    long long oid = 0;
    if (tid < NC * TY) {
        const int lx = DIR == 0 ? tid % NC : tid / TY, ly = DIR == 0 ? tid / NC : tid & (TY - 1);
        const int line = r0 + ly;
        T fp[5] = {(T)0, (T)0, (T)0, (T)0, (T)0}, fm[5] = {(T)0, (T)0, (T)0, (T)0, (T)0};
        if (line < nlines) {
            T u[5], v, P;
            line_state<T, DIR>(A, x0 - 2 * R + 1 + lx, line, u, v, P);
            split_flux_vp<T, DIR>(u, v, P, fp, fm);   // doubled split fluxes (eps scaled by 4 below)
        }
#pragma unroll
        for (int c = 0; c < 5; ++c) {
            sfp[c][lx * TY + ly] = fp[c];
            sfm[c][lx * TY + ly] = fm[c];
        }
    } else if (tid >= W0 && tid < W0 + NW * TY) {
        const int j = tid - W0;
        const int lx = DIR == 0 ? j % NW : j / TY, ly = DIR == 0 ? j / NW : j & (TY - 1);
        const int line = r0 + ly;
        int gx = x0 - R + lx;
        bool inside = line < nlines;
        if (inside && (gx < 0 || gx >= nd)) {
            if (periodic) {
                gx %= nd;
                if (gx < 0) gx += nd;
            } else {
                inside = false;   // weights vanish outside a non-periodic grid
            }
        }
        const long long id = inside ? line_cell<DIR>(A.n, line, gx) : 0;
#pragma unroll
        for (int c = 0; c < 5; ++c) sw[c][lx * TY + ly] = inside ? A.w[c * A.fstride + id] : (T)0;
    } else if (owner) {
        oid = line_cell<DIR>(A.n, r0 + oy, x0 + ox);
#pragma unroll
        for (int f = 0; f < 5; ++f) {
            const long long o = f * A.fstride + oid;
            uf[f] = A.u[o];
            base[f] = (T)0;
            if constexpr (DIR == 0) {
                if (init.X1) base[f] += init.a1 * init.X1[o];
                if (init.X2) base[f] += init.a2 * init.X2[o];
                if (init.X3) base[f] += init.a3 * init.X3[o];
            } else {
                base[f] = A.ub[o];
            }
        }
        const RecoveryPack o = recovery_pack((double)uf[0], (double)uf[1], (double)uf[2], (double)uf[3]);
        kap = (T)o.kap;
        kE = (T)o.kap_E;
        kM2 = (T)o.kap_M2;
        pE = (T)o.p_E;
        pM2 = (T)o.p_M2;
        if constexpr (PARK >= 5) {
            sr[0][own] = kap;
            sr[1][own] = kE;
            sr[2][own] = kM2;
            sr[3][own] = pE;
            sr[4][own] = pM2;
        }
        if constexpr (PARK >= 10) {
#pragma unroll
            for (int f = 0; f < 5; ++f) sr[5 + f][own] = uf[f];
        }
    }
    __syncthreads();

    const int fc = tid / (NF * TY), fj = tid - fc * (NF * TY);
    T op[K], om[K];
    if (tid < 5 * NF * TY) {
        const int c = fc, j = fj, i = x0 - R + j / TY;
#pragma unroll
        for (int k = 0; k < K; ++k) op[k] = om[k] = (T)0;
        if ((periodic || (i >= -1 && i <= nd - 1)) && r0 + (j & (TY - 1)) < nlines) {
            const T* cp = &sfp[c][j];
            const T* cm = &sfm[c][j];
            const T g = (sw[c][j + TY] - sw[c][j]) * A.inv_h;
            if constexpr (ORDER == 5) {
                weno5_grad_acc_e<T>(cp[0], cp[TY], cp[2 * TY], cp[3 * TY], cp[4 * TY], (T)16 * A.eps, g, op[0], op[1],
                                    op[2], op[3], op[4]);
                weno5_grad_acc_e<T>(cm[5 * TY], cm[4 * TY], cm[3 * TY], cm[2 * TY], cm[TY], (T)16 * A.eps, g, om[4],
                                    om[3], om[2], om[1], om[0]);
            } else {
                T sv[7], o[7];
#pragma unroll
                for (int q = 0; q < 7; ++q) sv[q] = cp[q * TY];
                weno7_grad_acc<T>(sv, (T)4 * A.eps, g, op);
#pragma unroll
                for (int q = 0; q < 7; ++q) {
                    sv[q] = cm[(7 - q) * TY];
                    o[q] = (T)0;
                }
                weno7_grad_acc<T>(sv, (T)4 * A.eps, g, o);
#pragma unroll
                for (int q = 0; q < 7; ++q) om[6 - q] = o[q];
            }
        }
#pragma unroll
        for (int k = 0; k < K; ++k) {
            sp[fc][k][fj] = op[k];
            if constexpr (!HALF) sm[fc][k][fj] = om[k];
        }
    }
    __syncthreads();
    // partials reaching staged cell q: plus from faces q-k, minus from faces q-1-k
    const int gc = tid / CELLS, cell = tid - gc * CELLS, gly = cell & (TY - 1);
    const int q = cell / TY + 2 * R - 1;   // every face reaching an owned cell is in the tile
    const int gx = x0 + cell / TY;
    const bool fold = A.bc == RH_BC_OUTFLOW && (gx == 0 || gx == nd - 1);
    auto gather = [&](const T (*part)[NF * TY], int f0) {
        T a = (T)0;
#pragma unroll
        for (int k = 0; k < K; ++k) a += part[k][(q - f0 - k) * TY + gly];
        if (fold) {
            // ghost positions beyond the edge fold onto the edge cell (same state, so
            // their split-flux adjoints add before the Jacobian)
            for (int e = 1; e < 2 * R; ++e) {
                const int qe = (gx == 0 ? q - e : q + e) - f0;
                for (int k = 0; k < K; ++k)
                    if (qe - k >= 0 && qe - k < NF) a += part[k][(qe - k) * TY + gly];
            }
        }
        return a;
    };
    if (tid < 5 * CELLS) sa[gc][cell] = gather(sp[gc], 0);
    if constexpr (HALF) {
        __syncthreads();
        if (tid < 5 * NF * TY) {
#pragma unroll
            for (int k = 0; k < K; ++k) sm[fc][k][fj] = om[k];
        }
        __syncthreads();
    }
    if (tid < 5 * CELLS) sa[5 + gc][cell] = gather(sm[gc], 1);
    __syncthreads();
    if (!owner) return;
    if constexpr (PARK >= 5) {
        kap = sr[0][own];
        kE = sr[1][own];
        kM2 = sr[2][own];
        pE = sr[3][own];
        pM2 = sr[4][own];
    }
    if constexpr (PARK >= 10) {
#pragma unroll
        for (int f = 0; f < 5; ++f) uf[f] = sr[5 + f][own];
    }
    T lam[5], g[5];
#pragma unroll
    for (int c = 0; c < 5; ++c) {
        const T ap = sa[c][ox * TY + oy], am = sa[5 + c][ox * TY + oy];
        lam[c] = half * (ap + am);
        g[c] = half * (ap - am);
    }
    // F = (M_d, M v + p e_d, N v) with v = kappa M_d
    const T Md = uf[1 + DIR], vd = kap * Md;
    g[1 + DIR] += lam[0];
    T S = (T)0;
#pragma unroll
    for (int c = 1; c < 5; ++c) {
        S += lam[c] * uf[c];
        g[c] += lam[c] * vd;
    }
    const T lp = lam[1 + DIR];
    g[0] += S * (Md * kE) + lp * pE;
    const T sk = (T)2 * S * Md * kM2, spp = (T)2 * lp * pM2;
#pragma unroll
    for (int m = 0; m < 3; ++m) g[1 + m] += (sk + spp) * uf[1 + m];
    g[1 + DIR] += S * kap;
#pragma unroll
    for (int f = 0; f < 5; ++f) A.ub[f * A.fstride + oid] = base[f] + A.scale * g[f];
}

// ---------------------------------------------------------------------------
// x axis of a periodic grid whose rows hold NX = 32 .. 256 cells: a block of
// (256 / NX) x NX lanes takes whole rows, one cell per lane.  The lane stages
// its own cell's split fluxes and weight (the periodic ghosts are extra LDS
// copies written by the cells they copy), differentiates the face to its right
// and gathers the partials of the faces that reach its cell.  No lane stages a
// ghost from HBM or differentiates a halo face, which the tiled kernel does for
// 2R - 1 faces per row (a fifth of its face rounds at 64 x 4).  The arithmetic
// and the order of every sum are those of adj_x, so both give the same bits.
// ---------------------------------------------------------------------------
// FP32 WENO5 rows: six waves per SIMD, the most that the LDS of 256-cell row
// blocks allows (62 registers instead of 82; 0.5% faster at 256^3).
template <class T, int ORDER>
struct AdjRowWaves {
    static constexpr int value = (sizeof(T) == 4 && ORDER == 5) ? 6 : 1;
};

template <class T, int ORDER, int NX>
__global__ void __launch_bounds__(256, (AdjRowWaves<T, ORDER>::value)) adj_xrow(AdjArgs<T> A, Lin3<T> init) {
    constexpr int R = (ORDER + 1) / 2, K = 2 * R - 1;
    constexpr int RPB = 256 / NX;        // rows per block
    constexpr int NP = NX + 2 * R - 1;   // padded row: cells -(R-1) .. NX+R-1 at p = cell + R - 1
    static_assert(NX >= 2 * R && RPB >= 1, "row longer than the stencil");
    __shared__ T sfp[5][RPB][NP];
    __shared__ T sfm[5][RPB][NP];
    __shared__ T sw[5][RPB][NX];
    __shared__ T sp[RPB][NX][K];         // plus partials of face x for cells x-R+1 .. x+R-1
    __shared__ T sm[RPB][NX][K];         // minus partials of face x for cells x-R+2 .. x+R
    const int tid = threadIdx.x;
    const int ly = tid / NX, x = tid - ly * NX;
    const long long row = (long long)blockIdx.x * RPB + ly;
    const bool live = row < (long long)A.n[1] * A.n[2];
    const long long id = x + (long long)NX * row;
    const T half = (T)0.5;

    T uf[5] = {(T)0, (T)0, (T)0, (T)0, (T)0};
    T kap = (T)0, kE = (T)0, kM2 = (T)0, pE = (T)0, pM2 = (T)0;
    {
        T fp[5] = {(T)0, (T)0, (T)0, (T)0, (T)0}, fm[5] = {(T)0, (T)0, (T)0, (T)0, (T)0};
        T w5[5] = {(T)0, (T)0, (T)0, (T)0, (T)0};
        if (live) {
#pragma unroll
            for (int f = 0; f < 5; ++f) {
                uf[f] = A.u[f * A.fstride + id];
                w5[f] = A.w[f * A.fstride + id];
            }
            // the recovery pack of the lane's cell (as adj_pack computes it),
            // also stored for the y and z sweeps
            const RecoveryPack o = recovery_pack((double)uf[0], (double)uf[1], (double)uf[2], (double)uf[3]);
            kap = (T)o.kap;
            const T P = (T)o.p;
            kE = (T)o.kap_E;
            kM2 = (T)o.kap_M2;
            pE = (T)o.p_E;
            pM2 = (T)o.p_M2;
            A.pk[id] = kap;
            A.pk[A.fstride + id] = P;
            A.pk[2 * A.fstride + id] = kE;
            A.pk[3 * A.fstride + id] = kM2;
            A.pk[4 * A.fstride + id] = pE;
            A.pk[5 * A.fstride + id] = pM2;
            const T v = kap * uf[1];
            T f[5];
            f[0] = uf[1];
            f[1] = uf[1] * v + P;
            f[2] = uf[2] * v;
            f[3] = uf[3] * v;
            f[4] = uf[4] * v;
#pragma unroll
            for (int c = 0; c < 5; ++c) {
                fp[c] = f[c] + uf[c];   // doubled split fluxes (eps scaled by 4 below)
                fm[c] = f[c] - uf[c];
            }
        }
        const int p = x + R - 1;
#pragma unroll
        for (int c = 0; c < 5; ++c) {
            sfp[c][ly][p] = fp[c];
            sfm[c][ly][p] = fm[c];
            sw[c][ly][x] = w5[c];
        }
        if (x >= NX - (R - 1)) {   // left ghosts -(R-1) .. -1
#pragma unroll
            for (int c = 0; c < 5; ++c) {
                sfp[c][ly][p - NX] = fp[c];
                sfm[c][ly][p - NX] = fm[c];
            }
        }
        if (x < R) {               // right ghosts NX .. NX+R-1
#pragma unroll
            for (int c = 0; c < 5; ++c) {
                sfp[c][ly][p + NX] = fp[c];
                sfm[c][ly][p + NX] = fm[c];
            }
        }
    }
    __syncthreads();

    const int xr = x + 1 < NX ? x + 1 : 0;
    T ap[5], am[5];
#pragma unroll 1
    for (int c = 0; c < 5; ++c) {
        {
            // face x (between cells x and x+1); its plus stencil starts at p = x
            T op[K], om[K];
#pragma unroll
            for (int k = 0; k < K; ++k) op[k] = om[k] = (T)0;
            const T g = (sw[c][ly][xr] - sw[c][ly][x]) * A.inv_h;
            if constexpr (ORDER == 5) {
                weno5_grad_acc_e<T>(sfp[c][ly][x], sfp[c][ly][x + 1], sfp[c][ly][x + 2], sfp[c][ly][x + 3],
                                    sfp[c][ly][x + 4], (T)16 * A.eps, g, op[0], op[1], op[2], op[3], op[4]);
                weno5_grad_acc_e<T>(sfm[c][ly][x + 5], sfm[c][ly][x + 4], sfm[c][ly][x + 3], sfm[c][ly][x + 2],
                                    sfm[c][ly][x + 1], (T)16 * A.eps, g, om[4], om[3], om[2], om[1], om[0]);
            } else {
                T sv[7], o[7];
#pragma unroll
                for (int j = 0; j < 7; ++j) {
                    sv[j] = sfp[c][ly][x + j];
                    o[j] = (T)0;
                }
                weno7_grad_acc<T>(sv, (T)4 * A.eps, g, o);
#pragma unroll
                for (int j = 0; j < 7; ++j) op[j] = o[j];
#pragma unroll
                for (int j = 0; j < 7; ++j) {
                    sv[j] = sfm[c][ly][x + 7 - j];
                    o[j] = (T)0;
                }
                weno7_grad_acc<T>(sv, (T)4 * A.eps, g, o);
#pragma unroll
                for (int j = 0; j < 7; ++j) om[6 - j] = o[j];
            }
#pragma unroll
            for (int k = 0; k < K; ++k) {
                sp[ly][x][k] = op[k];
                sm[ly][x][k] = om[k];
            }
        }
        __syncthreads();
        // partials reaching cell x: plus from faces x+R-1-k, minus from faces x+R-2-k
        T a_p = (T)0, a_m = (T)0;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            int fp_ = x + R - 1 - k, fm_ = x + R - 2 - k;
            fp_ = fp_ < 0 ? fp_ + NX : (fp_ >= NX ? fp_ - NX : fp_);
            fm_ = fm_ < 0 ? fm_ + NX : (fm_ >= NX ? fm_ - NX : fm_);
            a_p += sp[ly][fp_][k];
            a_m += sm[ly][fm_][k];
        }
        ap[c] = a_p;
        am[c] = a_m;
        __syncthreads();
    }
    if (!live) return;
    T lam[5], g[5];
#pragma unroll
    for (int c = 0; c < 5; ++c) {
        lam[c] = half * (ap[c] + am[c]);
        g[c] = half * (ap[c] - am[c]);
    }
    // F = (Mx, Mx v + p, My v, Mz v, N v) with v = kappa Mx
    const T Mx = uf[1], vd = kap * Mx;
    g[1] += lam[0];
    T S = (T)0;
#pragma unroll
    for (int c = 1; c < 5; ++c) {
        S += lam[c] * uf[c];
        g[c] += lam[c] * vd;
    }
    const T lp = lam[1];
    g[0] += S * (Mx * kE) + lp * pE;
    const T sk = (T)2 * S * Mx * kM2, spp = (T)2 * lp * pM2;
#pragma unroll
    for (int m = 0; m < 3; ++m) g[1 + m] += (sk + spp) * uf[1 + m];
    g[1] += S * kap;
#pragma unroll
    for (int f = 0; f < 5; ++f) {
        const long long o = f * A.fstride + id;
        T acc = (T)0;
        if (init.X1) acc += init.a1 * init.X1[o];
        if (init.X2) acc += init.a2 * init.X2[o];
        if (init.X3) acc += init.a3 * init.X3[o];
        A.ub[o] = acc + A.scale * g[f];
    }
}

// Tile of the x adjoint: the narrowest of 64, 32, 16 cells that wastes the
// least on a ragged row end (2R - 1 halo faces per row).  A 128 x 4 tile with
// two cells per lane halves the idle lanes of the last face round but needs
// twice the LDS; it measured 24% slower at 256^3 FP32.
int adjoint_tile_x(int nx) {
    int best = 64;
    double best_cost = 1e300;
    for (int tx : {64, 32, 16}) {
        const int ntx = (nx + tx - 1) / tx;
        const double cost = ntx * (tx + 5.0) / nx;
        if (cost < best_cost - 1e-12) {
            best_cost = cost;
            best = tx;
        }
    }
    return best;
}

template <class T>
__global__ void fill_zero(T* p, long long n) {
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x)
        p[i] = (T)0;
}

// out = a X + b Y + c Z + d V (null operands skipped)
template <class T>
__global__ void lincomb(T* out, long long n, T a, const T* X, T b, const T* Y, T c, const T* Z, T d,
                        const T* V) {
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x) {
        T v = (T)0;
        if (X) v += a * X[i];
        if (Y) v += b * Y[i];
        if (Z) v += c * Z[i];
        if (V) v += d * V[i];
        out[i] = v;
    }
}

static unsigned blocks_for(long long n) {
    long long b = (n + 255) / 256;
    if (b > 4096) b = 4096;
    if (b < 1) b = 1;
    return (unsigned)b;
}

// Axes whose adjoint is adj_small.  A rolling lane differentiates
// every face that reaches its segment, 2R - 1 more than it owns, one after another,
// and small grids give it few lanes.  Measured J^T w, rolls (with rows or adj_x along
// x) -> adj_small, us:
//   cells      33x20x17   48^3        64^3        72^3        80^3        96^3
//   WENO5 FP32  82 -> 14   91 -> 39    84 -> 57   122 -> 113              148 -> 180
//   WENO5 FP64 115 -> 18  132 -> 56   132 -> 91   196 -> 155  198 -> 183  251 -> 276
//   WENO7 FP32 139 -> 16  151 -> 46   145 -> 70   196 -> 125              247 -> 210
//   WENO7 FP64 168 -> 20  198 -> 69   186 -> 117  308 -> 200  271 -> 231  343 -> 352
// so the line lies at 400 000 cells in FP32 and 600 000 in FP64 (88^3: 249 -> 255 and
// 336 -> 322), and at 1.1 million for WENO7 in FP32, whose rolling window costs it a
// wave per SIMD (128x128x64: 251 -> 236).  A y or z axis of fewer than 16 cells counts
// as 16, the tile it occupies, where a rolling lane takes its few cells at once: y rolled
// -> y in tiles (z in tiles), us in the same order: 512x2x512 118 -> 297, 194 -> 479,
// 182 -> 375, 333 -> 643; 300x3x300 86 -> 130, 121 -> 199, 120 -> 158, 194 -> 260.
bool adjoint_small(int dir, const int n[3], int order, int elem) {
    const long long lines = (long long)n[0] * n[1] * n[2] / n[dir];
    const long long cells = lines * (dir > 0 && n[dir] < kSmallTX ? kSmallTX : n[dir]);
    return cells < (elem == 8 ? 600000 : order == 7 ? 1100000 : 400000);
}

// adj_x (FP32 WENO5) and the rolls read it.
bool adjoint_reads_pack(const int n[3], int bc_x, int order, int elem) {
    for (int d = 0; d < 3; ++d) {
        const bool recovers = d == 0 && (adjoint_x_rows(n, bc_x) || order != 5 || elem != 4);
        if (n[d] > 1 && !recovers && !adjoint_small(d, n, order, elem)) return true;
    }
    return false;
}

// Segment of the rolling adjoint: the length with the least estimated time, in
// units of one face of a block that has its CU to itself.  A lane differentiates
// seg + 2R - 1 faces after a fill worth about four; occ blocks share a CU (waves per
// SIMD that the registers allow) and slow each other to occ q.  Every length is
// tried, because whether the last blocks leave the chip idle counts for more than
// a few extra faces; a quarter of the estimate assumes that no CU is ever idle, as
// blocks of many rounds drift apart.  Lengths past 24 (WENO7 32) measured no faster.
// Against all lengths measured on nine grids of 405 000 to 16.8 million cells, the choices
// are within 7% of the best, 2% on average (the longest of 24, 16 and 8 with two
// blocks per CU: 28% and 6%).  J^T w by that rule and by this one, us: 96^3 FP64 WENO5 263
// -> 252, WENO7 353 -> 340; 110^3 FP64 WENO7 716 -> 567, FP32 WENO5 251 -> 238; 160^3 FP64
// WENO5 1416 -> 1308, WENO7 1781 -> 1667; 256^3 FP64 WENO7 5433 -> 5250; the largest loss
// 203x150x97 FP64 WENO5 1008 -> 1054.
int adjoint_segment(int nd, unsigned chunks, int order, int elem) {
    const int occ = elem == 4 ? 3 : order == 5 ? 2 : 1;
    const double q = occ == 3 ? 0.6 : occ == 2 ? 0.8 : 1.0;
    const int cap = order == 5 ? 24 : 32;
    int best = nd;
    double best_t = 1e300;
    for (int seg = nd < 4 ? nd : 4; seg <= (nd < cap ? nd : cap); ++seg) {
        const long long blocks = (long long)chunks * ((nd + seg - 1) / seg);
        const double alone = 4.0 + seg + order, all = occ * q * alone;   // 2R - 1 = order faces past the segment
        const long long per_cu = (blocks + 255) / 256, rest = per_cu % occ;
        double t = (per_cu / occ) * all;
        if (rest) t += occ > 1 ? alone * (1.0 + (occ * q - 1.0) * (rest - 1) / (occ - 1)) : alone;
        const double busy = blocks * q * alone / 256.0;
        t = 0.75 * t + 0.25 * (busy > alone ? busy : alone);
        if (t < best_t * (1.0 - 1e-9)) {
            best_t = t;
            best = seg;
        }
    }
    return best;
}

template <class T, int ORDER, int DIR>
static void launch_adjoint_small(AdjArgs<T> a, const Lin3<T>& init, hipStream_t s) {
    const long long lines = (long long)a.n[0] * a.n[1] * a.n[2] / a.n[DIR];
    const long long ntx = (a.n[DIR] + kSmallTX - 1) / kSmallTX, nrt = (lines + kSmallTY - 1) / kSmallTY;
    // A launch holds less than 2^32 lanes along x, and these tiles take eight per cell (x of
    // large grids runs to 10^9 cells): rows of at most 2^22 blocks, the few past the last
    // tile idle (no lane has a line).  Returning early there instead cost small grids a
    // second load of the arguments (12^3 FP32 WENO5: 11.4 against 12.0 us).
    const long long nblk = ntx * nrt, rows = (nblk + (1 << 22) - 1) >> 22;
    a.seg = (int)((nblk + rows - 1) / rows);
    const dim3 grid((unsigned)a.seg, (unsigned)rows);
    if constexpr (sizeof(T) == 8 && ORDER == 7) {
        if (nblk > 512) {
            adj_small<T, ORDER, DIR, true><<<grid, kSmallLanes, 0, s>>>(a, init);
            return;
        }
    }
    adj_small<T, ORDER, DIR, false><<<grid, kSmallLanes, 0, s>>>(a, init);
}

template <class T>
hipError_t launch_adjoint_sweep(int dir, int order, AdjArgs<T> a, hipStream_t s) {
    if (dir != 1 && dir != 2) return hipErrorInvalidValue;
    if (adjoint_small(dir, a.n, order, (int)sizeof(T))) {
        const Lin3<T> none = {(T)0, (T)0, (T)0, nullptr, nullptr, nullptr};
        if (order == 5) dir == 1 ? launch_adjoint_small<T, 5, 1>(a, none, s) : launch_adjoint_small<T, 5, 2>(a, none, s);
        else dir == 1 ? launch_adjoint_small<T, 7, 1>(a, none, s) : launch_adjoint_small<T, 7, 2>(a, none, s);
        return hipGetLastError();
    }
    if (!a.pk) return hipErrorInvalidValue;
    const int nd = a.n[dir];
    const long long plane = dir == 1 ? (long long)a.n[0] * a.n[2] : (long long)a.n[0] * a.n[1];
    const unsigned gx = (unsigned)((plane + 255) / 256);
    a.seg = adjoint_segment(nd, gx, order, (int)sizeof(T));
    const unsigned gy = (nd + a.seg - 1) / a.seg;
    const dim3 grid(gx, gy), block(256);
    const bool hub = a.bc == RH_BC_HUBBLE;
    auto go = [&](auto kernel) { kernel<<<grid, block, 0, s>>>(a); };
    if (order == 5) {
        if (dir == 1) hub ? go(adj_roll<T, 5, 1, true>) : go(adj_roll<T, 5, 1, false>);
        else hub ? go(adj_roll<T, 5, 2, true>) : go(adj_roll<T, 5, 2, false>);
    } else {
        if (dir == 1) hub ? go(adj_roll<T, 7, 1, true>) : go(adj_roll<T, 7, 1, false>);
        else hub ? go(adj_roll<T, 7, 2, true>) : go(adj_roll<T, 7, 2, false>);
    }
    return hipGetLastError();
}

// Whole-row x adjoint for periodic rows of these lengths (RH_ADJ_XROW=0 keeps
// the tiled kernel and the separate pack launch, for comparisons).
bool adjoint_x_rows(const int n[3], int bc_x) {
    static const bool enabled = [] {
        const char* e = getenv("RH_ADJ_XROW");
        return !(e && e[0] == '0');
    }();
    const int nx = n[0];
    return enabled && bc_x == RH_BC_PERIODIC &&
           (nx == 32 || nx == 64 || nx == 96 || nx == 128 || nx == 192 || nx == 256);
}

template <class T, int ORDER>
static void launch_adjoint_rows(const AdjArgs<T>& a, const Lin3<T>& init, hipStream_t s) {
    const int nx = a.n[0];
    const long long nrows = (long long)a.n[1] * a.n[2];
    auto go = [&](auto kernel, int nxk) {
        const int rpb = 256 / nxk;
        kernel<<<dim3((unsigned)((nrows + rpb - 1) / rpb)), dim3(rpb * nxk), 0, s>>>(a, init);
    };
    switch (nx) {
        case 32: go(adj_xrow<T, ORDER, 32>, 32); break;
        case 64: go(adj_xrow<T, ORDER, 64>, 64); break;
        case 96: go(adj_xrow<T, ORDER, 96>, 96); break;
        case 128: go(adj_xrow<T, ORDER, 128>, 128); break;
        case 192: go(adj_xrow<T, ORDER, 192>, 192); break;
        default: go(adj_xrow<T, ORDER, 256>, 256); break;
    }
}

template <class T>
hipError_t launch_adjoint_x(int order, AdjArgs<T> a, Lin3<T> init, hipStream_t s) {
    if (!a.pk) return hipErrorInvalidValue;
    if (adjoint_x_rows(a.n, a.bc)) {
        if (order == 5) launch_adjoint_rows<T, 5>(a, init, s);
        else launch_adjoint_rows<T, 7>(a, init, s);
        return hipGetLastError();
    }
    // adj_small on whatever size: three barriers a tile where adj_x has eleven.  Only
    // FP32 WENO5, whose faces are the cheapest, is ahead with adj_x's longer tiles on
    // large grids.  J^T w, adj_x -> adj_small along x, us: 130x128x128 FP64 915 -> 868,
    // WENO7 1253 -> 1171, FP32 WENO7 614 -> 578, but FP32 WENO5 390 -> 393; 300x200x60
    // FP64 1326 -> 1319, WENO7 1680 -> 1632, FP32 WENO7 846 -> 784, FP32 WENO5 545 -> 570.
    if constexpr (sizeof(T) == 4) {
        if (order == 5 && !adjoint_small(0, a.n, order, (int)sizeof(T))) {
            const int tx = adjoint_tile_x(a.n[0]);
            const int ty = tx == 64 ? 4 : 256 / tx;
            const long long ntx = (a.n[0] + tx - 1) / tx;
            const long long nrt = ((long long)a.n[1] * a.n[2] + ty - 1) / ty;
            const dim3 grid((unsigned)(ntx * nrt));
            if (tx == 64) adj_x<T, 64, 4><<<grid, 256, 0, s>>>(a, init);
            else if (tx == 32) adj_x<T, 32, 8><<<grid, 256, 0, s>>>(a, init);
            else adj_x<T, 16, 16><<<grid, 256, 0, s>>>(a, init);
            return hipGetLastError();
        }
    }
    order == 5 ? launch_adjoint_small<T, 5, 0>(a, init, s) : launch_adjoint_small<T, 7, 0>(a, init, s);
    return hipGetLastError();
}

template <class T>
hipError_t launch_adjoint_pack(const T* u, T* pk, long long ncell, hipStream_t s) {
    adj_pack<T><<<blocks_for(ncell), 256, 0, s>>>(u, pk, ncell);
    return hipGetLastError();
}

template <class T>
hipError_t launch_fill_zero(T* p, long long n, hipStream_t s) {
    fill_zero<T><<<blocks_for(n), 256, 0, s>>>(p, n);
    return hipGetLastError();
}

template <class T>
hipError_t launch_lincomb(T* out, long long n, T a, const T* X, T b, const T* Y, T c, const T* Z, T d,
                          const T* V, hipStream_t s) {
    lincomb<T><<<blocks_for(n), 256, 0, s>>>(out, n, a, X, b, Y, c, Z, d, V);
    return hipGetLastError();
}

#define RH_ADJ_INSTANTIATE(T)                                                                      \
    template hipError_t launch_adjoint_sweep<T>(int, int, AdjArgs<T>, hipStream_t);               \
    template hipError_t launch_fill_zero<T>(T*, long long, hipStream_t);                          \
    template hipError_t launch_adjoint_pack<T>(const T*, T*, long long, hipStream_t);             \
    template hipError_t launch_adjoint_x<T>(int, AdjArgs<T>, Lin3<T>, hipStream_t);                \
    template hipError_t launch_lincomb<T>(T*, long long, T, const T*, T, const T*, T, const T*, T, \
                                          const T*, hipStream_t);

RH_ADJ_INSTANTIATE(float)
RH_ADJ_INSTANTIATE(double)

}  // namespace rh
