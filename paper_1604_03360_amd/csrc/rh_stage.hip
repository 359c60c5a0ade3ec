// rh_stage.hip -- one launch per SSP-RK3 stage for gfx950.
//
// stage_fused evaluates the whole operator L(u) of Eq. (2) (Sikorski et al.,
// arXiv:1604.03360) -- the x, y and z flux differences -- and applies the
// Runge-Kutta stage combine (Sec. 1) in a single launch, with no L accumulator
// in memory.  A work item is (grid, x-y tile of TX x TY = 256 cells, z segment):
// the block rolls along its z segment one plane at a time.  Each lane owns one
// (x, y) column of the tile and keeps a register window of 2R doubled split
// fluxes along z (as the rolling sweeps do), R planes ahead of the plane that is
// finished.  For that plane the block stages the tile's doubled x and y split
// fluxes in LDS, with R halo cells on each side along x and along y (no corners
// are needed), and reconstructs every x and y face of the tile once; the z faces
// come from the window, so the plane is complete and stored at once.  A cell of
// the tile is loaded and recovered (FP64) twice, when it enters the z window and
// when its own plane is staged.  The second recovery costs about 50 of 1300
// instructions per cell; keeping the x + y part of L for R planes instead (one
// recovery, a register ring, the stage input loaded again for the combine) took
// 15 more registers and a fill of 2R dependent planes, and measured 2.18 against
// 1.94 ms per FP32 WENO5 step and 3.98 against 3.63 ms in FP64 at 256^3, and 34.6
// against 30.0 us at 16^3.  The window's 2R planes are loaded before the first
// is recovered, so that a segment of one plane waits for memory once.  What bounds
// it: VALU issue where the chip is full (FP32: three waves per SIMD, 165
// registers; capped at 128 registers for a fourth, the spills cost 14%); the dependent chains of
// recovery and reconstruction of one plane (about 5 us) where it is not.
//
// The arithmetic of every face, flux difference and combine is that of the
// split sweeps, summed in the same order (x, then y, then z), so the result is
// bitwise that of the x, y and z sweeps run one after another.
//
// Ensembles use the same kernel: each block finds its grid in a table sorted
// by first block, so one launch covers every grid of the batch.
//
// Two generalisations of the flux step are instantiated here as well: local
// Lax-Friedrichs splitting (LOCAL: the block stages the physical flux and the
// state of each cell with its largest characteristic speed, and every face
// reconstructs F +- alpha u with alpha the largest speed of its 2R stencil
// cells), and the ideal-gas equation of state (EOS_IDEAL: a recovery pass
// solves for every cell's velocity and pressure once per evaluation of L, and
// the stage reads them with the state).  An axis of one cell contributes
// nothing to L.
#include "rh_face.hpp"
#include "rh_internal.hpp"
#include "../../include/rh.h"

namespace rh {

// Minimum resident blocks per CU (= waves per SIMD) for the register budget.  FP32
// WENO5 runs three waves (local splitting too: 174 registers for two, 192^3 step 1256
// us; 168 for three, 1141), except where analytic ghosts and local splitting together
// would spill 41 registers.  FP64 blocks other than WENO5 16 x 16 with global
// splitting need more than half of the 160 KB LDS.
template <class T, int ORDER, int TX, bool HUB, bool LOCAL>
struct StageMinBlocks {
    static constexpr int value = sizeof(T) == 4 ? (ORDER == 5 && !(HUB && LOCAL) ? 3 : 2)
                                                : (ORDER == 5 && TX == 16 && !LOCAL ? 2 : 1);
};

template <class T, int DIR, bool LOCAL>
__device__ __forceinline__ void stage_pair(const T u[5], T v, T P, T a[5], T b[5]) {
    if constexpr (LOCAL) {
        a[0] = u[1 + DIR];
        a[1] = u[1] * v + (DIR == 0 ? P : (T)0);
        a[2] = u[2] * v + (DIR == 1 ? P : (T)0);
        a[3] = u[3] * v + (DIR == 2 ? P : (T)0);
        a[4] = u[4] * v;
#pragma unroll
        for (int c = 0; c < 5; ++c) b[c] = u[c];
    } else {
        split_flux_vp<T, DIR>(u, v, P, a, b);
    }
}

// SPARSE: for grids that fill a quarter of their tiles or less.  Waves without a cell then
// free their SIMD instead of following the z window (FP32 WENO7 ensemble of six 256x4x256
// grids 1256 -> 1106 us per step); on full tiles the branch keeps the loads of the next plane
// from overlapping it (33^3 62 -> 72, FP32 WENO5 128^3 265 -> 292).
template <class T, int ORDER, int TX, bool HUB, bool LOCAL, int EOS, bool SPARSE = false>
__global__ void __launch_bounds__(256, (StageMinBlocks<T, ORDER, TX, HUB, LOCAL>::value)) stage_fused(StageArgs<T> A) {
    constexpr int R = (ORDER + 1) / 2, W = 2 * R, TY = 256 / TX;
    static_assert(W * (TX + TY) <= 256, "one halo cell per lane and plane");
    static_assert(5 * (TX + TY) <= 256, "one edge face (all components) per lane");
    constexpr int SX = TX + 2 * R;            // staged x row: R ghosts, TX cells, R ghosts
    constexpr int SY = TY + 2 * R;
    constexpr int SPX = LOCAL ? TY : 1, SPY = LOCAL ? SY : 1;
    __shared__ T sx[2][5][TY][SX];            // doubled x split fluxes (plus, minus), or (F, u) with LOCAL
    __shared__ T sy[2][5][SY][TX];            // the same along y
    __shared__ T ssx[SPX][LOCAL ? SX : 1];    // LOCAL: largest speed along x of the staged cells
    __shared__ T ssy[SPY][LOCAL ? TX : 1];    // LOCAL: largest speed along y
    __shared__ T fx[5][TY][TX + 1];           // x face fluxes: column 0 = left face of the tile, 1 + i = right face of cell i
    __shared__ T fy[5][TY + 1][TX];           // y face fluxes: row 0 = lower face of the tile, 1 + j = upper face of row j

    const int b = xcd_logical((int)blockIdx.x, (int)gridDim.x);
    const StageGrid<T> G = A.ngrid > 0 ? A.grids[stage_grid_of(A, b)] : A.one;
    const int lb = b - G.blk0;
    const int tpp = G.ntx * G.nty;
    const int zs = lb / tpp, rem = lb - zs * tpp;
    const int tyi = rem / G.ntx, txi = rem - tyi * G.ntx;
    const int nx = G.n[0], ny = G.n[1], nz = G.n[2];
    const int x0 = txi * TX, y0 = tyi * TY;
    const int xa = min(TX, nx - x0), ya = min(TY, ny - y0);
    const int k0 = zs * G.seg, kend = min(k0 + G.seg, nz);
    const long long F = (long long)nx * ny * nz;
    const T* us = A.us + G.off;
    const T* u0 = A.u0 + G.off;
    T* out = A.out + G.off;
    const double t = A.t;
    // an axis of one cell contributes nothing to L
    const bool dox = nx > 1, doy = ny > 1, doz = nz > 1;

    const int tid = threadIdx.x, lx = tid % TX, ly = tid / TX;
    const bool act = lx < xa && ly < ya;
    // lanes outside a ragged tile follow the loop on a valid cell and store nothing; with
    // SPARSE they leave the z window out
    const bool inz = !SPARSE || act;
    const int cx = x0 + min(lx, xa - 1), cy = y0 + min(ly, ya - 1);
    const uint32_t sb = (uint32_t)sizeof(T) * (uint32_t)nx * (uint32_t)ny;   // z plane, bytes
    const uint32_t cb = (uint32_t)sizeof(T) * ((uint32_t)cx + (uint32_t)nx * (uint32_t)cy);

    // halo job of this lane: one x-halo cell (row r, staged column p; cell x0 - R + p)
    // or one y-halo cell (column c, staged row q; cell y0 - R + q), the same every plane
    const int nxh = W * ya, nyh = W * xa;
    int hkind = 0, hr = 0, hc = 0, hxc = 0, hyc = 0;
    if (tid < nxh) {
        const int j = tid % W;
        hkind = 1;
        hr = tid / W;
        hc = j < R ? j : xa + j;
        hxc = x0 - R + hc;
        hyc = y0 + hr;
    } else if (tid < nxh + nyh) {
        const int s = tid - nxh, j = s % W;
        hkind = 2;
        hc = s / W;
        hr = j < R ? j : ya + j;
        hxc = x0 + hc;
        hyc = y0 - R + hr;
    }

    // The halo cell's place in a plane is the same every plane: its ghost index is
    // taken once (per plane and cell: 53.9 against 52.6 us per step at 48^3 FP64).
    // Analytic ghost cells load the edge cell like outflow ones and are replaced
    // where they are used, so that the loads of the next plane stay in flight without
    // the evaluation's registers (evaluated in place of the load, the loads of the
    // next plane waited: 192^3 FP64 1670 against 1572 us, FP32 886 against 832).
    const int hxi = hxc >= 0 && hxc < nx ? hxc : ghost_index(hxc, nx, G.bc[0]);
    const int hyi = hyc >= 0 && hyc < ny ? hyc : ghost_index(hyc, ny, G.bc[1]);
    const uint32_t hb = (uint32_t)sizeof(T) * ((uint32_t)hxi + (uint32_t)nx * (uint32_t)hyi);
    const bool hana = HUB && hkind && ((G.bc[0] == RH_BC_HUBBLE && (hxc < 0 || hxc >= nx)) ||
                                       (G.bc[1] == RH_BC_HUBBLE && (hyc < 0 || hyc >= ny)));
    auto plane_of = [&](int m) { return m >= 0 && m < nz ? m : ghost_index(m, nz, G.bc[2]); };
    auto load_at = [&](const T* base, uint32_t at, int k, T u[5]) {   // plane k of the grid
        const uint32_t off = at + (uint32_t)k * sb;
#pragma unroll
        for (int f = 0; f < 5; ++f) u[f] = ld_off(base + f * F, off);
    };
    auto analytic = [&](int x, int y, int z, T u[5]) {
        HubbleBC hbc;
        hbc.t = t;
        hbc.t0 = G.t0;
        hbc.e0 = G.e0;
        hbc.n0 = G.n0;
        double uh[5];
        hubble_conserved(hbc, G.c0[0] + x * G.h[0], G.c0[1] + y * G.h[1], G.c0[2] + z * G.h[2], uh);
#pragma unroll
        for (int f = 0; f < 5; ++f) u[f] = (T)uh[f];
    };
    auto fetch_plane = [&](int k, T u[5]) { load_at(us, cb, k, u); };          // own cell of plane k
    auto fetch_own = [&](int m, T u[5]) { load_at(us, cb, plane_of(m), u); };  // the same, or a ghost plane's
    auto fetch_halo = [&](int k, T u[5]) {
        if (hkind) load_at(us, hb, k, u);
    };
    // ideal gas: the recovery pass's (vx, vy, vz, p, c_s^2) of the same cells
    const T* pr = EOS == EOS_IDEAL ? A.prim + G.off : nullptr;
    auto fetch_own_prim = [&](int m, T q[5]) {
        if constexpr (EOS == EOS_IDEAL) load_at(pr, cb, plane_of(m), q);
    };
    auto fetch_halo_prim = [&](int k, T q[5]) {
        if constexpr (EOS == EOS_IDEAL) load_at(pr, hb, k, q);
    };

    const T eps2 = (T)4 * G.eps;   // epsilon of the doubled split fluxes
    const T hxinv = (T)0.5 * G.inv_h[0], hyinv = (T)0.5 * G.inv_h[1], hzinv = (T)0.5 * G.inv_h[2];
    unsigned clamped = 0;

    T zp[5][W], zm[5][W];     // z window: staged pairs of cells k - R .. k + R - 1
    T zsp[LOCAL ? W : 1];     // LOCAL: their largest speeds along z

    // z pair of a cell entering the window (and its largest speed along z)
    auto z_pair = [&](int m, T u[5], T fp[5], T fm[5], T& speed) {
        if (HUB && G.bc[2] == RH_BC_HUBBLE && (m < 0 || m >= nz)) analytic(cx, cy, m, u);
        T VZ, P;
        if constexpr (EOS == EOS_IDEAL) {
            T q[5];
            fetch_own_prim(m, q);
            VZ = q[2];
            P = q[3];
            if constexpr (LOCAL) {
                const double vx = (double)q[0], vy = (double)q[1], vz = (double)VZ;
                speed = (T)max_char_speed(vz, vx * vx + vy * vy + vz * vz, (double)q[4]);
            }
        } else {
            unsigned dummy = 0;   // floors are counted when the cell's own plane is staged
            if constexpr (LOCAL) {
                double kap, Mxs, Mys, Mzs, p;
                recover_kp3<HUB>((double)u[0], (double)u[1], (double)u[2], (double)u[3], kap, Mxs, Mys, Mzs, p, dummy);
                VZ = (T)(kap * Mzs);
                P = (T)p;
                speed = (T)max_char_speed(kap * Mzs, kap * kap * (Mxs * Mxs + Mys * Mys + Mzs * Mzs), 1.0 / 3.0);
            } else {
                double vd, p;
                recover_vp<2, HUB>((double)u[0], (double)u[1], (double)u[2], (double)u[3], vd, p, dummy);
                VZ = (T)vd;
                P = (T)p;
            }
        }
        stage_pair<T, 2, LOCAL>(u, VZ, P, fp, fm);
    };

    // Stage the x and y pairs of the own cell of plane k and of the lane's halo
    // cell in LDS.
    auto stage_xy = [&](int k, const T u[5], T hu[5]) {
        T fp[5], fm[5];
        if (act) {
            T VX, VY, P;
            double vxd, vyd, v2 = 0.0, cs2 = 0.0;
            unsigned c0 = 0;
            if constexpr (EOS == EOS_IDEAL) {
                T q[5];
                fetch_own_prim(k, q);
                VX = q[0];
                VY = q[1];
                P = q[3];
                vxd = (double)VX;
                vyd = (double)VY;
                if constexpr (LOCAL) {
                    const double vzd = (double)q[2];
                    v2 = vxd * vxd + vyd * vyd + vzd * vzd;
                    cs2 = (double)q[4];
                }
            } else {
                double kap, Mxs, Mys, p;
                if constexpr (!LOCAL) {
                    recover_kp<HUB>((double)u[0], (double)u[1], (double)u[2], (double)u[3], kap, Mxs, Mys, p, c0);
                } else {
                    double Mzs;
                    recover_kp3<HUB>((double)u[0], (double)u[1], (double)u[2], (double)u[3], kap, Mxs, Mys, Mzs, p, c0);
                    v2 = kap * kap * (Mxs * Mxs + Mys * Mys + Mzs * Mzs);
                    cs2 = 1.0 / 3.0;
                }
                vxd = kap * Mxs;
                vyd = kap * Mys;
                VX = (T)vxd;
                VY = (T)vyd;
                P = (T)p;
            }
            clamped += c0;   // floors counted once per owned cell and evaluation of L
            stage_pair<T, 0, LOCAL>(u, VX, P, fp, fm);
#pragma unroll
            for (int c = 0; c < 5; ++c) {
                sx[0][c][ly][R + lx] = fp[c];
                sx[1][c][ly][R + lx] = fm[c];
            }
            stage_pair<T, 1, LOCAL>(u, VY, P, fp, fm);
#pragma unroll
            for (int c = 0; c < 5; ++c) {
                sy[0][c][R + ly][lx] = fp[c];
                sy[1][c][R + ly][lx] = fm[c];
            }
            if constexpr (LOCAL) {
                ssx[ly][R + lx] = (T)max_char_speed(vxd, v2, cs2);
                ssy[R + ly][lx] = (T)max_char_speed(vyd, v2, cs2);
            }
        }
        if (HUB && hana) analytic(hxc, hyc, k, hu);
        if (hkind) {
            T HX, HY, HP;
            double hxd, hyd, hv2 = 0.0, hcs2 = 0.0;
            if constexpr (EOS == EOS_IDEAL) {
                T phu[5];
                fetch_halo_prim(k, phu);
                HX = phu[0];
                HY = phu[1];
                HP = phu[3];
                hxd = (double)HX;
                hyd = (double)HY;
                if constexpr (LOCAL) {
                    const double hzd = (double)phu[2];
                    hv2 = hxd * hxd + hyd * hyd + hzd * hzd;
                    hcs2 = (double)phu[4];
                }
            } else {
                double hk, hMx, hMy, hp;
                unsigned hcl = 0;
                if constexpr (!LOCAL) {
                    recover_kp<HUB>((double)hu[0], (double)hu[1], (double)hu[2], (double)hu[3], hk, hMx, hMy, hp, hcl);
                } else {
                    double hMz;
                    recover_kp3<HUB>((double)hu[0], (double)hu[1], (double)hu[2], (double)hu[3], hk, hMx, hMy, hMz, hp,
                                hcl);
                    hv2 = hk * hk * (hMx * hMx + hMy * hMy + hMz * hMz);
                    hcs2 = 1.0 / 3.0;
                }
                hxd = hk * hMx;
                hyd = hk * hMy;
                HX = (T)hxd;
                HY = (T)hyd;
                HP = (T)hp;
            }
            if (hkind == 1) {
                stage_pair<T, 0, LOCAL>(hu, HX, HP, fp, fm);
#pragma unroll
                for (int c = 0; c < 5; ++c) {
                    sx[0][c][hr][hc] = fp[c];
                    sx[1][c][hr][hc] = fm[c];
                }
                if constexpr (LOCAL) ssx[hr][hc] = (T)max_char_speed(hxd, hv2, hcs2);
            } else {
                stage_pair<T, 1, LOCAL>(hu, HY, HP, fp, fm);
#pragma unroll
                for (int c = 0; c < 5; ++c) {
                    sy[0][c][hr][hc] = fp[c];
                    sy[1][c][hr][hc] = fm[c];
                }
                if constexpr (LOCAL) ssy[hr][hc] = (T)max_char_speed(hyd, hv2, hcs2);
            }
        }
    };

    // x and y faces of the staged plane
    auto faces_xy = [&]() {
        if (act) {
            T ax = (T)0, ay = (T)0;
            if constexpr (LOCAL) {
#pragma unroll
                for (int j = 0; j < W; ++j) {
                    ax = max(ax, ssx[ly][lx + 1 + j]);
                    ay = max(ay, ssy[ly + 1 + j][lx]);
                }
            }
#pragma unroll
            for (int c = 0; c < 5; ++c) {
                // window of face x + 1/2: staged columns lx + 1 .. lx + 2R
                if constexpr (LOCAL) {
                    T wa[W], wb[W];
#pragma unroll
                    for (int j = 0; j < W; ++j) {
                        wa[j] = sx[0][c][ly][lx + 1 + j];
                        wb[j] = sx[1][c][ly][lx + 1 + j];
                    }
                    fx[c][ly][lx + 1] = recon_local<T, ORDER>(wa, wb, ax, eps2);
                } else {
                    fx[c][ly][lx + 1] = stage_recon_plus<T, ORDER>(&sx[0][c][ly][lx + 1], eps2) +
                                        stage_recon_minus<T, ORDER>(&sx[1][c][ly][lx + 1], eps2);
                }
                T wp[W], wm[W];
#pragma unroll
                for (int j = 0; j < W; ++j) {
                    wp[j] = sy[0][c][ly + 1 + j][lx];
                    wm[j] = sy[1][c][ly + 1 + j][lx];
                }
                if constexpr (LOCAL) fy[c][ly + 1][lx] = recon_local<T, ORDER>(wp, wm, ay, eps2);
                else fy[c][ly + 1][lx] = stage_recon_plus<T, ORDER>(wp, eps2) + stage_recon_minus<T, ORDER>(wm, eps2);
            }
        }
        // faces on the lower edges of the tile, one (line, component) per lane:
        // 5 ya x jobs (window at staged column 0), then 5 xa y jobs (staged row 0)
        if (tid < 5 * ya) {
            const int r = tid / 5, c = tid - 5 * r;
            if constexpr (LOCAL) {
                T wa[W], wb[W], al = (T)0;
#pragma unroll
                for (int j = 0; j < W; ++j) {
                    wa[j] = sx[0][c][r][j];
                    wb[j] = sx[1][c][r][j];
                    al = max(al, ssx[r][j]);
                }
                fx[c][r][0] = recon_local<T, ORDER>(wa, wb, al, eps2);
            } else {
                fx[c][r][0] = stage_recon_plus<T, ORDER>(&sx[0][c][r][0], eps2) +
                              stage_recon_minus<T, ORDER>(&sx[1][c][r][0], eps2);
            }
        } else if (tid < 5 * (ya + xa)) {
            const int s = tid - 5 * ya, col = s / 5, c = s - 5 * col;
            T wp[W], wm[W];
#pragma unroll
            for (int j = 0; j < W; ++j) {
                wp[j] = sy[0][c][j][col];
                wm[j] = sy[1][c][j][col];
            }
            if constexpr (LOCAL) {
                T al = (T)0;
#pragma unroll
                for (int j = 0; j < W; ++j) al = max(al, ssy[j][col]);
                fy[c][0][col] = recon_local<T, ORDER>(wp, wm, al, eps2);
            } else {
                fy[c][0][col] = stage_recon_plus<T, ORDER>(wp, eps2) + stage_recon_minus<T, ORDER>(wm, eps2);
            }
        }
    };
    // z face above the window's centre, component c
    auto zface = [&](int c) {
        if constexpr (LOCAL) {
            T al = (T)0;
#pragma unroll
            for (int j = 0; j < W; ++j) al = max(al, zsp[j]);
            return recon_local<T, ORDER>(zp[c], zm[c], al, eps2);
        } else {
            return stage_recon_plus<T, ORDER>(zp[c], eps2) + stage_recon_minus<T, ORDER>(zm[c], eps2);
        }
    };

    // z window of face k0 - 1/2: planes k0 - R .. k0 + R - 1, all loads issued
    // before the first recovery (a block of few planes waits once, not 2R times)
    if (inz) {
        T fu[W][5];
#pragma unroll
        for (int j = 0; j < W; ++j) fetch_own(k0 - R + j, fu[j]);
#pragma unroll
        for (int j = 0; j < W; ++j) {
            T fp[5], fm[5], sz = (T)0;
            z_pair(k0 - R + j, fu[j], fp, fm, sz);
#pragma unroll
            for (int c = 0; c < 5; ++c) {
                zp[c][j] = fp[c];
                zm[c][j] = fm[c];
            }
            if constexpr (LOCAL) zsp[j] = sz;
        }
    }
    // operands of the next plane, in flight during this one
    T nz5[5], no5[5], nh5[5] = {(T)0, (T)0, (T)0, (T)0, (T)0};
    fetch_own(k0 + R, nz5);
    fetch_plane(k0, no5);
    fetch_halo(k0, nh5);
    T Fl[5];
    if (inz) {
#pragma unroll
        for (int c = 0; c < 5; ++c) Fl[c] = zface(c);
    }

    for (int k = k0; k < kend; ++k) {
        T uz[5], u[5];
#pragma unroll
        for (int f = 0; f < 5; ++f) {
            uz[f] = nz5[f];
            u[f] = no5[f];
        }
        stage_xy(k, u, nh5);
        if (k + 1 < kend) {
            fetch_own(k + 1 + R, nz5);
            fetch_plane(k + 1, no5);
            fetch_halo(k + 1, nh5);
        }
        T Lz[5];
        if (inz) {
            T fp[5], fm[5], sz = (T)0;
            z_pair(k + R, uz, fp, fm, sz);
#pragma unroll
            for (int c = 0; c < 5; ++c) {
#pragma unroll
                for (int j = 0; j < W - 1; ++j) {
                    zp[c][j] = zp[c][j + 1];
                    zm[c][j] = zm[c][j + 1];
                }
                zp[c][W - 1] = fp[c];
                zm[c][W - 1] = fm[c];
            }
            if constexpr (LOCAL) {
#pragma unroll
                for (int j = 0; j < W - 1; ++j) zsp[j] = zsp[j + 1];
                zsp[W - 1] = sz;
            }
#pragma unroll
            for (int c = 0; c < 5; ++c) {
                // the z face is reconstructed for every grid (on ghost copies where nz is
                // 1) and discarded by a select, which keeps it out of a branch
                const T Fr = zface(c);
                Lz[c] = doz ? (Fl[c] - Fr) * hzinv : (T)0;
                Fl[c] = Fr;
            }
        }
        const uint32_t off = cb + (uint32_t)k * sb;
        T u0k[5];
#pragma unroll
        for (int c = 0; c < 5; ++c) u0k[c] = A.stage >= STAGE_2 ? ld_off(u0 + c * F, off) : (T)0;
        __syncthreads();
        faces_xy();
        __syncthreads();
#pragma unroll
        for (int c = 0; c < 5; ++c) {
            const T Lx = dox ? (fx[c][ly][lx] - fx[c][ly][lx + 1]) * hxinv : (T)0;
            const T Ly = doy ? (fy[c][ly][lx] - fy[c][ly + 1][lx]) * hyinv : (T)0;
            const T L = (Lx + Ly) + Lz[c];
            T v;
            if (A.stage == STAGE_WRITE_L) {
                v = L;
            } else {
                v = u[c] + A.dt * L;
                if (A.stage == STAGE_2) v = (T)0.75 * u0k[c] + (T)0.25 * v;
                else if (A.stage == STAGE_3) v = rk3_last(u0k[c], v);
            }
            if (act) st_off(out + c * F, off, v);
        }
    }
    if (clamped) atomicAdd(A.clamps, clamped);
}

// Ideal-gas recovery pass: every cell of every grid once per evaluation of L
// (the stage kernel reads the result for its own and halo cells, so the Newton
// iteration runs once per cell instead of once per staging).
template <class T>
__global__ void __launch_bounds__(256) recover_ideal_cells(StageArgs<T> A) {
    const int b = (int)blockIdx.x;
    int g = 0;
    if (A.ngrid > 0) {
        int lo = 0, hi = A.ngrid - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (A.grids[mid].rblk0 <= b) lo = mid;
            else hi = mid - 1;
        }
        g = lo;
    }
    const StageGrid<T>& G = A.ngrid > 0 ? A.grids[g] : A.one;
    const long long n = (long long)G.n[0] * G.n[1] * G.n[2];
    const long long i = (long long)(b - G.rblk0) * 256 + threadIdx.x;
    unsigned cl = 0;
    if (i < n) {
        const T* u = A.us + G.off;
        T* q = A.prim + G.off;
        double kap, Mxs, Mys, Mzs, p, e;
        recover_ideal((double)u[i], (double)u[n + i], (double)u[2 * n + i], (double)u[3 * n + i],
                      (double)u[4 * n + i], G.gm1, kap, Mxs, Mys, Mzs, p, e, cl);
        q[i] = (T)(kap * Mxs);
        q[n + i] = (T)(kap * Mys);
        q[2 * n + i] = (T)(kap * Mzs);
        q[3 * n + i] = (T)p;
        q[4 * n + i] = (T)(e + p > 0.0 ? (G.gm1 + 1.0) * p / (e + p) : 0.0);
    }
    if (cl) atomicAdd(A.clamps, cl);
}

template <class T>
hipError_t launch_recover_ideal(const StageArgs<T>& a, long long nblocks, hipStream_t s) {
    if (nblocks <= 0 || nblocks > 0x7fffffffLL) return hipErrorInvalidValue;
    recover_ideal_cells<T><<<dim3((unsigned)nblocks), 256, 0, s>>>(a);
    return hipGetLastError();
}

template hipError_t launch_recover_ideal<float>(const StageArgs<float>&, long long, hipStream_t);
template hipError_t launch_recover_ideal<double>(const StageArgs<double>&, long long, hipStream_t);

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
// z segment of the stage kernels (fused WENO and MUSTA-FORCE) for the grids of a
// launch: the length with the least estimated time, in units of one plane of a block that has its CU to
// itself.  Such a block takes 1 + seg (its fill costs about one plane); occ blocks
// share a CU and then take occ q (0.6 + seg) together, and part of them a time in
// between.  Every length is tried: what a few planes more cost counts less than
// whether the last blocks leave the chip idle (96^3 FP64 WENO5: 214 us per step at 7
// planes, 504 blocks on 512 slots; 267 at 6, 233 at 8).  Against all segments measured
// for 64^3 .. 160^3, both orders and precisions, and MUSTA-FORCE for 24^3 .. 256^3, the
// choices are within 2% of the best (MUSTA-FORCE 5%).  Before, MUSTA-FORCE took segments
// of at least 8 planes: 24^3 172 us per FP32 step, now 36; 128^3 FP64 611, now 559.
int stage_segment(int ngrid, const int (*n)[3], int tx, int scheme, int elem, bool local, double* planes_out) {
    const bool musta = scheme == RH_SCHEME_MUSTA, light = scheme == 5 && (elem == 4 || !local);
    const int ty = musta ? kMustaTY : 256 / tx;
    int occ;
    double q;
    if (musta) {
        occ = elem == 4 ? 3 : 2;
        q = elem == 4 ? 0.51 : 0.70;
    } else if (elem == 4) {
        occ = light ? 3 : 2;
        q = light ? 0.46 : 0.62;
    } else {
        occ = light && tx == 16 ? 2 : 1;
        q = occ == 2 ? 0.74 : 1.05;
    }
    int best = 1;
    double best_t = 1e300;
    for (int seg = 1; seg <= 64; ++seg) {
        long long blocks = 0;
        int planes = 1;
        for (int g = 0; g < ngrid; ++g) {
            const int nseg = (n[g][2] + seg - 1) / seg;
            blocks += (long long)((n[g][0] + tx - 1) / tx) * ((n[g][1] + ty - 1) / ty) * nseg;
            if (n[g][2] > planes) planes = n[g][2];
        }
        const double alone = 1.0 + (seg < planes ? seg : planes), all = occ * q * (0.6 + seg);
        const long long per_cu = (blocks + 255) / 256, rest = per_cu % occ;
        double t = (per_cu / occ) * (all > alone ? all : alone);
        if (rest) t += occ > 1 ? alone * (1.0 + (occ * q - 1.0) * (rest - 1) / (occ - 1)) : alone;
        if (t < best_t * (1.0 - 1e-9)) {
            best_t = t;
            best = seg;
        }
        if (seg >= planes) break;
    }
    if (planes_out) *planes_out = best_t;
    return best;
}

bool stage_sparse(int ngrid, const int (*n)[3]) {
    long long cells = 0, lanes = 0;
    for (int g = 0; g < ngrid; ++g) {
        cells += (long long)n[g][0] * n[g][1] * n[g][2];
        lanes += 256LL * ((n[g][0] + 15) / 16) * ((n[g][1] + 15) / 16) * n[g][2];
    }
    return lanes >= 4 * cells;
}

template <class T>
void stage_shape(StageGrid<T>& g, int tx, int seg) {
    const int ty = 256 / tx;
    if (seg < 1) seg = 1;
    if (seg > g.n[2]) seg = g.n[2];
    g.ntx = (g.n[0] + tx - 1) / tx;
    g.nty = (g.n[1] + ty - 1) / ty;
    g.seg = seg;
    g.nseg = (g.n[2] + seg - 1) / seg;
}

template <class T, int ORDER, int TX>
static hipError_t launch_stage_t(bool hub, bool local, int eos, bool sparse, const StageArgs<T>& a, dim3 grid,
                                 hipStream_t s) {
    if (eos == EOS_CONFORMAL) {
        if constexpr (sizeof(T) == 4 && ORDER == 7) {
            // the other instances gain too little there for a second one
            if (sparse && !hub && !local) {
                stage_fused<T, ORDER, TX, false, false, EOS_CONFORMAL, true><<<grid, 256, 0, s>>>(a);
                return hipSuccess;
            }
        }
        if (hub && local) stage_fused<T, ORDER, TX, true, true, EOS_CONFORMAL><<<grid, 256, 0, s>>>(a);
        else if (hub) stage_fused<T, ORDER, TX, true, false, EOS_CONFORMAL><<<grid, 256, 0, s>>>(a);
        else if (local) stage_fused<T, ORDER, TX, false, true, EOS_CONFORMAL><<<grid, 256, 0, s>>>(a);
        else stage_fused<T, ORDER, TX, false, false, EOS_CONFORMAL><<<grid, 256, 0, s>>>(a);
    } else if (eos == EOS_IDEAL && !hub) {
        // analytic boundaries are the conformal fluid's
        if (local) stage_fused<T, ORDER, TX, false, true, EOS_IDEAL><<<grid, 256, 0, s>>>(a);
        else stage_fused<T, ORDER, TX, false, false, EOS_IDEAL><<<grid, 256, 0, s>>>(a);
    } else {
        return hipErrorInvalidValue;
    }
    return hipSuccess;
}

template <class T>
hipError_t launch_stage(int order, int tx, bool hub, bool local, int eos, bool sparse, const StageArgs<T>& a,
                        long long nblocks, hipStream_t s) {
    if (nblocks <= 0 || nblocks > 0x7fffffffLL) return hipErrorInvalidValue;
    const dim3 grid((unsigned)nblocks);
    hipError_t e;
    if (order == 5) {
        if (tx == 16) e = launch_stage_t<T, 5, 16>(hub, local, eos, sparse, a, grid, s);
        else if (tx == 32) e = launch_stage_t<T, 5, 32>(hub, local, eos, sparse, a, grid, s);
        else return hipErrorInvalidValue;
    } else if (order == 7) {
        // WENO7 tiles are 16 x 16 (a 32 x 8 tile has 320 halo cells per plane)
        if (tx == 16) e = launch_stage_t<T, 7, 16>(hub, local, eos, sparse, a, grid, s);
        else return hipErrorInvalidValue;
    } else {
        return hipErrorInvalidValue;
    }
    return e != hipSuccess ? e : hipGetLastError();
}

template void stage_shape<float>(StageGrid<float>&, int, int);
template void stage_shape<double>(StageGrid<double>&, int, int);
template hipError_t launch_stage<float>(int, int, bool, bool, int, bool, const StageArgs<float>&, long long, hipStream_t);
template hipError_t launch_stage<double>(int, int, bool, bool, int, bool, const StageArgs<double>&, long long, hipStream_t);

}  // namespace rh
