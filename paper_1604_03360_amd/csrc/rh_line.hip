// rh_line.hip -- several SSP-RK3 steps of a one-dimensional grid per launch for
// gfx950.
//
// A line of a few hundred cells (the shock tube of Sikorski et al.,
// arXiv:1604.03360, Sec. 3) is far too little work for a launch per stage: 400
// cells took 5.8 us per stage, all of it launch and dependent latency.  Here a
// block takes a tile of the line with `halo` cells of its neighbours' on each side
// and advances it `steps` whole steps in LDS and registers; every stage makes
// G more cells at each end stale (G ghost cells per side of the scheme), which
// is what the halo is for.  A line that fits one block needs no halo and stays
// there for all its steps.
//
// One lane holds one cell (ghost cells included: they evolve as copies of the
// cell they repeat) with its state and u^n in registers.  Per stage it recovers
// its primitives and puts its split fluxes in LDS; then the lanes of the block
// take the reconstructions one each -- (face, component, sign) -- so a 104-cell
// window is one round of 1024 lanes; then each lane forms its flux difference and
// the stage combine.  Two barriers per stage.  What bounds it is the chain
// recovery -> reconstruction -> combine of dependent FP64 operations.
//
// The arithmetic of every recovery, face and combine is that of the other paths,
// in the same order, so the results are bitwise theirs.
#include "rh_face.hpp"
#include "rh_internal.hpp"
#include "../../include/rh.h"

namespace rh {

namespace {

// LDS words of a window of q cells: the split fluxes (or the state for
// MUSTA-FORCE), the speeds of local splitting and the face fluxes.
constexpr int line_words(int q) { return 21 * q; }

}  // namespace

template <class T, int SCHEME, bool LOCAL, int EOS>
__global__ void __launch_bounds__(1024) line_steps(LineArgs<T> A) {
    constexpr bool MUSTA = SCHEME == RH_SCHEME_MUSTA;
    constexpr int G = MUSTA ? 2 : (SCHEME + 1) / 2;
    constexpr int W = 2 * G;
    extern __shared__ char line_lds[];
    const int n = A.n, dir = A.dir;
    const bool periodic = A.bc == RH_BC_PERIODIC, single = gridDim.x == 1;
    const int x0 = (int)blockIdx.x * A.tile, x1 = min(n, x0 + A.tile);
    // window of the block: the ghost cells of the line where it reaches them
    // (one block, or the ends of an outflow line), the neighbours' cells elsewhere
    int wl = x0 - A.halo, wh = x1 + A.halo;
    if (single) {
        wl = -G;
        wh = n + G;
    } else if (!periodic) {
        wl = max(wl, -G);
        wh = min(wh, n + G);
    }
    const int Q = wh - wl, nf = Q - W + 1;
    T* sa = (T*)line_lds;        // [5][Q]: plus fluxes (F with LOCAL, the state with MUSTA)
    T* sb = sa + 5 * Q;          // [5][Q]: minus fluxes (u with LOCAL)
    T* ss = sb + 5 * Q;          // [Q]: largest speeds (LOCAL)
    T* sf = ss + Q;              // [10][nf]: reconstructions, or [5][nf] face fluxes

    const int tid = threadIdx.x;
    const bool cell = tid < Q;
    const int g = wl + tid;
    int at = g;                  // the cell of the line this lane's cell is or repeats
    if (periodic) {
        at %= n;
        if (at < 0) at += n;
    } else {
        at = min(max(at, 0), n - 1);
    }
    // slot whose faces advance this lane's cell; cells without both faces go stale
    const int sq = (single || !periodic ? at : g) - wl;
    const bool moves = cell && sq >= G && sq + G < Q;
    const bool owned = cell && g >= x0 && g < x1;
    const T eps2 = (T)4 * A.eps;   // the split fluxes are doubled
    const T hinv = MUSTA ? A.inv_h : (T)0.5 * A.inv_h;
    unsigned clamped = 0;

    T us[5] = {(T)0, (T)0, (T)0, (T)0, (T)0}, un[5];
    if (cell) {
#pragma unroll
        for (int c = 0; c < 5; ++c) us[c] = A.in[(long long)c * n + at];
    }
    // this lane's first reconstruction of a stage (most windows have no second)
    const int j0c = tid / nf, j0f = tid - j0c * nf;
    for (int step = 0; step < A.steps; ++step) {
#pragma unroll
        for (int c = 0; c < 5; ++c) un[c] = us[c];
#pragma unroll 1
        for (int stage = STAGE_1; stage <= STAGE_3; ++stage) {
            if (cell) {
                if constexpr (MUSTA) {
#pragma unroll
                    for (int c = 0; c < 5; ++c) sa[c * Q + tid] = us[c];
                } else {
                    T q[3], P;
                    double v2 = 0.0, cs2 = 0.0, vd;
                    unsigned cl = 0;
                    double kap, Mxs, Mys, Mzs, p;
                    if constexpr (EOS == EOS_IDEAL) {
                        double e;
                        recover_ideal((double)us[0], (double)us[1], (double)us[2], (double)us[3], (double)us[4], A.gm1,
                                      kap, Mxs, Mys, Mzs, p, e, cl);
                        q[0] = (T)(kap * Mxs);
                        q[1] = (T)(kap * Mys);
                        q[2] = (T)(kap * Mzs);
                        // as read back from the recovery pass, in the plan precision
                        const double a = (double)q[0], b = (double)q[1], c = (double)q[2];
                        vd = dir == 0 ? a : (dir == 1 ? b : c);
                        v2 = a * a + b * b + c * c;
                        cs2 = (double)(T)(e + p > 0.0 ? (A.gm1 + 1.0) * p / (e + p) : 0.0);
                    } else {
                        recover_kp3((double)us[0], (double)us[1], (double)us[2], (double)us[3], kap, Mxs, Mys, Mzs, p,
                                    cl);
                        vd = kap * (dir == 0 ? Mxs : (dir == 1 ? Mys : Mzs));
                        v2 = kap * kap * (Mxs * Mxs + Mys * Mys + Mzs * Mzs);
                        cs2 = 1.0 / 3.0;
                    }
                    P = (T)p;
                    if (owned) clamped += cl;   // once per cell and evaluation of L
                    const T v = (T)vd;
                    T f[5];
                    f[0] = dir == 0 ? us[1] : (dir == 1 ? us[2] : us[3]);
                    f[1] = us[1] * v + (dir == 0 ? P : (T)0);
                    f[2] = us[2] * v + (dir == 1 ? P : (T)0);
                    f[3] = us[3] * v + (dir == 2 ? P : (T)0);
                    f[4] = us[4] * v;
#pragma unroll
                    for (int c = 0; c < 5; ++c) {
                        sa[c * Q + tid] = LOCAL ? f[c] : f[c] + us[c];
                        sb[c * Q + tid] = LOCAL ? us[c] : f[c] - us[c];
                    }
                    if constexpr (LOCAL) ss[tid] = (T)max_char_speed(vd, v2, cs2);
                }
            }
            __syncthreads();
            // face f lies right of slot f + G - 1; its stencil is slots f .. f + 2G - 1
            if constexpr (MUSTA) {
                const MustaFace<T> mf = {A.lam, A.gm1, A.limiter, A.mk};
                for (int f = tid; f < nf; f += 1024) {
                    T a[5], b[5], c2[5], d[5], F[5];
#pragma unroll
                    for (int c = 0; c < 5; ++c) {
                        a[c] = sa[c * Q + f];
                        b[c] = sa[c * Q + f + 1];
                        c2[c] = sa[c * Q + f + 2];
                        d[c] = sa[c * Q + f + 3];
                    }
                    unsigned cl = 0;
                    musta_face<T, kAnyAxis, EOS, kAnyLimiter, kAnyStages>(a, b, c2, d, mf, F, cl, dir);
                    const int left = wl + f + G - 1;   // every face of the line counted once
                    if ((left >= x0 && left < x1) || (left == -1 && x0 == 0)) clamped += cl;
#pragma unroll
                    for (int c = 0; c < 5; ++c) sf[c * nf + f] = F[c];
                }
            } else if constexpr (LOCAL) {
                for (int j = tid, c = j0c, f = j0f; j < 5 * nf; j += 1024, c = j / nf, f = j - c * nf) {
                    T wa[W], wb[W], al = (T)0;
#pragma unroll
                    for (int k = 0; k < W; ++k) {
                        wa[k] = sa[c * Q + f + k];
                        wb[k] = sb[c * Q + f + k];
                        al = max(al, ss[f + k]);
                    }
                    sf[j] = recon_local<T, SCHEME>(wa, wb, al, eps2);
                }
            } else {
                for (int j = tid, cs = j0c, f = j0f; j < 10 * nf; j += 1024, cs = j / nf, f = j - cs * nf) {
                    const int c = cs >> 1;
                    // plus: slots f .. ascending; minus: slots f + 2G - 1 .. descending
                    const T* w = (cs & 1) ? sb + c * Q + f + W - 1 : sa + c * Q + f;
                    const int d = (cs & 1) ? -1 : 1;
                    T s[W];
#pragma unroll
                    for (int k = 0; k < W - 1; ++k) s[k] = w[k * d];
                    sf[j] = stage_recon_plus<T, SCHEME>(s, eps2);
                }
            }
            __syncthreads();
            if (moves) {
                const int fr = sq - G + 1, fl = fr - 1;   // faces right and left of the cell
#pragma unroll
                for (int c = 0; c < 5; ++c) {
                    T Fl, Fr;
                    if constexpr (MUSTA || LOCAL) {
                        Fl = sf[c * nf + fl];
                        Fr = sf[c * nf + fr];
                    } else {
                        Fl = sf[2 * c * nf + fl] + sf[(2 * c + 1) * nf + fl];
                        Fr = sf[2 * c * nf + fr] + sf[(2 * c + 1) * nf + fr];
                    }
                    const T L = (Fl - Fr) * hinv;
                    T v = us[c] + A.dt * L;
                    if (stage == STAGE_2) v = (T)0.75 * un[c] + (T)0.25 * v;
                    else if (stage == STAGE_3) v = rk3_last(un[c], v);
                    us[c] = v;
                }
            }
        }
    }
    if (owned) {
#pragma unroll
        for (int c = 0; c < 5; ++c) A.out[(long long)c * n + g] = us[c];
    }
    if (clamped) atomicAdd(A.clamps, clamped);
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
// Tile and steps per launch of a line of several blocks.  The window is the tile
// and 2 * 3 G cells of halo per step; the fewer its reconstructions, the fewer waves share the
// SIMDs, the more steps, the fewer launches.  us per step at 400 cells (17.2 with a
// launch per stage): FP64 WENO5 4.25 with tiles of 16 and three steps, 4.56 with 32 and
// four, 5.17 with 32 and eight; FP32 3.99, 3.89, 4.23; WENO7 5.2 either way.  Tiles of
// 16 need 256 CUs for 4096 cells (8000 cells: 8.1 us against 4.7).  A line of up to
// kLineSingle cells stays in one block, for at most kLineMaxSteps steps, so that a
// launch ends within a millisecond or so.
static int line_ghosts(int scheme) { return scheme == RH_SCHEME_MUSTA ? 2 : (scheme + 1) / 2; }
static int line_tile(int elem, int n) { return elem == 8 && n <= 4096 ? 16 : 32; }

int line_max_steps(int scheme, int elem, int n) {
    if (n <= kLineSingle) return kLineMaxSteps;
    return scheme == 7 || line_tile(elem, n) == 16 ? 3 : 4;
}

template <class T, int SCHEME, bool LOCAL, int EOS>
static hipError_t launch_line_t(const LineArgs<T>& a, unsigned blocks, size_t lds, hipStream_t s) {
    line_steps<T, SCHEME, LOCAL, EOS><<<dim3(blocks), dim3(1024), lds, s>>>(a);
    return hipGetLastError();
}

template <class T>
hipError_t launch_line(int scheme, bool local, int eos, LineArgs<T> a, hipStream_t s) {
    const int G = line_ghosts(scheme);
    if (a.n < 2 || a.n > kLineMaxCells || a.steps < 1 || a.steps > line_max_steps(scheme, (int)sizeof(T), a.n) || a.dir < 0 || a.dir > 2 ||
        (a.bc != RH_BC_PERIODIC && a.bc != RH_BC_OUTFLOW) || (eos != EOS_CONFORMAL && eos != EOS_IDEAL) ||
        (scheme != 5 && scheme != 7 && scheme != RH_SCHEME_MUSTA))
        return hipErrorInvalidValue;
    const bool single = a.n <= kLineSingle;
    if (!single && a.in == a.out) return hipErrorInvalidValue;   // blocks read their neighbours' cells
    a.tile = single ? a.n : line_tile((int)sizeof(T), a.n);
    a.halo = single ? 0 : 3 * G * a.steps;
    const int q = single ? a.n + 2 * G : a.tile + 2 * a.halo;
    if (q > 1024) return hipErrorInvalidValue;
    const unsigned blocks = (unsigned)((a.n + a.tile - 1) / a.tile);
    const size_t lds = sizeof(T) * (size_t)line_words(q);
    if (scheme == RH_SCHEME_MUSTA) {
        return eos == EOS_IDEAL ? launch_line_t<T, RH_SCHEME_MUSTA, false, EOS_IDEAL>(a, blocks, lds, s)
                                : launch_line_t<T, RH_SCHEME_MUSTA, false, EOS_CONFORMAL>(a, blocks, lds, s);
    }
    if (scheme == 5) {
        if (eos == EOS_IDEAL) return local ? launch_line_t<T, 5, true, EOS_IDEAL>(a, blocks, lds, s)
                                           : launch_line_t<T, 5, false, EOS_IDEAL>(a, blocks, lds, s);
        return local ? launch_line_t<T, 5, true, EOS_CONFORMAL>(a, blocks, lds, s)
                     : launch_line_t<T, 5, false, EOS_CONFORMAL>(a, blocks, lds, s);
    }
    if (eos == EOS_IDEAL) return local ? launch_line_t<T, 7, true, EOS_IDEAL>(a, blocks, lds, s)
                                       : launch_line_t<T, 7, false, EOS_IDEAL>(a, blocks, lds, s);
    return local ? launch_line_t<T, 7, true, EOS_CONFORMAL>(a, blocks, lds, s)
                 : launch_line_t<T, 7, false, EOS_CONFORMAL>(a, blocks, lds, s);
}

template hipError_t launch_line<float>(int, bool, int, LineArgs<float>, hipStream_t);
template hipError_t launch_line<double>(int, bool, int, LineArgs<double>, hipStream_t);

}  // namespace rh
