"""The analytic ghost cells (HUBBLE boundaries) by themselves.

A first-order MUSTA-FORCE plan of vacuum cells hands them out: with the local
Courant number lam = 2^-40 the flux between a ghost state u and a cell of zeros is
u / (4 lam) + F(u) / 2 (the FORCE flux of one stage; F is homogeneous of degree one),
so L in the cells beside the boundary is 2^38 u / dx up to a term of 2e-12 of it,
which is known far better than that, and one rounding."""
import numpy as np
import pytest

from gpu_helpers import rh_module

pytestmark = pytest.mark.gpu

N = 64
DX, DY = 0.125, 0.15625          # exact cell positions
C0 = (1.25, -4.6875, -4.0625)
T0, E0, N0 = 10.0, 1.7, 0.37


def boundary_L(t):
    """L (5, 2, N, N) of the vacuum cells beside the lower and the upper x boundary."""
    rh = rh_module()
    h = rh.Hydro((2, N, N), (DX, DY, DY), C0, scheme=rh.RH_SCHEME_MUSTA, precision=rh.RH_PREC_FP64,
                 bc=(rh.RH_BC_HUBBLE, rh.RH_BC_PERIODIC, rh.RH_BC_PERIODIC), hub=(T0, E0, N0),
                 limiter=rh.RH_LIMITER_NONE, musta_stages=1, musta_cfl=2.0 ** -40)
    L = h.apply_L(t).cpu().numpy()
    h.close()
    return np.moveaxis(L, 3, 1)     # [5][x][z][y]


def ghost_states(t):
    """The ghost states there, as the library evaluates them."""
    L = boundary_L(t).astype(np.longdouble)
    u, v, p = plain(t, np.longdouble)
    f = np.stack([u[1], u[1] * v[0] + p, u[2] * v[0], u[3] * v[0], u[4] * v[0]])
    # lower cell: the flux u/(4 lam) + F/2 enters; upper cell: F/2 - u/(4 lam) leaves
    half = np.stack([f[:, 0], -f[:, 1]], axis=1) / 2
    return (L * DX - half) * np.longdouble(2.0) ** -38


def plain(t, dtype):
    """The flow's formulas as they are written, in dtype: states (5, 2, z, y), velocity, pressure."""
    x = np.array([C0[0] - DX, C0[0] + 2 * DX], dtype)[:, None, None]
    y = (C0[1] + DY * np.arange(N)).astype(dtype)[None, None, :]
    z = (C0[2] + DY * np.arange(N)).astype(dtype)[None, :, None]
    t = dtype(t)
    one = np.ones((2, N, N), dtype)
    s = dtype(T0) / np.sqrt(t * t - (x * x + y * y + z * z))
    e, n = dtype(E0) * s * s * s * s, dtype(N0) * s * s * s
    v = np.stack([x / t * one, y / t * one, z / t * one])
    p = e / dtype(3)
    g2 = dtype(1) / (dtype(1) - (v[0] * v[0] + v[1] * v[1] + v[2] * v[2]))
    w = e + p
    return np.stack([w * g2 - p, w * g2 * v[0], w * g2 * v[1], w * g2 * v[2], n * np.sqrt(g2)]), v, p


@pytest.mark.parametrize("t", [10.3, 8.1, -10.3])
def test_ghosts_follow_the_formulas(t):
    """Also at t < 0, where the flow contracts and the charge is positive all the same.
    1e-14: about 30 roundings, most of them to a high power."""
    got, ref = ghost_states(t), plain(t, np.longdouble)[0]
    assert np.all(ref[4] > 0) and np.all(got[4] > 0)
    assert np.all(np.abs(got - ref) <= 1e-14 * np.abs(ref))


@pytest.mark.parametrize("t", [10.3, 8.1, -10.3])
def test_ghosts_are_as_accurate_as_the_formulas(t):
    """Their errors, rms and largest, are no larger than those of the formulas evaluated
    in double precision with correctly rounded roots and divisions."""
    ref = plain(t, np.longdouble)[0]
    scale = np.where(ref == 0, 1, np.abs(ref))
    got = np.abs(ghost_states(t) - ref) / scale
    bar = np.abs(plain(t, np.float64)[0] - ref) / scale
    rms = lambda e: np.sqrt((e * e).mean(axis=(1, 2, 3)))
    print(rms(got), rms(bar), got.max(axis=(1, 2, 3)), bar.max(axis=(1, 2, 3)), flush=True)
    assert np.all(rms(got) <= rms(bar))
    assert np.all(got.max(axis=(1, 2, 3)) <= bar.max(axis=(1, 2, 3)))


def test_ghosts_outside_the_light_cone_are_not_finite():
    assert not np.any(np.isfinite(boundary_L(1.0)))
