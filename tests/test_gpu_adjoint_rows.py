"""The whole-row x adjoint (periodic x rows of 32, 64, 96, 128, 192 or 256
cells) against the FP64 oracle's adjoint: FP64 (1e-12) and FP32 (5e-5), WENO5
and WENO7, row counts that leave part of the last block empty, non-periodic and
analytic y/z boundaries; the adjoint of a step; and bitwise equality with the
tiled x adjoint (forced in a child process with RH_ADJ_XROW=0)."""
import numpy as np
import pytest

import oracle
from paper_1604_03360_amd import inputs
from gpu_helpers import rh_module

pytestmark = pytest.mark.gpu

P, O, H = inputs.BC_PERIODIC, inputs.BC_OUTFLOW, inputs.BC_HUBBLE


def hubble_periodic_x(o):
    spec = inputs.hubble(n=32, order=o, half_width=3.0)
    spec["bc"] = (P, H, H)
    return spec


CASES = {
    # 15 rows: the second block of eight rows holds one empty row
    "rows_32_hubble_yz": hubble_periodic_x,
    "rows_64_outflow_yz": lambda o: inputs.random_smooth((64, 7, 3), h=0.1, seed=91, bc=(P, O, O), order=o),
    "rows_96": lambda o: inputs.random_smooth((96, 5, 3), h=0.1, seed=92, order=o),
    "rows_128_outflow_z": lambda o: inputs.random_smooth((128, 3, 3), h=0.05, seed=93, bc=(P, P, O), order=o),
    "rows_192_one_row": lambda o: inputs.random_smooth((192, 1, 1), h=0.05, seed=94, order=o),
    "rows_256": lambda o: inputs.random_smooth((256, 3, 2), h=0.05, seed=95, order=o),
}


def vjp_errors(got, ref, w, h):
    """Per-field max|got - ref| normalised by max(max|ref|, max|w|/h)."""
    got = np.asarray(got, np.float64).reshape(5, -1)
    ref = np.asarray(ref, np.float64).reshape(5, -1)
    scale = max(np.abs(ref).max(), np.abs(w).max() / h)
    return np.abs(got - ref).max(axis=1) / scale


def _setup(rh, spec, prec, seed=7):
    h = rh.Hydro.from_spec(spec, precision=prec)
    u = oracle.prim2con(spec["prim"])
    w = np.random.default_rng(seed).normal(size=u.shape)
    return h, u, w


@pytest.mark.parametrize("order", [5, 7])
@pytest.mark.parametrize("case", sorted(CASES))
def test_row_vjp_fp64_matches_oracle(case, order):
    rh = rh_module()
    spec = CASES[case](order)
    assert spec["bc"][0] == P
    h, u, w = _setup(rh, spec, rh.RH_PREC_FP64)
    t = spec["t0"] + 0.2
    got = h.vjp(u, w, t=t).cpu().numpy()
    h.close()
    ref = oracle.vjp_L(oracle.grid_from_spec(spec), u, w, t=t)
    err = vjp_errors(got, ref, w, min(spec["h"]))
    print(case, order, err, flush=True)
    assert np.all(err <= 1e-12), err


@pytest.mark.parametrize("order", [5, 7])
@pytest.mark.parametrize("case", sorted(CASES))
def test_row_vjp_fp32_close_to_oracle(case, order):
    rh = rh_module()
    spec = CASES[case](order)
    h, u, w = _setup(rh, spec, rh.RH_PREC_FP32)
    t = spec["t0"] + 0.2
    got = h.vjp(u, w, t=t).double().cpu().numpy()
    h.close()
    u32 = u.astype(np.float32).astype(np.float64)
    w32 = w.astype(np.float32).astype(np.float64)
    ref = oracle.vjp_L(oracle.grid_from_spec(spec), u32, w32, t=t)
    err = vjp_errors(got, ref, w32, min(spec["h"]))
    print(case, order, "fp32", err, flush=True)
    assert np.all(err <= 5e-5), err


@pytest.mark.parametrize("order", [5, 7])
def test_row_step_vjp_fp64_matches_oracle(order):
    rh = rh_module()
    spec = CASES["rows_64_outflow_yz"](order)
    h, u, w = _setup(rh, spec, rh.RH_PREC_FP64)
    dt, t = spec["dt"], spec["t0"]
    got = h.step_vjp(u, w, dt, t=t).cpu().numpy()
    h.close()
    ref = oracle.vjp_step(oracle.grid_from_spec(spec), u, w, dt, t=t)
    err = np.abs(got - ref).reshape(5, -1).max(axis=1) / np.abs(ref).max()
    print(order, err, flush=True)
    assert np.all(err <= 1e-12), err


TILED_SCRIPT = r"""
import sys, numpy as np
sys.path.insert(0, sys.argv[1]); sys.path.insert(0, sys.argv[1] + "/tests")
import oracle
from paper_1604_03360_amd import inputs
from gpu_helpers import rh_module
rh = rh_module()
for o in (5, 7):
    for shape in ((64, 11, 5), (96, 7, 3)):
        spec = inputs.random_smooth(shape, h=0.1, seed=96, bc=(0, 1, 0), order=o)
        u = oracle.prim2con(spec["prim"])
        w = np.random.default_rng(9).normal(size=u.shape)
        for name, prec in (("fp64", rh.RH_PREC_FP64), ("fp32", rh.RH_PREC_FP32)):
            h = rh.Hydro.from_spec(spec, precision=prec)
            got = h.vjp(u, w, t=0.1).cpu().numpy()
            h.close()
            np.save("%s_%s_%d_%d.npy" % (sys.argv[2], name, o, shape[0]), got)
"""


def test_row_vjp_is_bitwise_the_tiled_kernel(tmp_path):
    import os
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    out = str(tmp_path / "tiled")
    env = dict(os.environ, RH_ADJ_XROW="0")
    r = subprocess.run([sys.executable, "-c", TILED_SCRIPT, root, out], env=env, capture_output=True,
                       text=True, timeout=240)
    assert r.returncode == 0, r.stderr[-2000:]
    rh = rh_module()
    for o in (5, 7):
        for shape in ((64, 11, 5), (96, 7, 3)):
            spec = inputs.random_smooth(shape, h=0.1, seed=96, bc=(P, O, P), order=o)
            u = oracle.prim2con(spec["prim"])
            w = np.random.default_rng(9).normal(size=u.shape)
            for name, prec in (("fp64", rh.RH_PREC_FP64), ("fp32", rh.RH_PREC_FP32)):
                h = rh.Hydro.from_spec(spec, precision=prec)
                got = h.vjp(u, w, t=0.1).cpu().numpy()
                h.close()
                tiled = np.load("%s_%s_%d_%d.npy" % (out, name, o, shape[0]))
                assert np.array_equal(got, tiled), (name, o, shape, np.abs(got - tiled).max())


LARGE = {
    # around and above the sizes from which y and z roll instead of taking tiles; ragged axes
    "periodic": lambda o: inputs.random_smooth((76, 75, 71), h=0.1, seed=301, order=o),
    "outflow": lambda o: inputs.random_smooth((61, 83, 81), h=0.1, seed=302, order=o, bc=(inputs.BC_OUTFLOW,) * 3),
    "hubble": lambda o: inputs.hubble(n=75, order=o, half_width=3.0),
    "periodic_600k": lambda o: inputs.random_smooth((86, 85, 83), h=0.1, seed=307, order=o),
    "outflow_600k": lambda o: inputs.random_smooth((71, 93, 92), h=0.1, seed=308, order=o, bc=(inputs.BC_OUTFLOW,) * 3),
    "hubble_600k": lambda o: inputs.hubble(n=85, order=o, half_width=3.0),
}
# below it: one short of, at and past a tile edge along every axis
SMALL = {
    "edge_15_16_17": lambda o: inputs.random_smooth((15, 16, 17), h=0.1, seed=303, order=o),
    "edge_33_31_32": lambda o: inputs.random_smooth((33, 31, 32), h=0.1, seed=304, order=o, bc=(inputs.BC_OUTFLOW,) * 3),
    "two_cells": lambda o: inputs.random_smooth((9, 2, 3), h=0.1, seed=305, order=o, bc=(inputs.BC_OUTFLOW,) * 3),
    "hubble": lambda o: inputs.hubble(n=18, order=o, half_width=3.0),
}


@pytest.mark.parametrize("order", [5, 7])
@pytest.mark.parametrize("case", sorted(LARGE) + sorted("small_" + k for k in SMALL))
def test_yz_adjoint_tiles_and_rolls_match_reference(case, order):
    """FP64 J^T w on both sides of the size at which the y and z adjoint change
    kernel, to the 1e-12 of the other adjoint tests.
    The reference is the gradient of the plain 64-bit right-hand side of the
    measured workloads (the oracle's own WENO7 adjoint is 3e-12 from it at the
    edge of the ragged outflow grid, the library 3e-13)."""
    import importlib.util
    import os

    import torch
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    mod = importlib.util.spec_from_file_location("measured_cases", os.path.join(root, "perf", "cases.py"))
    cases = importlib.util.module_from_spec(mod)
    rh = rh_module()
    mod.loader.exec_module(cases)
    spec = (SMALL[case[6:]] if case.startswith("small_") else LARGE[case])(order)
    u = oracle.prim2con(spec["prim"])
    w = np.random.default_rng(9).normal(size=u.shape)
    t = spec["t0"] + 0.1
    h = rh.Hydro.from_spec(spec, precision=rh.RH_PREC_FP64)
    got = h.vjp(u, w, t=t).cpu().numpy()
    h.close()
    ut = torch.tensor(u, device="cuda", requires_grad=True)
    L = cases._rhs(ut, dict(spec, lf_local=False, eos=0), t)
    ref = torch.autograd.grad(L, ut, torch.tensor(w, device="cuda"))[0].cpu().numpy()
    err = np.abs(got - ref).reshape(5, -1).max(axis=1) / max(np.abs(ref).max(), np.abs(w).max() / min(spec["h"]))
    assert np.all(err <= 1e-12), err


@pytest.mark.parametrize("order", [5, 7])
@pytest.mark.parametrize("prec", ["RH_PREC_FP64", "RH_PREC_FP32"])
@pytest.mark.parametrize("bc", [P, O])
def test_long_x_adjoint_repeats_the_short_one(bc, prec, order):
    """A line of 401 000 cells that repeats one of 802: the x adjoint of large
    grids gives the bits of the small grids' at every cell whose stencils see the
    same data (all of them when periodic; up to 401 cells from either outflow end)."""
    rh = rh_module()
    spec = inputs.random_smooth((401, 1, 1), h=0.1, seed=306, order=order, bc=(bc, P, P))
    w1 = np.random.default_rng(10).normal(size=(5, 1, 1, 401))

    def vjp(copies):
        s = dict(spec, shape=(401 * copies, 1, 1), prim=np.concatenate([spec["prim"]] * copies, axis=-1))
        h = rh.Hydro.from_spec(s, precision=getattr(rh, prec))
        got = h.vjp(oracle.prim2con(s["prim"]), np.concatenate([w1] * copies, axis=-1), t=0.1).cpu().numpy()
        h.close()
        return got.reshape(5, -1)

    short, long = vjp(2), vjp(1000)
    assert np.array_equal(long[:, :401], short[:, :401])
    assert np.array_equal(long[:, -401:], short[:, -401:])
    if bc == P:
        assert np.array_equal(long, np.concatenate([short] * 500, axis=1))
