"""The directional sweeps by themselves (RH_PATH_SWEEPS; the default path takes them for
some grids only): the fused x-y sweep and the separate ones against the FP64 oracle
(1e-12, FP32 2e-5), over every row length, boundary kind along y and z and a single z
plane (the fused launch then applies the stage combine); graph replays; bitwise
equality of the fused and the separate sweeps; and states that hold floored cells."""
import os
import subprocess
import sys

import numpy as np
import pytest

import oracle
from paper_1604_03360_amd import inputs
from gpu_helpers import L_errors, assert_fields_close, field_errors, oracle_steps, rh_module
from test_gpu_floors import CASES as FLOOR_CASES, FP32_TOL, FP64_TOL, planted_state

pytestmark = pytest.mark.gpu

P, O, H = inputs.BC_PERIODIC, inputs.BC_OUTFLOW, inputs.BC_HUBBLE


def hubble_periodic_x(shape, o):
    spec = inputs.hubble(order=o, half_width=3.0, shape=shape)
    spec["bc"] = (P, H, H)
    return spec


CASES = {
    "rows_64_outflow_yz": lambda o: inputs.random_smooth((64, 27, 13), h=0.1, seed=81, bc=(P, O, O), order=o),
    "rows_128_one_z_plane": lambda o: inputs.random_smooth((128, 20, 1), h=0.1, seed=82, order=o),
    "rows_192": lambda o: inputs.random_smooth((192, 17, 5), h=0.05, seed=83, bc=(P, P, O), order=o),
    "rows_64_hubble_yz": lambda o: hubble_periodic_x((64, 20, 18), o),
    "rows_256": lambda o: inputs.random_smooth((256, 9, 3), h=0.05, seed=84, order=o),
    "rows_256_outflow_yz": lambda o: inputs.random_smooth((256, 13, 9), h=0.1, seed=86, bc=(P, O, O), order=o),
    "rows_256_one_z_plane": lambda o: inputs.random_smooth((256, 20, 1), h=0.1, seed=87, order=o),
    "rows_256_hubble_yz": lambda o: hubble_periodic_x((256, 18, 11), o),
    "ragged_outflow": lambda o: inputs.random_smooth((70, 37, 23), h=0.1, seed=88, bc=(O, O, O), order=o),
}
KINDS = [("fp64", 1e-12, 5), ("fp64", 1e-12, 7), ("fp32", 2e-5, 5), ("fp32", 2e-5, 7)]


def sweeps(rh, spec, precision):
    h = rh.Hydro.from_spec(spec, precision=rh.RH_PREC_FP64 if precision == "fp64" else rh.RH_PREC_FP32)
    rh.rh_set_path(h.plan, rh.RH_PATH_SWEEPS)
    h.set_primitive(spec["prim"])
    return h


def fused(spec, precision, order):
    nx = spec["shape"][0]
    return spec["bc"][0] == P and nx <= 256 and nx % (64 if (precision, order) == ("fp32", 5) else 256) == 0


@pytest.mark.parametrize("precision,tol,order", KINDS)
@pytest.mark.parametrize("case", sorted(CASES))
def test_sweeps_match_oracle(case, precision, tol, order):
    rh = rh_module()
    spec = CASES[case](order)
    h = sweeps(rh, spec, precision)
    rh.rh_set_timing(h.plan, True)
    t = h.step(spec["dt"], 3)
    got = h.get()
    launches = {k: v[1] for k, v in rh.rh_kernel_times(h.plan).items()}
    cnt = h.totals()[1]
    h.close()
    xy = 9 if fused(spec, precision, order) else 0
    assert [launches[k] for k in ("sweep_xy", "sweep_x", "sweep_y", "stage")] == [xy, 9 - xy, 9 - xy, 0]
    ref, tr = oracle_steps(spec, 3)
    assert t == pytest.approx(tr, abs=1e-12)
    print(case, precision, order, field_errors(got, ref), flush=True)
    assert_fields_close(got, ref, tol, "%s %s WENO%d" % (case, precision, order))
    assert cnt[1] == 0


@pytest.mark.parametrize("precision,tol,order", KINDS)
def test_fused_sweep_graph_replay_matches_eager(precision, tol, order):
    import torch
    rh = rh_module()
    spec = CASES["rows_256_outflow_yz"](order)
    dt = spec["dt"]
    eager, graphed = sweeps(rh, spec, precision), sweeps(rh, spec, precision)
    rh.rh_set_graph(graphed.plan, True)
    for _ in range(3):
        eager.step(dt, 2)
        graphed.step(dt, 2)
        torch.randn(1 << 18, device="cuda").mul_(3.0).sum().item()
        torch.cuda.synchronize()
        assert np.array_equal(graphed.get(), eager.get())
    eager.close()
    graphed.close()


BITWISE = [((256, 27, 11), (P, O, P)), ((128, 27, 11), (P, O, P)), ((256, 19, 1), (P, P, P))]
SPLIT_SCRIPT = r"""
import sys, numpy as np
sys.path.insert(0, sys.argv[1]); sys.path.insert(0, sys.argv[1] + "/tests")
from gpu_helpers import rh_module
from test_gpu_sweeps_explicit import bitwise_runs
for name, got in bitwise_runs(rh_module()):
    np.save(sys.argv[2] + name + ".npy", got)
"""


def bitwise_runs(rh):
    for k, (shape, bc) in enumerate(BITWISE):
        for precision, _, order in KINDS:
            spec = inputs.random_smooth(shape, h=0.1, seed=85, bc=bc, order=order)
            h = sweeps(rh, spec, precision)
            h.step(spec["dt"], 3)
            yield "%d_%s_%d" % (k, precision, order), h.get()
            h.close()


def test_fused_sweep_is_bitwise_the_separate_sweeps(tmp_path):
    """The separate sweeps are forced in a child process with RH_FUSE_XY=0."""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    out = str(tmp_path) + "/split_"
    r = subprocess.run([sys.executable, "-c", SPLIT_SCRIPT, root, out], env=dict(os.environ, RH_FUSE_XY="0"),
                       capture_output=True, text=True, timeout=240)
    assert r.returncode == 0, r.stderr[-2000:]
    for name, got in bitwise_runs(rh_module()):
        split = np.load(out + name + ".npy")
        assert np.array_equal(got, split), (name, np.abs(got - split).max())


FLOORS = dict(FLOOR_CASES, rows_256=lambda o: inputs.random_smooth((256, 12, 10), h=0.1, seed=94, bc=(P, O, P), order=o))


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("order", [5, 7])
@pytest.mark.parametrize("case", sorted(FLOORS))
def test_sweeps_with_floors_match_oracle(case, order, precision):
    """L and one step of planted states, and the floors counted once per cell and evaluation."""
    rh = rh_module()
    tol = FP64_TOL if precision == "fp64" else FP32_TOL
    spec = FLOORS[case](order)
    u, planted = planted_state(spec, 15)
    if precision == "fp32":
        u = u.astype(np.float32).astype(np.float64)
    h = sweeps(rh, spec, precision)
    h.set_conserved(u)
    rh.rh_reset_counters(h.plan)
    L = h.apply_L().double().cpu().numpy()
    cnt = h.totals()[1]
    h.step(spec["dt"], 1)
    got = h.get()
    h.close()
    g = oracle.grid_from_spec(spec)
    assert np.all(np.isfinite(L)) and np.all(np.isfinite(got))
    err = L_errors(L, oracle.apply_L(g, u), u, min(spec["h"]))
    assert np.all(err <= tol), err
    assert cnt[0] == len(planted)
    err = field_errors(got, oracle.step(g, u, spec["dt"], 1)[0])
    assert np.all(err <= tol), err
