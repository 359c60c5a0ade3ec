"""The default evaluation path of single grids: whatever it picks for a grid, the
result is bitwise that of the directional sweeps, over tile and segment edges,
every boundary kind, both orders and both precisions, and the sweeps hold to the
oracle (FP64 1e-12, FP32 2e-5 after three steps, as in the other parity files)."""
import numpy as np
import pytest

from paper_1604_03360_amd import inputs
from gpu_helpers import assert_fields_close, oracle_steps, rh_module

pytestmark = pytest.mark.gpu

P, O, H = inputs.BC_PERIODIC, inputs.BC_OUTFLOW, inputs.BC_HUBBLE

CASES = {
    # one below, at and above a tile edge; axes shorter than the stencil; one long axis
    "edge_15_16_17": lambda o: inputs.random_smooth((15, 16, 17), h=0.1, seed=201, order=o),
    "edge_33_17_5": lambda o: inputs.random_smooth((33, 17, 5), h=0.1, seed=202, bc=(O, P, O), order=o),
    "short": lambda o: inputs.random_smooth((2, 3, 4), h=0.1, seed=203, bc=(P, O, P), order=o),
    "long_z": lambda o: inputs.random_smooth((7, 5, 90), h=0.1, seed=204, bc=(O, O, P), order=o),
    # whole periodic rows: the sweeps fuse x and y
    "rows_256": lambda o: inputs.random_smooth((256, 11, 9), h=0.05, seed=205, bc=(P, O, P), order=o),
    "rows_128": lambda o: inputs.random_smooth((128, 21, 6), h=0.05, seed=206, order=o),
    "hubble": lambda o: inputs.hubble(n=20, order=o, half_width=3.0),
}


@pytest.mark.parametrize("precision,tol", [("fp64", 1e-12), ("fp32", 2e-5)])
@pytest.mark.parametrize("order", [5, 7])
@pytest.mark.parametrize("case", sorted(CASES))
def test_default_path_is_bitwise_the_sweeps(case, order, precision, tol):
    rh = rh_module()
    spec = CASES[case](order)
    prec = rh.RH_PREC_FP64 if precision == "fp64" else rh.RH_PREC_FP32
    out = {}
    for path in (rh.RH_PATH_AUTO, rh.RH_PATH_SWEEPS):
        h = rh.Hydro.from_spec(spec, precision=prec)
        rh.rh_set_path(h.plan, path)
        h.set_primitive(spec["prim"])
        h.step(spec["dt"], 3)
        out[path] = h.get()
        h.close()
    assert np.array_equal(out[rh.RH_PATH_AUTO], out[rh.RH_PATH_SWEEPS])
    ref, _ = oracle_steps(spec, 3)
    assert_fields_close(out[rh.RH_PATH_SWEEPS], ref, tol, "%s %s WENO%d" % (case, precision, order))


def test_timing_keeps_the_sweeps():
    """While per-launch timing is on, the default path reports the directional sweeps."""
    rh = rh_module()
    spec = CASES["edge_15_16_17"](5)
    h = rh.Hydro.from_spec(spec, precision=rh.RH_PREC_FP32)
    h.set_primitive(spec["prim"])
    assert rh.rh_get_path(h.plan) == rh.RH_PATH_STAGE
    rh.rh_set_timing(h.plan, True)
    assert rh.rh_get_path(h.plan) == rh.RH_PATH_SWEEPS
    h.step(spec["dt"], 1)
    times = rh.rh_kernel_times(h.plan)
    assert [times[k][1] for k in ("sweep_x", "sweep_y", "sweep_z", "stage")] == [3, 3, 3, 0]
    rh.rh_set_timing(h.plan, False)
    assert rh.rh_get_path(h.plan) == rh.RH_PATH_STAGE
    h.close()
