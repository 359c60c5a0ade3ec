"""Steps of one-dimensional grids: the line kernel (several steps per launch) must
give bitwise what a launch per stage gives, and count the same floors, over lines
that fit one block or not, tile remainders, step counts that leave odd numbers of
launches, every axis, both boundary kinds and every scheme."""
import numpy as np
import pytest

from paper_1604_03360_amd import inputs
from gpu_helpers import rh_module

pytestmark = pytest.mark.gpu

P, O = inputs.BC_PERIODIC, inputs.BC_OUTFLOW
SCHEMES = {
    "weno5": (5, {}), "weno7": (7, {}), "musta": (2, {}), "musta_mc_3": (2, {"limiter": 1, "musta_k": 3}),
    "local5": (5, {"lf_local": True}), "local7": (7, {"lf_local": True}),
    "ideal5": (5, {"eos": 1, "gamma": 5.0 / 3.0}), "ideal_local7": (7, {"eos": 1, "gamma": 1.4, "lf_local": True}),
    "ideal_musta": (2, {"eos": 1, "gamma": 5.0 / 3.0}),
}
# cells, axis, boundary, steps: around one block (96), around its tiles (16 and 32), short lines
LINES = [(2, 0, P, 3), (5, 1, O, 4), (31, 2, P, 7), (96, 0, O, 9), (97, 0, P, 1), (97, 1, O, 2), (129, 2, O, 5),
         (160, 0, P, 8), (400, 0, O, 13)]


def run(rh, spec, prec, path, steps, u=None):
    h = rh.Hydro.from_spec(spec, precision=prec)
    rh.rh_set_path(h.plan, path)
    h.set_primitive(spec["prim"])
    if u is not None:
        h.set_conserved(u)
    rh.rh_reset_counters(h.plan)
    h.step(spec["dt"], steps)
    out = h.get()
    counters = h.totals()[1]
    h.close()
    return out, counters


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("scheme", sorted(SCHEMES))
def test_line_steps_are_bitwise_the_stages(scheme, precision):
    rh = rh_module()
    prec = rh.RH_PREC_FP64 if precision == "fp64" else rh.RH_PREC_FP32
    order, opts = SCHEMES[scheme]
    for n, axis, bc, steps in LINES:
        shape = [1, 1, 1]
        shape[axis] = n
        spec = inputs.random_smooth(tuple(shape), h=0.05, seed=400 + n, bc=(bc,) * 3, order=order)
        if "eos" in opts:
            spec = inputs.hot_gas(spec)
        spec = inputs.with_scheme(spec, **opts)
        line, c0 = run(rh, spec, prec, rh.RH_PATH_AUTO, steps)
        ref, c1 = run(rh, spec, prec, rh.RH_PATH_STAGE, steps)
        assert np.array_equal(line, ref), (scheme, n, axis, bc, steps, np.abs(line - ref).max())
        assert c0 == c1


@pytest.mark.parametrize("scheme", ["weno5", "musta", "ideal5"])
@pytest.mark.parametrize("n", [64, 200])
def test_line_counts_floors_once(n, scheme):
    """Cells below the energy floor and beyond the velocity cap."""
    rh = rh_module()
    order, opts = SCHEMES[scheme]
    spec = inputs.with_scheme(inputs.random_smooth((n, 1, 1), h=0.05, seed=77, bc=(O,) * 3, order=order), **opts)
    h = rh.Hydro.from_spec(spec)
    h.set_primitive(spec["prim"])
    u = h.get()
    h.close()
    u[0, 0, 0, [0, 31, 33, n - 1]] = 1e-13
    u[1, 0, 0, 40] = 2.0 * u[0, 0, 0, 40]
    line, c0 = run(rh, spec, rh.RH_PREC_FP64, rh.RH_PATH_AUTO, 1, u)
    ref, c1 = run(rh, spec, rh.RH_PREC_FP64, rh.RH_PATH_STAGE, 1, u)
    assert c0 == c1 and c0[0] > 0
    assert np.array_equal(line, ref, equal_nan=True)


def test_line_repeated_and_split_runs_agree():
    """Graphs asked for, runs cut into pieces and one run give the same bits."""
    import torch
    rh = rh_module()
    spec = inputs.sod(nx=400)
    whole, _ = run(rh, spec, rh.RH_PREC_FP64, rh.RH_PATH_AUTO, 23)
    h = rh.Hydro.from_spec(spec)
    rh.rh_set_graph(h.plan, True)
    h.set_primitive(spec["prim"])
    for k in (1, 4, 2, 13, 3):
        h.step(spec["dt"], k)
        torch.randn(1 << 16, device="cuda").sum().item()
    assert np.array_equal(h.get(), whole)
    h.close()
