"""J(u)^T w of grids past the sizes at which the adjoint leaves the short tiles: FP32
(the rolling y and z sweeps of both orders with periodic, outflow and analytic ends,
the three tile widths of the FP32 WENO5 x sweep and its ghosts, whole rows), and planted
floors through the recovery pack.

FP32 references are the gradient of the plain 64-bit right-hand side at the FP32-rounded
inputs.  Their bar is 5e-5 as in the other adjoint tests, or four times what
that gradient itself moves by when u moves by half an FP32 ulp, where that is more
(outflow edges and WENO7), but never more than 2.5e-4."""
import numpy as np
import pytest

import oracle
from paper_1604_03360_amd import inputs
from gpu_helpers import rh_module
from test_gpu_adjoint_thin import measured_cases
from test_gpu_floors import FP32_ADJ_TOL, FP64_TOL, _rounding_sensitivity, planted_state

pytestmark = pytest.mark.gpu

P, O = inputs.BC_PERIODIC, inputs.BC_OUTFLOW
CASES = {
    "tiles_of_32": lambda: inputs.random_smooth((86, 70, 69), h=0.1, seed=751),
    "tiles_of_16_outflow": lambda: inputs.random_smooth((71, 78, 75), h=0.1, seed=752, bc=(O, O, O)),
    "tiles_of_64_outflow_xz": lambda: inputs.random_smooth((125, 58, 57), h=0.1, seed=753, bc=(O, P, O)),
    "tiles_of_16_hubble": lambda: inputs.hubble(n=75, half_width=3.0),
    "rows_of_128_outflow_yz": lambda: inputs.random_smooth((128, 58, 57), h=0.1, seed=754, bc=(P, O, O)),
    "weno7": lambda: inputs.random_smooth((104, 106, 105), h=0.1, seed=755, order=7),
    "weno7_outflow": lambda: inputs.random_smooth((107, 103, 101), h=0.1, seed=756, bc=(O, O, O), order=7),
    "weno7_hubble": lambda: inputs.hubble(n=104, half_width=3.0, order=7),
    "weno7_rows_of_128_outflow_yz": lambda: inputs.random_smooth((128, 96, 94), h=0.1, seed=757, bc=(P, O, O), order=7),
}


@pytest.mark.parametrize("case", sorted(CASES))
def test_fp32_vjp_of_large_grids(case):
    import torch
    rh = rh_module()
    cases = measured_cases()
    spec = CASES[case]()
    t = spec["t0"] + 0.1
    u = torch.tensor(oracle.prim2con(spec["prim"]), dtype=torch.float32, device="cuda")
    w = torch.tensor(np.random.default_rng(14).normal(size=u.shape), dtype=torch.float32, device="cuda")
    h = rh.Hydro.from_spec(spec, precision=rh.RH_PREC_FP32)
    rh.rh_set_timing(h.plan, True)
    got = h.vjp(u, w, t=t).double()
    # the rolls read the pack; rows fill it themselves
    assert rh.rh_kernel_times(h.plan)["other"][1] == (0 if "rows" in case else 1)
    h.close()

    def gradient(at):
        at = at.clone().requires_grad_(True)
        return torch.autograd.grad(cases._rhs(at, dict(spec, lf_local=False, eos=0), t), at, w.double())[0]

    ref = gradient(u.double())
    scale = torch.maximum(ref.abs().max(), w.abs().max().double() / min(spec["h"]))
    half_ulp = 0.5 * (torch.nextafter(u.abs(), torch.full_like(u, float("inf"))) - u.abs()).double()
    sign = torch.randint(0, 2, u.shape, device="cuda", generator=torch.Generator(device="cuda").manual_seed(15)) * 2 - 1
    sens = float((gradient(u.double() + half_ulp * sign) - ref).abs().max() / scale)
    err = ((got - ref).abs().reshape(5, -1).max(dim=1).values / scale).cpu().numpy()
    bar = min(2.5e-4, max(5e-5, 4.0 * sens))
    print(case, err, "sensitivity %.2e" % sens, flush=True)
    assert np.all(err <= bar), (err, bar)


@pytest.mark.parametrize("order,prec,shape,bc", [
    (5, "fp64", (86, 85, 83), (P, O, P)), (7, "fp64", (86, 85, 83), (P, P, P)), (5, "fp32", (86, 70, 69), (P, O, P)),
    (5, "fp32", (128, 58, 57), (P, P, O))])
def test_vjp_of_large_grids_with_floors(order, prec, shape, bc):
    rh = rh_module()
    spec = inputs.random_smooth(shape, h=0.1, seed=758, bc=bc, order=order)
    u, _ = planted_state(spec, 16)
    w = np.random.default_rng([16, 9]).normal(size=u.shape)
    bar = FP64_TOL
    if prec == "fp32":
        u, w = (a.astype(np.float32).astype(np.float64) for a in (u, w))
        bar = max(FP32_ADJ_TOL[order], 4.0 * _rounding_sensitivity(oracle, spec, u, w).max())
    h = rh.Hydro.from_spec(spec, precision=rh.RH_PREC_FP64 if prec == "fp64" else rh.RH_PREC_FP32)
    got = h.vjp(u, w).double().cpu().numpy()
    h.close()
    ref = oracle.vjp_L(oracle.grid_from_spec(spec), u, w)
    err = np.abs(got - ref).reshape(5, -1).max(axis=1) / max(np.abs(ref).max(), np.abs(w).max() / min(spec["h"]))
    print(order, prec, shape, err, bar, flush=True)
    assert np.all(np.isfinite(got))
    assert np.all(err <= bar), (err, bar)
