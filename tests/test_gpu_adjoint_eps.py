"""J(u)^T w with a small epsilon of the nonlinear weights, where the data are flat: the
smoothness indicators are then epsilon alone and their powers come near the ends of
the FP32 range.  At a uniform state the weights are the linear ones, whatever epsilon
is; 5e-5 is the FP32 bar of the other adjoint tests."""
import numpy as np
import pytest

import oracle
from paper_1604_03360_amd import inputs
from gpu_helpers import rh_module

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(13, 11, 10), (64, 6, 5), (106, 104, 102)])   # tiles, rows of x, rolls
@pytest.mark.parametrize("order,eps", [(5, 1e-9), (7, 1e-15), (7, 5e-20)])
def test_fp32_vjp_of_flat_data(order, eps, shape):
    rh = rh_module()
    spec = dict(inputs.random_smooth(shape, h=0.1, seed=801, order=order), eps=eps)
    spec["prim"] = np.ones_like(spec["prim"]) * np.array([1.0, 0.1, -0.2, 0.05, 0.5])[:, None, None, None]
    u = oracle.prim2con(spec["prim"]).astype(np.float32).astype(np.float64)
    w = np.random.default_rng(13).normal(size=u.shape).astype(np.float32).astype(np.float64)
    h = rh.Hydro.from_spec(spec, precision=rh.RH_PREC_FP32)
    got = h.vjp(u, w, t=0.0).double().cpu().numpy()
    h.close()
    ref = oracle.vjp_L(oracle.grid_from_spec(dict(spec, eps=1e-6)), u, w, t=0.0)
    err = np.abs(got - ref).max() / max(np.abs(ref).max(), np.abs(w).max() / min(spec["h"]))
    assert err <= 5e-5, err
