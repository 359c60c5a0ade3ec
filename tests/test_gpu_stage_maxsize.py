"""The fused stage on the largest grids the boundary accepts (one field below 4 GiB):
rows that are not 256 cells long take it by default.  As in the sweeps' test of that
size, the data repeat with a period of 16 cells along every axis, so every 16^3 tile of the
result must equal every other one bit for bit, and tile 0 the FP64 oracle on one tile
(1e-12 FP64, 2e-5 FP32)."""
import numpy as np
import pytest
import torch

from gpu_helpers import field_errors, oracle_steps, rh_module
from test_gpu_maxsize import FIELD_LIMIT, P, STEPS, tile_spec

pytestmark = pytest.mark.gpu

CASES = [
    ((272, 1984, 1984), "fp32", 5, 2e-5),
    ((272, 1984, 992), "fp64", 5, 1e-12),
    ((1984, 272, 1984), "fp32", 7, 2e-5),
    ((992, 1984, 272), "fp64", 7, 1e-12),
]


@pytest.mark.parametrize("shape,precision,order,tol", CASES)
def test_stage_at_the_field_limit(shape, precision, order, tol):
    rh = rh_module()
    nx, ny, nz = shape
    share = nx * ny * nz * (4 if precision == "fp32" else 8) / FIELD_LIMIT
    assert 0.98 < share < 1.0
    print("grid %s %s WENO%d, %.3f of the field limit" % (shape, precision, order, share), flush=True)
    tile = tile_spec(order)
    h = rh.Hydro.from_spec(dict(tile, shape=shape, prim=None),
                           precision=rh.RH_PREC_FP32 if precision == "fp32" else rh.RH_PREC_FP64)
    try:
        if order == 5:
            assert rh.rh_get_path(h.plan) == rh.RH_PATH_STAGE
        rh.rh_set_path(h.plan, rh.RH_PATH_STAGE)
        prim = torch.as_tensor(tile["prim"], device="cuda").repeat(1, nz // P, ny // P, nx // P)
        h.set_primitive(prim)
        del prim
        h.step(tile["dt"], STEPS)
        _, cnt = h.totals()
        st = h.state.view(5, nz // P, P, ny // P, P, nx // P, P)
        ref = st[:, :1, :, :1, :, :1, :]
        same = all(torch.equal(st[f], ref[f].expand_as(st[f])) for f in range(5))
        tile0 = st[:, 0, :, 0, :, 0, :].double().cpu().numpy()
        del st, ref
    finally:
        h.close()
        del h
        torch.cuda.empty_cache()
    assert same and cnt == [0, 0]
    err = field_errors(tile0, oracle_steps(tile, STEPS)[0])
    print("tile 0 against the oracle", err, flush=True)
    assert np.all(err <= tol), err
