"""J(u)^T w of a grid whose x adjoint needs more lanes than one row of a launch holds
(2^32; the short tiles take eight lanes a cell, more where they overhang the axis).

The data repeat with a period of 16 cells along y and z, so every 33 x 16 x 16 tile of
the result must equal every other one bit for bit, and tile 0 must be that of a
small grid of one tile (5e-5, the FP32 bar: the small grid's y and z take other kernels)."""
import numpy as np
import pytest

import oracle
from paper_1604_03360_amd import inputs
from gpu_helpers import rh_module

pytestmark = pytest.mark.gpu

P = 16
SHAPE = (33, 4000, 2800)


def test_x_adjoint_beyond_one_launch_row():
    import torch
    rh = rh_module()
    nx, ny, nz = SHAPE
    # three tiles of 16 positions, four lines each, 512 lanes a tile
    assert 3 * (ny * nz // 4) * 512 > 1 << 32
    tile = inputs.random_smooth((nx, P, P), h=0.1, seed=701, order=7)
    u = torch.tensor(oracle.prim2con(tile["prim"]), dtype=torch.float32, device="cuda")
    w = torch.tensor(np.random.default_rng(12).normal(size=u.shape), dtype=torch.float32, device="cuda")
    h = rh.Hydro.from_spec(tile, precision=rh.RH_PREC_FP32)
    ref = h.vjp(u, w, t=0.0)
    h.close()
    h = rh.Hydro.from_spec(dict(tile, shape=SHAPE, prim=None), precision=rh.RH_PREC_FP32)
    try:
        print("J^T w of %d x %d x %d" % SHAPE, flush=True)
        out = h.vjp(u.repeat(1, nz // P, ny // P, 1), w.repeat(1, nz // P, ny // P, 1), t=0.0)
        tiles = out.view(5, nz // P, P, ny // P, P, nx)
        first = tiles[:, :1, :, :1]
        assert all(torch.equal(tiles[c], first[c].expand_as(tiles[c])) for c in range(5))
        err = (first[:, 0, :, 0] - ref).abs().reshape(5, -1).max(dim=1).values / ref.abs().max()
        assert bool((err <= 5e-5).all()), err
    finally:
        h.close()
        del h
        torch.cuda.empty_cache()
