"""The launch shape an ensemble starts with is one of those its autotuning times: a
small ensemble, whose default z segments are shorter than every fixed candidate and
take less than half of the time, keeps them."""
import pytest

from paper_1604_03360_amd import inputs
from gpu_helpers import rh_module

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order,prec", [(7, "fp64"), (7, "fp32"), (2, "fp64")])
def test_autotune_times_the_default(order, prec):
    rh = rh_module()
    specs = [inputs.random_smooth((24, 20, 24), h=0.1, seed=901 + k, order=order) for k in range(2)]
    b = rh.Batch(specs, precision=rh.RH_PREC_FP64 if prec == "fp64" else rh.RH_PREC_FP32)
    b.set_primitive([sp["prim"] for sp in specs])
    default = tuple(rh.rh_batch_get_stage_tuning(b.batch))
    shape, source = b.autotune(20)
    assert source == "timed"
    assert default[1] < 4 and shape == default
    b.close()
