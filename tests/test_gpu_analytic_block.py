"""Analytic solves with a workgroup size that is no multiple of a wavefront
(FP64 Van der Pol instances take two lanes each, which must both be there):
bitwise the results of the default size."""
import numpy as np
import pytest

from gpu_helpers import run_gpu
from paper_2210_12375_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("block", [1, 33, 95, 130, 255])
def test_any_block(precision, block):
    print(f"analytic {precision} block {block}", flush=True)
    p = W.uneven_batch(B=301)
    a, _ = run_gpu(p, precision=precision)
    b, _ = run_gpu(p, precision=precision, tune_block=block)
    for k in ("status", "n_accepted", "n_rejected", "y_eval", "y_final"):
        np.testing.assert_array_equal(a[k], b[k], err_msg=k)
