"""Analytic batches on both sides of the rules that spread small ones over
wavefronts (evaluation times per instance, instances): an instance's results
are the same bits on either."""
import numpy as np
import pytest

from gpu_helpers import run_gpu
from paper_2210_12375_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("E", [7, 8, 47, 48, 63, 64])
def test_spread(precision, E):
    print(f"analytic spread {precision} E={E}", flush=True)
    p = W.uneven_batch(seed=4, B=64, E=E)
    q = W.subset(p, np.tile(np.arange(64), 10))  # 320 of each kind: not spread
    a, _ = run_gpu(p, precision=precision)
    b, _ = run_gpu(q, precision=precision)
    for k in ("y_eval", "y_final", "n_attempted", "n_accepted", "status"):
        want = np.tile(a[k], (10,) + (1,) * (a[k].ndim - 1))
        np.testing.assert_array_equal(b[k], want, err_msg=k)
