"""Analytic instances on one lane, on pairs of lanes (FP64 Van der Pol) and
spread over wavefronts: an instance's arithmetic is the same wherever it
runs, so a batch of copies equals the small batch bitwise, whatever the
batch sizes around a wavefront and around the spreading rule."""
import numpy as np
import pytest

from gpu_helpers import run_gpu
from paper_2210_12375_amd import binding as bd
from paper_2210_12375_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("n,copies,E,kw", [
    (1, 65, 3, {}), (31, 3, 8, {}), (32, 9, 130, {}), (33, 16, 127, {}),
    (64, 4, 64, {}), (51, 51, 128, dict(beta1=0.25, beta2=0.07, beta3=0.03)),
    (43, 7, 5, dict(max_steps=60)), (40, 10, 6, dict(tune_lanes=37)),
    (40, 10, 6, dict(tune_lanes=300, tune_block=256))])
def test_copies(precision, n, copies, E, kw):
    print(f"{precision} {n} x {copies} E={E} {kw}", flush=True)
    p = W.uneven_batch(seed=9, B=n, E=E)
    q = W.subset(p, np.tile(np.arange(n), copies))
    a, _ = run_gpu(p, method="dopri5", precision=precision, **kw)
    b, _ = run_gpu(q, method="dopri5", precision=precision, **kw)
    for k in ("y_eval", "y_final", "n_attempted", "n_accepted", "status"):
        want = np.tile(a[k], (copies,) + (1,) * (a[k].ndim - 1))
        np.testing.assert_array_equal(b[k], want, err_msg=k)
