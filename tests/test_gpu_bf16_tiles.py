"""BF16 forward kernels at the edges of their tile shapes: state widths with
one to four output tiles a wavefront, streamed and resident weights, one and
two row tiles per workgroup, ragged batches, evaluation times in LDS and not.

Widths: the attempt-by-attempt check against the oracle with the BF16 bars of
the neural parity tests.  Row tiles: an instance's arithmetic does not depend
on its tile, so a batch of copies must equal the small batch bitwise."""
import numpy as np
import pytest

from gpu_helpers import run_gpu
from paper_2210_12375_amd import binding as bd
from paper_2210_12375_amd import workloads as W
from test_gpu_neural import replay_rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,d,hidden,E", [
    (17, 256, 64, 2), (5, 128, 64, 1), (19, 208, 128, 0), (7, 256, 512, 1),
    (33, 80, 256, 3), (1, 16, 256, 70)])
def test_widths(B, d, hidden, E):
    print(f"bf16 mlp B={B} d={d} hidden={hidden} E={E}", flush=True)
    p = W.neural_ode_fit(B=B, d=d, hidden=hidden, n_times=E)
    g, _ = run_gpu(p, method="dopri5", precision="bf16", rhs=bd.RHS_MLP,
                   record_cap=256)
    assert np.all(g["status"] == bd.SUCCESS)
    assert replay_rel(p, g, "dopri5", "bf16").max() <= 1e-2


@pytest.mark.parametrize("field,d,hidden,n,copies", [
    ("mlp", 64, 256, 41, 101), ("mlp", 16, 128, 41, 101),
    ("mlp", 32, 512, 37, 113), ("cnf", 16, 512, 21, 98),
    ("cnf", 48, 256, 21, 98)])
def test_two_row_tiles(field, d, hidden, n, copies):
    print(f"bf16 {field} d={d} hidden={hidden} {n} x {copies}", flush=True)
    p = (W.neural_ode_fit(B=n, d=d, hidden=hidden, n_times=2)
         if field == "mlp" else W.cnf_density(B=n, d=d, hidden=hidden))
    rhs = bd.RHS_MLP if field == "mlp" else bd.RHS_CNF
    q = W.subset(p, np.tile(np.arange(n), copies))
    a, _ = run_gpu(p, method="tsit5", precision="bf16", rhs=rhs)
    b, _ = run_gpu(q, method="tsit5", precision="bf16", rhs=rhs)
    for k in ("y_eval", "y_final", "n_attempted", "n_accepted", "status"):
        want = np.tile(a[k], (copies,) + (1,) * (a[k].ndim - 1))
        np.testing.assert_array_equal(b[k], want, err_msg=k)
