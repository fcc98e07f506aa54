"""BF16 stage launches of batches with more than a row tile a compute unit
(kept interpolants), whose weights are streamed with one or two row tiles a
workgroup: a batch of copies equals the small batch, on resident weights,
bitwise, and the one-launch solves to 1e-6 (their commits add the same terms
in another order)."""
import numpy as np
import pytest

from gpu_helpers import run_gpu
from paper_2210_12375_amd import binding as bd
from paper_2210_12375_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("field,d,hidden,n,copies", [
    ("mlp", 48, 128, 41, 103), ("mlp", 64, 256, 41, 101),
    ("mlp", 16, 64, 41, 101), ("mlp", 16, 128, 41, 803),
    ("cnf", 16, 256, 21, 98), ("cnf", 32, 64, 21, 98)])
def test_kept_interpolants(field, d, hidden, n, copies):
    print(f"bf16 stages {field} d={d} hidden={hidden} {n} x {copies}",
          flush=True)
    p = (W.neural_ode_fit(B=n, d=d, hidden=hidden, n_times=2)
         if field == "mlp" else W.cnf_density(B=n, d=d, hidden=hidden))
    rhs = bd.RHS_MLP if field == "mlp" else bd.RHS_CNF
    q = W.subset(p, np.tile(np.arange(n), copies))
    a, _ = run_gpu(p, method="dopri5", precision="bf16", rhs=rhs)
    for r, c, keep in ((p, 1, 1), (q, copies, 1), (q, copies, 0)):
        b, _ = run_gpu(r, method="dopri5", precision="bf16", rhs=rhs,
                       keep_dense=keep)
        for k in ("n_attempted", "n_accepted", "status"):
            np.testing.assert_array_equal(b[k], np.tile(a[k], c), err_msg=k)
        for k in ("y_eval", "y_final"):
            want = np.tile(a[k], (c,) + (1,) * (a[k].ndim - 1))
            assert np.abs(b[k] - want).max(initial=0) <= 1e-6 * max(
                1.0, np.abs(want).max(initial=0)), k
            if keep and c > 1:
                np.testing.assert_array_equal(b[k], np.tile(
                    small[k], (c,) + (1,) * (a[k].ndim - 1)), err_msg=k)
        if keep and c == 1:
            small = b
