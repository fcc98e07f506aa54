"""Training steps whose segment of stored stages would exceed 2 GiB: FP32
fields on the one-step store (regular and padded widths), FP64 fields with
their layers recomputed by the plain kernels.  The batch is copies of a small
one, which has the segment store: state gradients agree with the small batch's
and the parameter gradient is the small one's multiplied, to the bars of the
precision's gradient tests (FP32 1e-4, FP64 1e-9)."""
import numpy as np
import pytest

from paper_2210_12375_amd import binding as bd
from paper_2210_12375_amd import workloads as W
from test_gpu_adjoint import cotangents, gpu_grad

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,field,n,copies,d,hidden,cap", [
    ("fp32", "mlp", 33, 251, 16, 64, 80), ("fp32", "mlp", 33, 251, 6, 50, 100),
    ("fp32", "cnf", 21, 197, 7, 60, 80), ("fp64", "mlp", 33, 251, 16, 64, 45),
    ("fp64", "cnf", 21, 197, 5, 40, 60)])
def test_copies(precision, field, n, copies, d, hidden, cap):
    print(f"{precision} {field} d={d} hidden={hidden} {n} x {copies}",
          flush=True)
    B = n * copies
    rows = B * (2 if field == "cnf" else 1)
    size = 8 if precision == "fp64" else 4
    D = d + (field == "cnf")
    assert cap * 7 * (B * D + rows * 2 * hidden) * size > 2 << 30
    if field == "mlp":
        p, rhs = W.neural_ode_fit(B=n, d=d, hidden=hidden, n_times=3), bd.RHS_MLP
    else:
        p, rhs = W.cnf_density(B=n, d=d, hidden=hidden), bd.RHS_CNF
    p["t_end"][::3] = 0.25  # fewer steps than the others of their tile
    p["t_eval"][::3] *= 0.25
    q = W.subset(p, np.tile(np.arange(n), copies))
    ge, gf = cotangents(p)
    tile = lambda a: None if a is None else np.tile(
        a, (copies,) + (1,) * (a.ndim - 1))
    a = gpu_grad(p, "dopri5", precision, rhs, 2, ge, gf)
    b = gpu_grad(q, "dopri5", precision, rhs, 0, tile(ge), tile(gf),
                 record_cap=cap)
    assert np.all(b["status"] == bd.SUCCESS)
    want = tile(a["dy0"])
    err = np.abs(b["dy0"] - want).max() / np.abs(want).max()
    dth = copies * a["dth"]
    eth = np.linalg.norm(b["dth"] - dth) / np.linalg.norm(dth)
    print(f"  dy0 {err:.1e} dtheta {eth:.1e}", flush=True)
    assert max(err, eth) <= (1e-9 if precision == "fp64" else 1e-4)
