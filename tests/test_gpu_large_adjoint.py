"""Training steps of batches with more than two tiles a compute unit: the
BF16 step VJPs there, with the segment store and with the one-step store that
replaces it when a segment would not fit (here one segment of the whole
solve).  The batch is copies of a small one.  A row's sums do not depend on
its tile, so state gradients agree with the small batch's to 1e-5 of the
largest; the parameter gradient is the small one's multiplied, to 1e-4 (the
tape products accumulate in another order)."""
import numpy as np
import pytest

from paper_2210_12375_amd import binding as bd
from paper_2210_12375_amd import workloads as W
from test_gpu_adjoint import cotangents, gpu_grad

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("field,n,copies,d,hidden,ck,cap", [
    ("mlp", 33, 251, 16, 64, 2, 64),   # 518 tiles, segment store
    ("mlp", 33, 251, 16, 64, 0, 80),   # one-step store (2.6 GB a segment)
    ("mlp", 41, 203, 48, 128, 3, 64),
    ("cnf", 21, 197, 16, 64, 2, 64),
    ("cnf", 21, 197, 32, 256, 1, 64)])
def test_copies(field, n, copies, d, hidden, ck, cap):
    print(f"bf16 {field} d={d} hidden={hidden} {n} x {copies} ck={ck}",
          flush=True)
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
    a = gpu_grad(p, "tsit5", "bf16", rhs, 2, ge, gf)
    b = gpu_grad(q, "tsit5", "bf16", rhs, ck, tile(ge), tile(gf),
                 record_cap=cap)
    assert np.all(b["status"] == bd.SUCCESS)
    want = tile(a["dy0"])
    err = np.abs(b["dy0"] - want).max() / np.abs(want).max()
    dth = copies * a["dth"]
    eth = np.linalg.norm(b["dth"] - dth) / np.linalg.norm(dth)
    print(f"  dy0 {err:.1e} dtheta {eth:.1e}", flush=True)
    assert err <= 1e-5
    assert eth <= 1e-4
