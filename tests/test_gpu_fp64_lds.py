"""FP64 neural fields at the shapes whose tile, with its block of stages or
cotangents, comes within some bytes of a compute unit's LDS: each takes the
next smaller form and agrees with the FP64 oracle (identical counts, 1e-9).
The batches repeat a few instances, so the oracle solves few."""
import numpy as np
import pytest

import oracle
from gpu_helpers import assert_fp64_parity, assert_grads, run_gpu
from paper_2210_12375_amd import binding as bd
from paper_2210_12375_amd import workloads as W
from test_gpu_adjoint import cotangents, gpu_grad, oracle_grad

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("field,d,hidden,B", [
    ("mlp", 128, 112, 2100), ("mlp", 96, 240, 2049), ("mlp", 64, 353, 2049),
    ("mlp", 128, 737, 1025), ("mlp", 5, 620, 2049), ("mlp", 512, 490, 9),
    ("cnf", 64, 580, 1025)])
def test_solve(field, d, hidden, B):
    print(f"fp64 {field} d={d} hidden={hidden} B={B}", flush=True)
    p, rhs = ((W.neural_ode(B=3, d=d, hidden=hidden), bd.RHS_MLP)
              if field == "mlp" else
              (W.cnf_density(B=3, d=d, hidden=hidden), bd.RHS_CNF))
    r = oracle.solve(p, method="dopri5")
    rep = np.arange(B) % 3
    for keep in (0, 1):
        g, _ = run_gpu(W.subset(p, rep), method="dopri5", rhs=rhs,
                       keep_dense=keep)
        assert_fp64_parity(g, {k: v[rep] if isinstance(v, np.ndarray) and
                               v.shape[:1] == (3,) else v
                               for k, v in r.items()})


def test_adjoint():
    print("fp64 mlp adjoint d=64 hidden=330 B=2049", flush=True)
    p = W.neural_ode_fit(B=3, d=64, hidden=330, n_times=2)
    ge, gf = cotangents(p)
    q = W.subset(p, np.arange(2049) % 3)
    g = gpu_grad(q, "dopri5", "fp64", bd.RHS_MLP, 2, ge[np.arange(2049) % 3],
                 gf[np.arange(2049) % 3])
    s = {k: v[:3] for k, v in g.items() if k != "dth"}
    (dy0, dth), _ = oracle_grad(p, s, "dopri5", ge, gf)
    # 2049 = 683 copies of each
    assert_grads(p, dict(s, dth=g["dth"] / 683.0), dy0, dth, 1e-9)
