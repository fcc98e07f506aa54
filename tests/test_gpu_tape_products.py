"""Parameter-gradient products at the edges of their tiles: every tile shape
of the FP32 and FP64 kernels with ragged widths and row counts, one and many
k-splits, and the split-BF16 kernel's 128- and 256-row tiles.

Small batches go against the oracle's adjoint at the bars of the adjoint
tests (FP64 1e-9, FP32 1e-4).  The 256-row tiles need long tapes: there the
batch is 100 copies of a small one, whose gradient is 100 times the small
batch's; both are sums of products exact to 2^-16 with FP32 accumulation
(the rest of the arithmetic is the same for a copy), so they agree to 1e-4."""
import numpy as np
import pytest
import torch

from gpu_helpers import as_float_inputs, assert_grads
from paper_2210_12375_amd import binding as bd
from paper_2210_12375_amd import workloads as W
from test_gpu_adjoint import cotangents, gpu_grad, oracle_grad
from test_gpu_bf16_adjoint_tiles import bf16_model

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,B,d,hidden", [
    ("fp64", 3, 16, 17), ("fp64", 5, 48, 70), ("fp64", 7, 80, 100),
    ("fp64", 2, 130, 140), ("fp64", 61, 20, 33), ("fp32", 5, 16, 17),
    ("fp32", 3, 48, 70), ("fp32", 67, 80, 100), ("fp32", 2, 130, 140),
    ("bf16", 9, 256, 256), ("bf16", 21, 256, 512)])
def test_shapes(precision, B, d, hidden):
    print(f"{precision} tape products B={B} d={d} hidden={hidden}", flush=True)
    p = W.neural_ode_fit(B=B, d=d, hidden=hidden, n_times=2)
    ge, gf = cotangents(p)
    g = gpu_grad(p, "dopri5", precision, bd.RHS_MLP, 2, ge, gf)
    assert np.all(g["status"] == bd.SUCCESS)
    q = (p if precision == "fp64" else
         bf16_model(p, d) if precision == "bf16" else as_float_inputs(p))
    (dy0, dth), _ = oracle_grad(q, g, "dopri5", ge, gf)
    assert_grads(p, g, dy0, dth, 1e-9 if precision == "fp64" else 1e-4)


@pytest.mark.parametrize("field,n,d,hidden", [
    ("cnf", 27, 16, 512), ("mlp", 53, 256, 512), ("mlp", 51, 64, 256)])
def test_long_tapes(field, n, d, hidden):
    copies = 100
    print(f"bf16 {field} d={d} hidden={hidden} {n} x {copies}", flush=True)
    if field == "mlp":
        p, rhs = W.neural_ode_fit(B=n, d=d, hidden=hidden, n_times=2), bd.RHS_MLP
    else:
        p, rhs = W.cnf_density(B=n, d=d, hidden=hidden), bd.RHS_CNF
    q = W.subset(p, np.tile(np.arange(n), copies))
    ge, gf = cotangents(p)
    tile = lambda a: None if a is None else np.tile(
        a, (copies,) + (1,) * (a.ndim - 1))
    a = gpu_grad(p, "dopri5", "bf16", rhs, 2, ge, gf)
    b = gpu_grad(q, "dopri5", "bf16", rhs, 2, tile(ge), tile(gf))
    assert np.all(b["status"] == bd.SUCCESS)
    want = copies * a["dth"]
    err = np.linalg.norm(b["dth"] - want) / np.linalg.norm(want)
    print(f"  dtheta {err:.1e}", flush=True)
    assert err <= 1e-4
