"""FP32 neural fields on the matrix cores (values split into three BF16 terms)
at the edges of their tile shapes: widths that fill no tile and are padded
inside the kernels, streamed and resident weights, one and two row tiles per
workgroup, ragged batches, rows with fewer steps than their tile.

The split leaves about 2^-24 of each value, so FP32 results are FP32
arithmetic in another order: the FP32 bars of the parity tests apply (1e-4
per attempt and per gradient).  A batch of copies equals the small batch
bitwise, whatever tile an instance lies in."""
import numpy as np
import pytest

from gpu_helpers import as_float_inputs, assert_grads, run_gpu
from paper_2210_12375_amd import binding as bd
from paper_2210_12375_amd import workloads as W
from test_gpu_adjoint import cotangents, gpu_grad, oracle_grad
from test_gpu_neural import replay_rel

pytestmark = pytest.mark.gpu


def problem(field, B, d, hidden, E):
    if field == "mlp":
        return W.neural_ode_fit(B=B, d=d, hidden=hidden, n_times=E), bd.RHS_MLP
    return W.cnf_density(B=B, d=d, hidden=hidden), bd.RHS_CNF


@pytest.mark.parametrize("B,d,hidden,E", [
    (17, 1, 1, 2), (5, 17, 50, 1), (19, 33, 100, 0), (7, 256, 128, 1),
    (33, 31, 129, 3), (1, 64, 256, 70), (16, 129, 300, 2), (9, 255, 512, 2)])
def test_widths(B, d, hidden, E):
    print(f"fp32 mlp B={B} d={d} hidden={hidden} E={E}", flush=True)
    p, rhs = problem("mlp", B, d, hidden, E)
    g, _ = run_gpu(p, method="dopri5", precision="fp32", rhs=rhs,
                   record_cap=256)
    assert np.all(g["status"] == bd.SUCCESS)
    assert replay_rel(p, g, "dopri5", "fp32").max() <= 1e-4


@pytest.mark.parametrize("field,d,hidden,n,copies", [
    ("mlp", 33, 50, 41, 101), ("mlp", 64, 256, 41, 101),
    ("mlp", 20, 300, 37, 113), ("cnf", 7, 70, 21, 98), ("cnf", 3, 500, 21, 98)])
def test_two_row_tiles(field, d, hidden, n, copies):
    print(f"fp32 {field} d={d} hidden={hidden} {n} x {copies}", flush=True)
    p, rhs = problem(field, n, d, hidden, 2)
    q = W.subset(p, np.tile(np.arange(n), copies))
    a, _ = run_gpu(p, method="tsit5", precision="fp32", rhs=rhs)
    b, _ = run_gpu(q, method="tsit5", precision="fp32", rhs=rhs)
    for k in ("y_eval", "y_final", "n_attempted", "n_accepted", "status"):
        want = np.tile(a[k], (copies,) + (1,) * (a[k].ndim - 1))
        np.testing.assert_array_equal(b[k], want, err_msg=k)


@pytest.mark.parametrize("field,B,d,hidden,ck", [
    ("mlp", 17, 1, 1, 2), ("mlp", 5, 17, 50, 1), ("mlp", 19, 33, 100, 3),
    ("mlp", 7, 256, 128, 2), ("mlp", 33, 31, 129, 2), ("mlp", 9, 129, 300, 2),
    ("mlp", 4, 255, 512, 1), ("mlp", 4200, 6, 50, 2), ("cnf", 9, 1, 1, 2),
    ("cnf", 11, 17, 65, 1), ("cnf", 4, 47, 256, 2), ("cnf", 5, 130, 300, 2)])
def test_adjoint(field, B, d, hidden, ck):
    print(f"fp32 adjoint {field} B={B} d={d} hidden={hidden}", flush=True)
    p, rhs = problem(field, B, d, hidden, 3)
    p["t_end"][::3] = 0.25  # fewer steps than the others of their tile
    p["t_eval"][::3] *= 0.25
    ge, gf = cotangents(p)
    g = gpu_grad(p, "dopri5", "fp32", rhs, ck, ge, gf)
    assert np.all(g["status"] == bd.SUCCESS)
    (dy0, dth), _ = oracle_grad(as_float_inputs(p), g, "dopri5", ge, gf)
    assert_grads(p, g, dy0, dth, 1e-4)
