"""FP64 neural fields on the matrix cores at the edges of their tiles (4, 8
and 16 rows, 16 columns, 8-wide k blocks, one and two column tiles a
wavefront) against the FP64 oracle: identical counts, outputs and gradients
within 1e-9, the bars of every FP64 check here."""
import numpy as np
import pytest

import oracle
from gpu_helpers import assert_fp64_parity, assert_grads, run_gpu
from paper_2210_12375_amd import binding as bd
from paper_2210_12375_amd import workloads as W
from test_gpu_adjoint import cotangents, gpu_grad, oracle_grad

pytestmark = pytest.mark.gpu


def problem(field, B, d, hidden):
    if field == "mlp":
        return W.neural_ode_fit(B=B, d=d, hidden=hidden, n_times=3), bd.RHS_MLP
    return W.cnf_density(B=B, d=d, hidden=hidden), bd.RHS_CNF


@pytest.mark.parametrize("field,B,d,hidden", [
    ("mlp", 1, 1, 1), ("mlp", 5, 3, 17), ("mlp", 9, 16, 130),
    ("mlp", 6, 257, 300), ("mlp", 1025, 17, 33), ("mlp", 2049, 2, 20),
    ("cnf", 3, 1, 5), ("cnf", 5, 17, 130), ("cnf", 1025, 2, 9)])
def test_tile_edges(field, B, d, hidden):
    print(f"fp64 {field} B={B} d={d} hidden={hidden}", flush=True)
    p, rhs = problem(field, B, d, hidden)
    g, _ = run_gpu(p, method="dopri5", rhs=rhs)
    r = oracle.solve(p, method="dopri5")
    assert_fp64_parity(g, r)
    # the per-stage kernels (kept interpolant) take the same decisions
    k, _ = run_gpu(p, method="dopri5", rhs=rhs, keep_dense=1)
    assert_fp64_parity(k, r)
    ge, gf = cotangents(p)
    b = gpu_grad(p, "tsit5", "fp64", rhs, 2, ge, gf)
    (dy0, dth), _ = oracle_grad(p, b, "tsit5", ge, gf)
    assert_grads(p, b, dy0, dth, 1e-9)


def test_beyond_the_tiles_lds():
    print("fp64 mlp d=1024 hidden=2048", flush=True)
    p = W.neural_ode(B=2, d=1024, hidden=2048)
    g, _ = run_gpu(p, method="dopri5", rhs=bd.RHS_MLP)
    assert_fp64_parity(g, oracle.solve(p, method="dopri5"))


def test_saturated_unit_beside_padding():
    """A pre-activation that overflows to infinity saturates its tanh; the
    padding columns of its tile must not turn it into NaN."""
    print("fp64 saturated unit", flush=True)
    p = W.neural_ode(B=3, d=3, hidden=17)
    p["y0"] = np.abs(p["y0"]) + 30.0
    p["mlp"]["W1"][:, 0] = 1e308
    g, _ = run_gpu(p, method="dopri5", rhs=bd.RHS_MLP)
    r = oracle.solve(p, method="dopri5")
    assert np.all(np.isfinite(r["y_final"]))
    assert_fp64_parity(g, r)
