"""FP64 CNFs whose state is wider than the hidden layer (the probe-tangent
products of the log-density take more columns than a layer's row): solves,
kept interpolants and both adjoints against the FP64 oracle, at the bars of
every FP64 check (identical counts, 1e-9)."""
import numpy as np
import pytest

import oracle
from gpu_helpers import assert_fp64_parity, assert_grads, run_gpu
from paper_2210_12375_amd import binding as bd
from paper_2210_12375_amd import workloads as W
from test_gpu_adjoint import cotangents, gpu_grad, oracle_grad
from test_gpu_cadjoint import reference, run

pytestmark = pytest.mark.gpu


# 4 instances a tile up to 1024 of them, 8 beyond
@pytest.mark.parametrize("B,d,hidden", [
    (9, 25, 1), (5, 60, 20), (9, 64, 16), (3, 130, 20), (3, 200, 16),
    (1025, 64, 16)])
def test_solve_and_adjoint(B, d, hidden):
    print(f"fp64 cnf B={B} d={d} hidden={hidden}", flush=True)
    p = W.cnf_density(B=B, d=d, hidden=hidden)
    r = oracle.solve(p, method="dopri5")
    for keep in (0, 1):  # one launch a solve; one a stage
        g, _ = run_gpu(p, method="dopri5", rhs=bd.RHS_CNF, keep_dense=keep)
        assert_fp64_parity(g, r)
    ge, gf = cotangents(p)
    b = gpu_grad(p, "tsit5", "fp64", bd.RHS_CNF, 2, ge, gf)
    assert np.all(b["status"] == bd.SUCCESS)
    (dy0, dth), _ = oracle_grad(p, b, "tsit5", ge, gf)
    assert_grads(p, b, dy0, dth, 1e-9)


@pytest.mark.parametrize("joint", [0, 1])
def test_continuous_adjoint(joint):
    print(f"fp64 cnf cadjoint d=40 hidden=6 joint={joint}", flush=True)
    p = W.cnf_density(B=7, d=40, hidden=6)
    ge, gf = cotangents(p)
    g = run(p, "fp64", bd.RHS_CNF, joint, ge, gf)
    assert np.all(g["fwd"] == bd.SUCCESS)
    r = reference(p, g, joint)
    assert np.array_equal(g["st"][0], r["n_attempted"])
    assert_grads(p, g, r["dy0"], r["dtheta"], 1e-9)
