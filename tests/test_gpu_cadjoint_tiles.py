"""Continuous adjoint at the edges of what its matrix-core stages split:
widths that fill no tile, ragged batches around a tile and around the
sixteen instances whose gradients are summed at a time, both tableaux, and
instances without backward steps, against the oracle's continuous adjoint of
the same forward result, at the bars of the continuous-adjoint tests (FP32
1e-4, BF16 1e-2)."""
import numpy as np
import pytest

from gpu_helpers import as_float_inputs, assert_grads
from paper_2210_12375_amd import binding as bd
from test_gpu_cadjoint import cotangents, problem, reference, run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("joint", [0, 1])
@pytest.mark.parametrize("precision,kind,B,d,hidden,method", [
    ("fp32", "mlp", 1, 1, 1, "dopri5"), ("fp32", "mlp", 15, 17, 50, "tsit5"),
    ("fp32", "mlp", 17, 33, 100, "dopri5"), ("fp32", "cnf", 9, 7, 65, "tsit5"),
    ("bf16", "mlp", 16, 16, 64, "tsit5"), ("bf16", "cnf", 7, 48, 128, "dopri5"),
    ("fp64", "mlp", 33, 5, 9, "dopri5")])
def test_edges(precision, kind, B, d, hidden, method, joint):
    print(f"cadjoint {precision} {kind} B={B} d={d} H={hidden} {method} "
          f"joint={joint}", flush=True)
    p, rhs = problem(kind, B=B, d=d, hidden=hidden)
    ge, gf = cotangents(p, 3)
    g = run(p, precision, rhs, joint, ge, gf, method)
    assert np.all(g["fwd"] == bd.SUCCESS)
    assert np.all(g["st"][4] == bd.SUCCESS)
    q = p if precision == "fp64" else as_float_inputs(p)
    r = reference(q, g, joint, method)
    assert_grads(p, g, r["dy0"], r["dtheta"],
                 {"fp64": 1e-9, "fp32": 1e-4, "bf16": 1e-2}[precision])


@pytest.mark.parametrize("precision", ["fp32", "bf16"])
def test_no_backward_steps(precision):
    print(f"cadjoint {precision} empty spans", flush=True)
    p, rhs = problem("mlp", B=18, d=16, hidden=64)
    p["t_end"][::4] = 0.0
    p["t_eval"][::4] = 0.0
    ge, gf = cotangents(p, 4)
    g = run(p, precision, rhs, 0, ge, gf)
    r = reference(as_float_inputs(p), g, 0)
    assert np.array_equal(g["st"][4], r["status"])
    assert_grads(p, g, r["dy0"], r["dtheta"],
                 1e-4 if precision == "fp32" else 1e-2)
