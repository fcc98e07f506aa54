"""FP32 and BF16 neural fields at the edge of the type's range:
pre-activations far beyond the largest float and (FP32) infinite stage inputs
saturate their units, as plain products do, and do not turn the row into NaN.
Saturated units are +-1 exactly, so the rest is the arithmetic, and the bars,
of every parity test (FP32 1e-4, BF16 1e-2)."""
import numpy as np
import pytest

import oracle
from gpu_helpers import as_float_inputs, run_gpu
from paper_2210_12375_amd import binding as bd
from paper_2210_12375_amd import workloads as W
from test_gpu_neural import replay_rel

pytestmark = pytest.mark.gpu

SHAPES = [(3, 17), (16, 64), (40, 130), (64, 256), (20, 300)]


@pytest.mark.parametrize("keep", [0, 1])
@pytest.mark.parametrize("precision,tol,d,hidden", [
    ("fp32", 1e-4) + s for s in SHAPES] + [
    ("bf16", 1e-2) + s for s in [(16, 64), (64, 256), (96, 128), (32, 512)]])
def test_overflowing_products(precision, tol, d, hidden, keep):
    print(f"{precision} overflowing products d={d} hidden={hidden}", flush=True)
    p = W.neural_ode(B=5, d=d, hidden=hidden)
    m = {k: np.array(v) for k, v in p["mlp"].items()}
    p["y0"] = np.abs(p["y0"]) + 1e6
    # each column one sign, so the products (1e44) are too; their rounding to
    # any shorter type's residuals (1e41) is of both
    w = np.random.default_rng(5).uniform(1e38, 3.3e38, (d, hidden))
    m["W1"][:d] = np.where(np.arange(hidden) % 2, w, -w)
    p["mlp"] = m
    g, _ = run_gpu(p, precision=precision, rhs=bd.RHS_MLP, record_cap=256,
                   keep_dense=keep)
    assert np.all(g["status"] == bd.SUCCESS)
    assert np.all(np.isfinite(g["y_final"]))
    assert replay_rel(p, g, "dopri5", precision).max() <= tol


@pytest.mark.parametrize("keep", [0, 1])
@pytest.mark.parametrize("d,hidden", SHAPES)
def test_infinite_inputs(d, hidden, keep):
    """The first component grows past the largest float, the others see only
    saturated units."""
    print(f"fp32 infinite inputs d={d} hidden={hidden}", flush=True)
    p = W.neural_ode(B=5, d=d, hidden=hidden)
    m = {k: np.array(v) for k, v in p["mlp"].items()}
    p["y0"][:, 0] = 3.3e38
    p["t_end"][:] = 4.0
    p["h0"] = np.full(5, 0.5)
    m["W1"][0] = np.where(np.arange(hidden) % 3, 0.3, -0.7)
    m["W3"][:, 0] = 0.0
    m["b3"][0] = 1e37
    p["mlp"] = m
    g, _ = run_gpu(p, precision="fp32", rhs=bd.RHS_MLP, keep_dense=keep,
                   fixed_step=1)
    q = as_float_inputs(p)
    r = oracle.solve(q, method="dopri5", h_replay=np.full((5, 8), 0.5),
                     n_replay=np.full(5, 8, np.int32))
    assert np.all(np.isposinf(g["y_final"][:, 0])), g["y_final"][:, 0]
    a, b = g["y_final"][:, 1:], r["y_final"][:, 1:]
    assert np.abs(a - b).max() <= 1e-4 * np.abs(b).max()
