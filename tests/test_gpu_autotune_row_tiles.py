"""The autotuner times one against two row tiles per workgroup only where the
kernels are built for both: elsewhere it keeps the default (0)."""
import pytest

from paper_2210_12375_amd import binding as bd
from paper_2210_12375_amd import workloads as W
from test_gpu_analytic import autotune

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,d,hidden,choice", [
    ("bf16", 64, 128, True), ("bf16", 80, 128, False), ("bf16", 80, 512, True),
    ("bf16", 144, 512, False), ("fp32", 80, 100, True),
    ("fp32", 130, 128, False), ("fp32", 16, 64, False)])
def test_candidates(precision, d, hidden, choice):
    print(f"autotune {precision} d={d} hidden={hidden}", flush=True)
    p = W.neural_ode(B=33, d=d, hidden=hidden)
    shape = autotune(p, precision, rhs=bd.RHS_MLP)
    assert shape["waves"] in ((4, 8) if choice else (0,))
