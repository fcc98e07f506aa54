"""Rounding of the FP32 parameter gradients, sums over ten thousand tape rows
taken in few k-splits (batches whose tiles leave the products few workgroups):
against the FP64 oracle on the same steps, in the l2 norm of each layer.

A product's two factors come with two to three roundings each, and a sum is
closed after at most 384 rows (96 additions on the matrix cores, random
roundings): about (2.5^2 + 96 / 12)^(1/2) = 3.8 u with u = 2^-24.  Bar: 4 u;
a chain of 2600 rows, 650 additions, comes to 7.8 u."""
import numpy as np
import pytest

from gpu_helpers import as_float_inputs
from paper_2210_12375_amd import binding as bd
from paper_2210_12375_amd import workloads as W
from test_gpu_adjoint import PARAMS, gpu_grad, oracle_grad

pytestmark = pytest.mark.gpu

U = 2.0 ** -24


@pytest.mark.parametrize("B,d,hidden", [
    (500, 16, 256), (700, 31, 60), (250, 20, 500)])
def test_layers(B, d, hidden):
    print(f"fp32 gradient error cnf B={B} d={d} H={hidden}", flush=True)
    p, rhs = W.cnf_density(B=B, d=d, hidden=hidden), bd.RHS_CNF
    q = as_float_inputs(p)
    ge = None
    # cotangents of one sign, as a loss's bias gradients sum them
    gf = np.abs(np.random.default_rng(3).standard_normal(
        p["y0"].shape)).astype(np.float32).astype(np.float64)
    g = gpu_grad(p, "dopri5", "fp32", rhs, 2, ge, gf)
    assert np.all(g["status"] == bd.SUCCESS)
    (dy0, dth), _ = oracle_grad(q, g, "dopri5", ge, gf)
    off = 0
    for k in PARAMS:
        n = np.asarray(p["mlp"][k]).size
        a, b = g["dth"][off:off + n], dth[off:off + n]
        off += n
        err = np.linalg.norm(a - b) / np.linalg.norm(b) / U
        print(f"  {k} {err:.2f} u", flush=True)
        assert err <= 4.0, k
