"""State-typed inputs and cotangents that begin one element past an aligned
address (slices of larger tensors): bitwise the results of aligned ones."""
import numpy as np
import pytest
import torch

from paper_2210_12375_amd import binding as bd
from paper_2210_12375_amd import workloads as W
from paper_2210_12375_amd.autograd import PARAMS

pytestmark = pytest.mark.gpu


def shifted(t):
    buf = torch.empty(t.numel() + 1, dtype=t.dtype, device=t.device)
    v = buf[1:].view(t.shape)
    v.copy_(t)
    assert v.is_contiguous() and v.data_ptr() % 16 != 0
    return v


def everything(dp, precision, rhs, ge, gf):
    s = bd.Solver(dp, precision=precision, rhs=rhs, record_cap=64,
                  ckpt_every=2)
    s.solve()
    n = sum(dp[k].numel() for k in PARAMS)
    out = [s.y_final, s.y_eval, *s.backward(ge, gf, n),
           *s.cadjoint(ge, gf, n, False)]
    out = [t.cpu().numpy() for t in out]
    s.close()
    return out


@pytest.mark.parametrize("precision", ["fp32", "bf16", "fp64"])
@pytest.mark.parametrize("field,d", [("mlp", 16), ("cnf", 48), ("cnf", 16)])
def test_shifted_inputs(field, d, precision):
    print(f"{precision} {field} d={d} shifted inputs", flush=True)
    p, rhs = ((W.neural_ode_fit(B=21, d=d, hidden=64, n_times=3), bd.RHS_MLP)
              if field == "mlp" else
              (W.cnf_density(B=21, d=d, hidden=64), bd.RHS_CNF))
    dp = bd.device_problem(p, precision)
    rng = np.random.default_rng(2)
    B, D = p["y0"].shape
    E = p["t_eval"].shape[1]
    g = lambda *n: torch.as_tensor(rng.standard_normal(n), device="cuda").to(
        dp["y0"].dtype)
    ge, gf = (g(B, E, D) if E else None), g(B, D)
    a = everything(dp, precision, rhs, ge, gf)
    q = {k: shifted(v) if k in PARAMS + ("y0", "eps") else v
         for k, v in dp.items()}
    b = everything(q, precision, rhs, None if ge is None else shifted(ge),
                   shifted(gf))
    for x, y in zip(a, b):
        np.testing.assert_array_equal(x, y)
