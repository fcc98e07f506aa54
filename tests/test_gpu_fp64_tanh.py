"""FP64 fields whose hidden units run through the whole range of tanh, from
the linear part to saturation, against the FP64 oracle at the bars of every
FP64 check (identical counts, 1e-9)."""
import numpy as np
import pytest

import oracle
from gpu_helpers import assert_fp64_parity, run_gpu
from paper_2210_12375_amd import binding as bd
from paper_2210_12375_amd import workloads as W

pytestmark = pytest.mark.gpu

# With first-layer gains up to 1e4 the field is close to a step function and
# the solve amplifies the last bits of any FP64 evaluation: the math
# library's tanh differs from the oracle there as well (2 of 9 instances in
# their counts, y by 5e-5), so the oracle says nothing about this range.
STEEP = pytest.mark.skip(reason="ill-conditioned: rounding alone changes the "
                                "accepted steps, also with the library's tanh")


@pytest.mark.parametrize("lo,hi", [(-12, -8), (-3, -0.5), (-0.5, 0.7),
                                   (0.7, 1.5),
                                   pytest.param(1.5, 4, marks=STEEP)])
def test_ranges(lo, hi):
    print(f"fp64 tanh arguments 1e{lo} .. 1e{hi}", flush=True)
    p = W.neural_ode(B=9, d=6, hidden=40)
    q = dict(p["mlp"])
    # columns of the first layer scaled over the decades; the second layer's
    # arguments are then of order one, and the field's output bounded
    q["W1"] = np.array(q["W1"]) * np.logspace(lo, hi, 40)[None, :]
    p["mlp"] = q
    g, _ = run_gpu(p, method="dopri5", rhs=bd.RHS_MLP)
    assert_fp64_parity(g, oracle.solve(p, method="dopri5"))
