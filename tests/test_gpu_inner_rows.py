"""GPU parity: the inner solvers with the operator's rows in registers, at row counts around
what one workgroup keeps (16), and the streaming form where they do not fit."""
import numpy as np
import pytest

import workloads as W
from oracle import sketches, solver as O
from gpu_common import announce, rel, requires_gpu, to_dev, torch

pytestmark = [pytest.mark.gpu, requires_gpu]


@pytest.mark.parametrize("inner", ["cg", "aab"])
@pytest.mark.parametrize("prec", ["plain", "mixed"])
@pytest.mark.parametrize("n,d,m", [(40, 3, 2), (200, 17, 16), (600, 300, 17), (900, 257, 129),
                                   (1500, 700, 320), (2600, 1025, 515), (300, 40, 5000)])
def test_streaming_operators_follow_oracle(n, d, m, prec, inner):
    """m < d streams SA (CG and AAb_Solver); m = 5000 rows over 300 rows' worth of
    workgroups do not fit registers and, for AAb, stream through memory.  Three fixed outer
    steps at an inner tolerance of 1e-12: both sides end within a few times that tolerance
    of the exact sub-solution, times the sub-problem's condition ||M||/lam <= 1 + m_max
    sigma^2 / lam, kept below 1e3 by the flat spectrum."""
    import paper_1912_03514_amd as mihs
    P = W.make_problem(n, d, W.sigma_profile("exp", d, 1.0), d / 2, n + m)
    SA = sketches.gaussian_sketch(P.A, m, 5)
    sa = SA.astype(np.float32) if prec == "mixed" else SA
    a, b = O.momentum_cor4(min(d / 2, 0.5 * m), m)
    ref = O.mihs(P.A, P.b, P.lam, sa.astype(np.float64), a, b, inner=inner, eps_sub=1e-12,
                 n_iter=3, max_inner=8 * d)
    announce(f"inner rows {inner} {prec} n={n} d={d} m={m}")
    x, info = mihs.mihs_solve(to_dev(P.A), to_dev(P.b), P.lam, to_dev(sa), a, b, eps_sub=1e-12,
                              tol=0.0, max_outer=3, max_inner=8 * d, precision=prec, inner=inner)
    assert info["outer_iters"] == 3
    assert rel(x.cpu().numpy(), ref.x) <= 1e-8
