"""Primal-Dual solves whose first sketch has more rows than the outer variable has entries
(m1 > cols): the dual steps then run on a matrix Q with fewer rows than columns, and the CG's
Gram matrix needs more workgroups than the rows of Q give."""
import numpy as np
import pytest

import workloads as W
from oracle import sketches, solver as O
from gpu_common import announce, rel, requires_gpu, to_dev

pytestmark = [pytest.mark.gpu, requires_gpu]


@pytest.mark.parametrize("prec", ["plain", "mixed"])
@pytest.mark.parametrize("rows,cols,m", [(500, 96, 97), (512, 100, 200), (700, 300, 1100)])
def test_more_sketch_rows_than_columns_reach_closed_form(rows, cols, m, prec):
    """m1 = m2 = m, CG on the Gram matrix of WQ, the stop rule at 1e-11: both algorithms are
    within 1e-10 of the closed form (the bound of the ordinary shapes)."""
    import paper_1912_03514_amd as mihs
    sd = 16.0
    P = W.make_problem(rows, cols, W.sigma_profile("exp", cols, 10.0), sd, seed=rows)
    SA = sketches.gaussian_sketch(P.A, m, 5)                  # S A: m x cols
    WQ = sketches.gaussian_sketch(SA.T.copy(), m, 6)
    a, b = O.momentum_cor4(sd, m)
    cast = (lambda X: X) if prec == "plain" else (lambda X: X.astype(np.float32))
    # (the entry points take rows on 16-byte boundaries)
    al = mihs._binding._row_aligned
    A, Q, Wq = to_dev(P.A), al(to_dev(cast(SA.T.copy()))), al(to_dev(cast(WQ)))
    kw = dict(M=10, eps_sub=0.1, tol=1e-11, max_outer=200, precision=prec, inner="cg")
    announce(f"pd rows={rows} cols={cols} m={m} {prec}")
    x, info = mihs.mihs_solve_pd(A, to_dev(P.b), P.lam, Q, Wq, a, b, a, b, **kw)
    assert info["status"] == 0, info
    assert rel(x.cpu().numpy(), O.ridge_lstsq(P.A, P.b, P.lam)) <= 1e-10
    bw = np.random.default_rng(5).standard_normal(cols)       # P.A = A^T, A is cols x rows
    announce(f"pd dual n={cols} d={rows} m={m} {prec}")
    x2, _, info2 = mihs.mihs_solve_pd_dual(A, to_dev(bw), P.lam, Q, Wq, a, b, a, b, **kw)
    assert info2["status"] == 0, info2
    assert rel(x2.cpu().numpy(), O.ridge_lstsq(P.A.T.copy(), bw, P.lam)) <= 1e-10
