"""GPU parity: the block kernel's team CG over the shapes of its sub-team: a member per 64
rows of H, two waves per block (a member per 32 rows), rows of H through the ring, and
1024-wide rows."""
import numpy as np
import pytest

import workloads as W
from oracle import sketches, solver as O
from gpu_common import announce, rel, requires_gpu, to_dev, torch

pytestmark = [pytest.mark.gpu, requires_gpu]


@pytest.mark.parametrize("sdt", [np.float64, np.float32])
@pytest.mark.parametrize("d", [33, 64, 65, 130, 257, 500, 700, 1000])
@pytest.mark.parametrize("cg_cols", [16, 64, 128])
def test_team_cg_follows_oracle(d, cg_cols, sdt):
    """One problem with 16 right-hand sides' worth of lambdas on a large team; cg_cols sets
    the sub-team: d / 16 members (two waves per block; at most d / 32 take part), d / 64
    (one per 64 rows) and d / 128 (two quads per member through the ring).  Four fixed
    outer steps with inner solves to 1e-12 follow the oracle's: both end within a few times
    that tolerance of the exact sub-solution, times the condition (H + lam I) / lam < 1e3."""
    import paper_1912_03514_amd as mihs
    n = 4 * d + 37
    P = W.make_problem(n, d, W.sigma_profile("exp", d, 1.0), d / 2, d)
    m = 2 * d
    SA = sketches.gaussian_sketch(P.A, m, 3).astype(sdt)
    lams = P.lam * 10.0 ** np.linspace(0, 1, 16)
    a, b = O.momentum_cor4(d / 2, m)
    ld = (d + 1) // 2 * 2
    A = torch.zeros((n, ld), dtype=torch.float64, device="cuda")[:, :d]
    A.copy_(to_dev(P.A))
    T = lambda v: to_dev(np.full((1, 16), v))
    announce(f"team cg d={d} cols={cg_cols} {np.dtype(sdt).name}")
    s = mihs.BatchedSolver([(A, to_dev(P.b), to_dev(SA))], to_dev(lams[None]), T(a), T(b),
                           eps_sub=1e-12, tol=0.0, max_outer=4, max_inner=3 * d,
                           tuning=dict(cg_cols=cg_cols, a_dma=1, inner_weight=100.0))
    s.run()
    torch.cuda.synchronize()
    X = s.xs[0].cpu().numpy()
    s.close()
    for j in (0, 7, 15):
        ref = O.mihs(P.A, P.b, float(lams[j]), SA.astype(np.float64), a, b, inner="cg",
                     eps_sub=1e-12, n_iter=4, max_inner=3 * d)
        assert rel(X[:, j], ref.x) <= 1e-8, j
