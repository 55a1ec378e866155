"""GPU parity: the block kernel's pass over A at the widths of its classes, where every column
of the class is used and no product is conditional, and one column below them."""
import numpy as np
import pytest

import workloads as W
from oracle import sketches, solver as O
from gpu_common import announce, rel, requires_gpu, to_dev, torch

pytestmark = [pytest.mark.gpu, requires_gpu]


@pytest.mark.parametrize("adt", [np.float64, np.float32])
@pytest.mark.parametrize("d", [63, 64, 127, 128, 255, 256, 511, 512, 1023, 1024])
def test_block_pass_at_class_widths(d, adt):
    """Four fixed outer steps of one problem with 11 lambdas, rows of A no multiple of a
    tile, inner solves to 1e-12: device and oracle both end within a few times that tolerance
    of the exact sub-solution, times the condition (H + lam I) / lam < 1e3."""
    import paper_1912_03514_amd as mihs
    n = 2 * d + 37
    P = W.make_problem(n, d, W.sigma_profile("exp", d, 1.0), d / 2, d)
    A64 = P.A.astype(adt).astype(np.float64)
    m = 2 * d
    SA = sketches.gaussian_sketch(A64, m, 5)
    lams = P.lam * 10.0 ** np.linspace(0, 1, 11)
    a, b = O.momentum_cor4(d / 2, m)
    ld = (d + 3) // 4 * 4
    A = torch.zeros((n, ld), dtype=getattr(torch, np.dtype(adt).name), device="cuda")[:, :d]
    A.copy_(to_dev(P.A.astype(adt)))
    b_dev, S = to_dev(P.b), to_dev(SA)
    announce(f"block width d={d} {np.dtype(adt).name}")
    if adt is np.float64:
        T = lambda v: to_dev(np.full((1, 11), v))
        s = mihs.BatchedSolver([(A, b_dev, S)], to_dev(lams[None]), T(a), T(b),
                               eps_sub=1e-12, tol=0.0, max_outer=4, max_inner=3 * d,
                               tuning=dict(cg_cols=64, a_dma=1, inner_weight=100.0))
        s.run()
        torch.cuda.synchronize()
        X = s.xs[0].cpu().numpy()
        s.close()
    else:  # a batch takes float64 A: right-hand sides b, 2 b, ... and one lambda
        lams[:] = lams[5]
        B = b_dev[:, None] * torch.arange(1, 12, device="cuda", dtype=torch.float64)
        X, _ = mihs.mihs_solve_multi(A, B, float(lams[0]), S, a, b, eps_sub=1e-12, tol=0.0,
                                     max_outer=4, max_inner=3 * d)
        X = X.cpu().numpy() / np.arange(1, 12)
    for j in (0, 5, 10):
        ref = O.mihs(A64, P.b, float(lams[j]), SA, a, b, inner="cg", eps_sub=1e-12, n_iter=4,
                     max_inner=3 * d)
        assert rel(X[:, j], ref.x) <= 1e-8, j
