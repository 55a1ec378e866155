"""GPU parity: the FP64 matrix-core products (Gaussian sketch, A W, Gram matrices) and the
row products at tile edges, remainders and odd strides."""
import numpy as np
import pytest

import workloads as W
from oracle import sketches, solver as O
from gpu_common import announce, rel, requires_gpu, to_dev, torch

pytestmark = [pytest.mark.gpu, requires_gpu]

U = 2.0 ** -53


def _mihs():
    import paper_1912_03514_amd as mihs
    return mihs


@pytest.mark.parametrize("adt", [np.float64, np.float32])
@pytest.mark.parametrize("n,d,m", [(1, 1, 1), (15, 3, 2), (16, 64, 64), (17, 65, 63),
                                   (1500, 61, 200), (2049, 129, 65)])
def test_gaussian_plain_edges(n, d, m, adt):
    """Rows, columns and k around the 64-wide tiles and 16-deep steps, one split and
    several.  Any summation order of n products errs by at most n u |S||A|, the entries of
    S by a few u (Box-Muller in FP64, then the scale): 16 u covers them."""
    mihs = _mihs()
    A = np.random.default_rng(n + d).standard_normal((n, d)).astype(adt)
    S = sketches.gaussian_matrix(m, n, 5)
    announce(f"gaussian plain edges n={n} d={d} m={m} {np.dtype(adt).name}")
    got = mihs.mihs_sketch(to_dev(A), "gaussian", m, 5).cpu().numpy()
    A64 = A.astype(np.float64)
    bound = (n + 16) * U * (np.abs(S) @ np.abs(A64)) + 1e-300
    # the reference product rounds as well: twice the bound
    assert np.all(np.abs(got - S @ A64) <= 2 * bound)


@pytest.mark.parametrize("adt", [np.float64, np.float32])
@pytest.mark.parametrize("n,d,k", [(300, 5, 1), (1001, 130, 1), (1001, 130, 2), (700, 63, 3),
                                   (640, 64, 32), (700, 65, 33), (513, 100, 64), (300, 40, 65)])
def test_apply_rows_edges(n, d, k, adt):
    """dB = A W for one column (row products), up to 32 and more (64 x 32 and 64 x 64
    tiles), even and odd numbers of columns (aligned and unaligned rows of W)."""
    mihs = _mihs()
    P = W.make_problem(n, d, W.sigma_profile("exp", d, 2.0), d / 4, n + k, adt)
    SA = sketches.gaussian_sketch(P.A, 4 * d, 3)
    G = np.random.default_rng(k).standard_normal((d, k))
    announce(f"apply rows n={n} d={d} k={k} {np.dtype(adt).name}")
    a, b = O.momentum_cor4(d / 4, 4 * d)
    Wm, dB, _, _ = mihs.mihs_solve_backward(to_dev(P.A), to_dev(SA), P.lam, to_dev(G), to_dev(G),
                                            a, b, max_outer=3)
    A64, Wm, dB = P.A.astype(np.float64), Wm.cpu().numpy(), dB.cpu().numpy()
    assert np.any(Wm != 0)
    bound = 2 * (d + 2) * U * (np.abs(A64) @ np.abs(Wm)) + 1e-300
    assert np.all(np.abs(dB - A64 @ Wm) <= bound)


@pytest.mark.parametrize("sdt", [np.float64, np.float32])
@pytest.mark.parametrize("d,m", [(3, 17), (31, 33), (33, 40), (64, 64), (65, 100), (500, 515),
                                 (513, 530)])
def test_gram_edges(d, m, sdt):
    """The inner CG through the Gram matrix at sizes around its 32- and 64-wide blocks
    (blocks of padding among them): one step with an exact inner solve is
    x = alpha (H + lam I)^-1 A^T b.  H carries at most m u |M|^T |M| (FP32: its rounding
    2^-24 too), which the solve amplifies by at most ||H + lam I|| / lam."""
    mihs = _mihs()
    n = 2 * m
    P = W.make_problem(n, d, W.sigma_profile("exp", d, 1.0), d / 4, d)
    SA = sketches.gaussian_sketch(P.A, m, 9).astype(sdt)
    announce(f"gram edges d={d} m={m} {np.dtype(sdt).name}")
    x, info = mihs.mihs_solve(to_dev(P.A), to_dev(P.b), P.lam, to_dev(SA), 1.0, 0.0,
                              eps_sub=1e-13, tol=0.0, max_outer=1, max_inner=4 * d + 50)
    M = SA.astype(np.float64)
    H = M.T @ M + P.lam * np.eye(d)
    ref = np.linalg.solve(H, P.A.T @ P.b)
    kappa = np.linalg.norm(H, 2) / P.lam
    u = U if sdt == np.float64 else 2.0 ** -24
    assert rel(x.cpu().numpy(), ref) <= kappa * (1e-13 + (m + d) * U * np.sqrt(d) + u * np.sqrt(d))
