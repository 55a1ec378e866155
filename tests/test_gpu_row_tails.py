"""Rows that end inside a 16-byte chunk: what lies in the padding of A and SA never reaches the
result, whatever it is."""
import numpy as np
import pytest

import workloads as W
from gpu_common import announce, requires_gpu, torch

pytestmark = [pytest.mark.gpu, requires_gpu]


def _padded(X, dt, fill):
    n, d = X.shape
    buf = torch.full((n, (d + 3) // 4 * 4 + 4), fill, dtype=dt, device="cuda")[:, :d]
    buf.copy_(torch.from_numpy(X))
    return buf


@pytest.mark.parametrize("n,d,m", [(131, 61, 40), (999, 67, 80), (1500, 259, 100),
                                   (2100, 1021, 600), (2101, 2047, 2100), (3103, 3001, 700),
                                   (4201, 3001, 3100)])
@pytest.mark.parametrize("inner", ["cg", "aab"])
def test_padding_does_not_matter(n, d, m, inner):
    """NaN and zero padding give the same bits, in every width of the row loops, rows left over
    from the groups of a wave, FP64 and FP32 A and SA, Gram and streaming operators."""
    import paper_1912_03514_amd as mihs
    rng = np.random.default_rng(n)
    sig = W.sigma_profile("exp", d, 6.0)
    A = rng.standard_normal((n, d)) * sig / np.sqrt(n)
    SA = rng.standard_normal((m, d)) * sig / np.sqrt(m)
    b = torch.from_numpy(rng.standard_normal(n)).cuda()
    for adt in (torch.float64, torch.float32):
        for sdt in (torch.float64, torch.float32):
            announce(f"row tails n={n} d={d} m={m} {inner} A {adt} SA {sdt}")
            x = [mihs.mihs_solve(_padded(A, adt, f), b, 1e-2, _padded(SA, sdt, f), 0.5, 0.25,
                                 eps_sub=0.1, tol=0.0, max_outer=3, max_inner=20, inner=inner)[0]
                 for f in (0.0, float("nan"))]
            assert torch.isfinite(x[0]).all()
            assert torch.equal(x[0], x[1])
