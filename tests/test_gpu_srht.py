"""GPU parity: the one-read SRHT over the sample counts and column counts at which its
register and thread layout changes."""
import math

import numpy as np
import pytest

from oracle import sketches
from gpu_common import announce, requires_gpu, to_dev, torch

pytestmark = [pytest.mark.gpu, requires_gpu]


@pytest.mark.parametrize("adt", [np.float64, np.float32])
@pytest.mark.parametrize("prec", ["plain", "mixed"])
@pytest.mark.parametrize("n,d,m", [(1 << 10, 1, 1), (1 << 11, 15, 512), (1 << 12, 17, 513),
                                   (1 << 13, 33, 1025), (1 << 12, 16, 2048), (1 << 11, 18, 2049),
                                   (1 << 12, 35, 3073), (1 << 12, 5, 4096), (1 << 11, 7, 4097)])
def test_sample_counts(n, d, m, prec, adt):
    """m at the edges of 512, 1024, 2048, 3072 and 4096 samples per strip (the two-stage form
    above 2048 in FP64 and 4096 in FP32), d around the 16-column strips and the 2- and
    4-column threads.  The transform adds n terms in log2(n) levels and block sums: a few
    u log2(n) of sum |A| / sqrt(m), as in the other SRHT tests."""
    import paper_1912_03514_amd as mihs
    A = np.random.default_rng(n + m).standard_normal((n, d)).astype(adt)
    ref = sketches.srht_sketch(A, m, 31)
    announce(f"srht n={n} d={d} m={m} {prec} {np.dtype(adt).name}")
    SA = mihs.mihs_sketch(to_dev(A), "srht", m, 31, precision=prec).double().cpu().numpy()
    u = 2.0 ** -52 if prec == "plain" else 2.0 ** -23
    bound = 4 * math.log2(n) * u * np.abs(A).astype(np.float64).sum(axis=0).max() / math.sqrt(m)
    assert np.max(np.abs(SA - ref)) <= bound
