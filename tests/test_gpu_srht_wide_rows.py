"""GPU parity: the one-read SRHT of matrices whose rows are so long that a block of rows spans
2 GiB and more (a few columns of a wide matrix): the workspace query does not know the row
stride, and what it answers has to do for them."""
import math

import numpy as np
import pytest

from oracle import sketches
from gpu_common import announce, requires_gpu, to_dev, torch

pytestmark = [pytest.mark.gpu, requires_gpu]


@pytest.mark.parametrize("adt,prec,log_ld", [(np.float64, "mixed", 18), (np.float32, "mixed", 19),
                                             (np.float64, "plain", 19)])
@pytest.mark.parametrize("m", [100, 2100])
def test_rows_of_two_mebibytes(adt, prec, log_ld, m):
    """37 columns of 2048 rows, row stride 2 or 4 MiB (1024 rows per block in FP32, 512 in FP64);
    m on both sides of 2048 (two-stage above it in FP64).  Bound as for the other SRHT tests."""
    import paper_1912_03514_amd as mihs
    n, d = 2048, 37
    A = np.random.default_rng(m).standard_normal((n, d)).astype(adt)
    ref = sketches.srht_sketch(A, m, 17)
    wide = torch.empty((n, 1 << log_ld), dtype=to_dev(A).dtype, device="cuda")[:, :d]
    wide.copy_(to_dev(A))
    announce(f"srht rows of {A.itemsize << log_ld} bytes, m={m} {prec}")
    SA = mihs.mihs_sketch(wide, "srht", m, 17, precision=prec).double().cpu().numpy()
    u = 2.0 ** -52 if prec == "plain" else 2.0 ** -23
    bound = 4 * math.log2(n) * u * np.abs(A).astype(np.float64).sum(axis=0).max() / math.sqrt(m)
    assert np.max(np.abs(SA - ref)) <= bound
