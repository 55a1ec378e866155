"""GPU parity: CountSketch over the lengths of its row lists and the widths of its column
blocks."""
import numpy as np
import pytest

from oracle import sketches
from gpu_common import announce, requires_gpu, to_dev, torch

pytestmark = [pytest.mark.gpu, requires_gpu]


@pytest.mark.parametrize("adt,prec", [(np.float64, "plain"), (np.float32, "plain"),
                                      (np.float32, "mixed")])
@pytest.mark.parametrize("n,d,m", [(5, 1, 4096), (511, 513, 1), (513, 1025, 1), (4000, 3, 5),
                                   (7168, 2, 1), (7169, 2, 1), (60000, 5, 8), (20000, 1030, 2)])
def test_row_lists_bit_exact(n, d, m, adt, prec):
    """Lists sorted by rank (up to 512 rows), by the bitonic network, and buckets whose rows
    are found by hashing (above 7168 rows on average): every bucket sums its rows in ascending
    order, in the result's precision, like the oracle's loop, so the results are the same
    bits."""
    import paper_1912_03514_amd as mihs
    A = np.random.default_rng(n).standard_normal((n, d)).astype(adt)
    bucket, sign = sketches.countsketch_hash(n, m, 99)
    ref = np.zeros((m, d), dtype=np.float64 if prec == "plain" else np.float32)
    np.add.at(ref, bucket, sign.astype(ref.dtype)[:, None] * A.astype(ref.dtype))
    announce(f"countsketch lists n={n} d={d} m={m} {np.dtype(adt).name} {prec}")
    SA = mihs.mihs_sketch(to_dev(A), "countsketch", m, 99, precision=prec)
    assert np.array_equal(SA.cpu().numpy(), ref)
