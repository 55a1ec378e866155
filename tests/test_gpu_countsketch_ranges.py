"""GPU parity: CountSketch of so many rows per bucket that its row lists go by ranges of rows."""
import numpy as np
import pytest

from oracle import sketches
from gpu_common import announce, requires_gpu, to_dev

pytestmark = [pytest.mark.gpu, requires_gpu]


@pytest.mark.parametrize("adt,prec", [(np.float64, "plain"), (np.float32, "mixed")])
@pytest.mark.parametrize("n,d,m", [(716800, 3, 100), (716801, 3, 100), (1500001, 2, 103),
                                   (720000, 3, 99)])
def test_ranges_bit_exact(n, d, m, adt, prec):
    """7168 rows per bucket (one range), one row more (two), 14563 (three), and fewer than 100
    buckets (by hashing): a bucket's rows are summed in ascending order whatever the split, so
    the results are the same bits as the oracle's loop."""
    import paper_1912_03514_amd as mihs
    A = np.random.default_rng(n).standard_normal((n, d)).astype(adt)
    bucket, sign = sketches.countsketch_hash(n, m, 99)
    ref = np.zeros((m, d), dtype=np.float64 if prec == "plain" else np.float32)
    np.add.at(ref, bucket, sign.astype(ref.dtype)[:, None] * A.astype(ref.dtype))
    announce(f"countsketch ranges n={n} d={d} m={m} {np.dtype(adt).name} {prec}")
    SA = mihs.mihs_sketch(to_dev(A), "countsketch", m, 99, precision=prec)
    assert np.array_equal(SA.cpu().numpy(), ref)


def test_workspace_is_proportional_to_the_rows():
    """Few rows per bucket take few slots (16 at one row per bucket on average), many rows per
    bucket little more than a slot each."""
    import paper_1912_03514_amd as mihs
    n = 1 << 20
    assert mihs.sketch_workspace_bytes(n, 16, n, "countsketch") <= 4 * n * (16 + 1) + 512
    assert mihs.sketch_workspace_bytes(1 << 27, 16, 1 << 13, "countsketch") <= 4 * 1.1 * (1 << 27)
