"""The bucketed ranking of the overlap partition at the edges of its range and of its bucket counts, bit for bit."""
import numpy as np
import pytest

from oracle import dw_data as OD
from paper_2409_09242_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,o,k", [
    (2047, 5, 3),                    # the last size that compares every pair
    (2048, 0, 2), (2049, 2049, 1),   # the first ones with buckets, 1024 of them
    (32767, 100, 7), (32768, 0, 64), # 1024 buckets, then 2048
    (1 << 17, 1000, 5),              # the largest set of the form with a fixed scratch array
    (1 << 21, 12345, 16),            # DW_MAX_POINTS
])
def test_bucketed_partition_matches_the_oracle(n, o, k):
    print("bucketed partition", n, o, k, flush=True)
    for seed in (3, (1 << 63) + n):
        got = B.overlap_partition(n, o, k, seed, "cuda:0").cpu().numpy()
        np.testing.assert_array_equal(got, OD.worker_datasets(n, o, k, seed))
