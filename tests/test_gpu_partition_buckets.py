"""The overlap partition at sizes of the two-launch form inside its range, and of the five-launch form at the edges of its bucket counts,
bit for bit."""
import numpy as np
import pytest

from oracle import dw_data as OD
from paper_2409_09242_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,o,k", [
    (2047, 5, 3), (2048, 0, 2), (2049, 2049, 1),          # two launches: 64 buckets, then 128
    (32767, 100, 7), (32768, 0, 64),                      # 1024 buckets, then 2048
    (1 << 17, 1000, 5),                                   # the largest set of the form with a fixed scratch array
    ((1 << 18) + 1, 99, 4),                               # five launches from here on: 2^14 buckets
    ((1 << 19) - 1, 0, 8), (1 << 19, 7777, 3),            # and 2^15
    ((1 << 20) - 1, 1 << 19, 2), (1 << 20, 0, 16),        # and 2^16
    (1 << 21, 12345, 16),                                 # DW_MAX_POINTS
])
def test_bucketed_partition_matches_the_oracle(n, o, k):
    print("bucketed partition", n, o, k, flush=True)
    for seed in (3, (1 << 63) + n):
        got = B.overlap_partition(n, o, k, seed, "cuda:0").cpu().numpy()
        np.testing.assert_array_equal(got, OD.worker_datasets(n, o, k, seed))
