"""The overlap partition at the edges of its chunks, of the sizes that one chunk size takes and of the two-launch form, bit for bit."""
import numpy as np
import pytest

from oracle import dw_data as OD
from paper_2409_09242_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,o,k", [
    (1, 0, 1), (1, 1, 2), (31, 7, 3),
    (1023, 100, 4), (1024, 0, 64), (1025, 1025, 1),   # one chunk of 1024 points, then two
    (4095, 10, 5), (4096, 512, 7),                    # 32 buckets, then 64
    (1 << 16, 9000, 6), ((1 << 16) + 1, 3, 2),        # chunks of 1024, then of 4096 points
    (100003, 12500, 16),
    (1 << 18, 777, 9), ((1 << 18) + 1, 0, 3),         # two launches, then five
])
def test_partition_in_chunks_matches_the_oracle(n, o, k):
    print("partition in chunks", n, o, k, flush=True)
    for seed in (1, (1 << 62) + 3 * n):
        got = B.overlap_partition(n, o, k, seed, "cuda:0").cpu().numpy()
        np.testing.assert_array_equal(got, OD.worker_datasets(n, o, k, seed))
