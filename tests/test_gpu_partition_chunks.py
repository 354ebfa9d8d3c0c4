"""The overlap partition at the edges of its chunks, of the sizes that one chunk size takes and of the two-launch form, bit for bit, and
with scratch of exactly the stated size."""
import ctypes

import numpy as np
import pytest
import torch

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


@pytest.mark.parametrize("n", [1, 1000, 1 << 16, (1 << 16) + 1, (1 << 18) + 1])
def test_nothing_is_written_beside_the_scratch_or_the_index(n):
    """Exactly the bytes that dw_partition_scratch_bytes states, between guard words, and so the index: the guards stay as they are.
    (n = 2^16 uses the scratch to its last byte.)"""
    print("partition guards", n, flush=True)
    o, k, seed, guard = n // 5, 3, 11, 4096
    m, nbytes = o + (n - o) // k, B.lib().dw_partition_scratch_bytes(n)
    scratch = torch.full((guard + nbytes + guard,), 0xA5, dtype=torch.uint8, device="cuda:0")
    index = torch.full((guard + k * m + guard,), -7, dtype=torch.int32, device="cuda:0")
    assert scratch.data_ptr() % 256 == 0
    s = B.lib().dw_overlap_partition(n, o, k, seed, ctypes.c_void_p(index.data_ptr() + 4 * guard), ctypes.c_void_p(scratch.data_ptr() + guard),
                                     nbytes, ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    torch.cuda.synchronize()
    assert s == (n - o) // k
    np.testing.assert_array_equal(index[guard:guard + k * m].cpu().numpy().reshape(k, m), OD.worker_datasets(n, o, k, seed))
    for edge in (scratch[:guard], scratch[guard + nbytes:]):
        assert bool((edge == 0xA5).all())
    for edge in (index[:guard], index[guard + k * m:]):
        assert bool((edge == -7).all())
