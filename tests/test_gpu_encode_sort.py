"""The counting sort of the bulk insert: lists that are put in place in LDS and lists that are too long for it, on both sides of
the line, slot numbers of every width that has all bits set, groups of four 64-token chunks that end anywhere, tokens of a bad
source row.  Bit for bit against the oracle's sequential sum, which any other order of a slot's tokens fails."""
import numpy as np
import pytest
import torch

from tests.test_gpu_parity import kvr, run_encode_case, say  # noqa: F401

pytestmark = pytest.mark.gpu
LDS_INTS = 160 * 1024 // 4


@pytest.mark.parametrize("w,cap,counts", [
    (1, 65, [[65, 64, 1]]),
    (3, 5000, [[4096, 4097, 63]]),               # one group of four chunks per wave, and one token more
    (511, 1300, [[1300, 0]]),
    (512, 1300, [[1299, 1]]),
    (29, LDS_INTS - 17 * 29 - 1, [[300, 2]]),    # the longest list that LDS holds
    (29, LDS_INTS - 17 * 29, [[300, 2]]),
    (8191, LDS_INTS - 2 * 8191 - 1, [[700]]),    # one wave
    (8192, LDS_INTS - 2 * 8192, [[700]]),
])
def test_sorted_lists(kvr, w, cap, counts):  # noqa: F811
    say("encode sort", w, cap)
    run_encode_case(kvr, torch.bfloat16, 3, w, cap, np.array(counts), 40, 2, 31 + w, bad_slot=max(counts[0]) > 100)
