"""Retained slots ahead of the Vague list: on all CUs of the list's launch, where the list would leave them a few, and in a launch of
their own, where there are hardly any; and slices of as many slots as LDS holds.  (Which plan a size has is asked on the CPU,
tests/test_plan_cpu.py.)  Reference and tolerances of tests/test_gpu_pair.py."""
import pytest

from tests import test_gpu_pair as P
from tests.test_plan_cpu import SLOTS_AHEAD

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def kvr():
    from paper_2512_17917_amd import binding
    return binding


@pytest.mark.parametrize("units,G,r,w,ret_cap,cap,how", [c for c in SLOTS_AHEAD if c[1] < 8])
def test_staged_list(kvr, units, G, r, w, ret_cap, cap, how):
    P.test_rounds_and_slices(kvr, units, G, r, w, ret_cap, cap)


@pytest.mark.parametrize("units,G,n_q,w,ret_cap,cap", [(c[0], 8, 1, *c[3:6]) for c in SLOTS_AHEAD if c[1] == 8] + [
    (246, 4, 2, 21, 585, 1755),      # several queries: first, eight columns
    (246, 4, 4, 21, 585, 300),       # and 16
    (400, 1, 2, 1, 7, 220),          # a launch of their own, two columns
    (400, 4, 4, 1, 256, 220),        # 16, the longest slice
    (144, 8, 1, 341, 11000, 2800),   # more CUs for the slots than the list's turns leave, slices near what LDS holds
])
def test_streamed_list(kvr, units, G, n_q, w, ret_cap, cap):
    P.test_streamed_list(kvr, units, G, n_q, w, ret_cap, cap)
