"""The fp32 input gradient where four waves do not share the output channels: the layers of test_gpu_backward_dgrad.py with as many samples
as make more tiles than two per compute unit."""
import pytest

from paper_2603_13810_amd import api
from test_gpu_backward_dgrad import BITS, MAX, MEAN, test_input_gradient as check_input_gradient

pytestmark = pytest.mark.gpu

CASES = [
    (40, 37, 21, 9, 11, BITS, False, 3, 7),     # weights not readable 16 bytes at a time, two channel blocks
    (30, 130, 9, 6, 70, BITS, True, 2, 3),      # two row segments, rounds of eight with a rest of one
    (60, 72, 40, 16, 16, BITS, True, 4, 6),
    (128, 32, 64, 14, 14, MEAN, False, 4, 7),
    (100, 20, 16, 5, 40, MAX, False, 2, 3),
    (16, 64, 8, 33, 20, BITS, False, 1, 2),     # strips with a remainder
    (700, 40, 12, 4, 4, BITS, True, 4, 8),      # several samples per tile, the last tile partly filled
]


@pytest.mark.parametrize("case", CASES, ids=["%d_to_%d_%dx%d_f%d" % c[1:6] for c in CASES])
def test_input_gradient_of_many_tiles(case):
    check_input_gradient(case)
