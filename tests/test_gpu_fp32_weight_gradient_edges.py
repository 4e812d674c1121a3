"""The fp32 weight gradient where its positions wrap: images smaller than a step of four positions, runs that end inside a
round of loads, a wavefront without any.  Reference and bound as in the helper."""
import pytest

import test_gpu_small_problems as layers
from test_gpu_parity import torch_mod  # noqa: F401

pytestmark = pytest.mark.gpu

CASES = [
    # name          N  H     W  Cin Cout R
    ("one_pixel",   6, 1,    1,  32,  16, 3),      # four images to a step
    ("row_of_two",  5, 1,    2,  32,  48, 3),
    ("2x2",         5, 2,    2,  32,  16, 3),      # a step is an image
    ("3x3",         4, 3,    3,  32,  16, 3),
    ("2x5",         3, 2,    5,  32,  16, 3),
    ("rounds",      3, 33,  31,  32,  16, 3),      # 192 positions to a wavefront, the last has 189
    ("plain",       1, 1031, 1,  32,  48, 1),      # 68 to a wavefront: one round and one step; the last has 11
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: c[0])
def test_positions_wrap(torch_mod, case):  # noqa: F811
    layers.test_fp32_weight_gradient_matches_float64(torch_mod, case)
