"""Where the split-reduction kernel's range ends for middling reductions: the last size inside and the first outside (the
helper asserts which kernel runs), against the CPU oracle with its bound."""
import pytest

import test_gpu_small_problems as layers
from test_gpu_parity import torch_mod  # noqa: F401

pytestmark = pytest.mark.gpu

CASES = [
    # name                N  H   W   Cin Cout R st relu  res
    ("three_steps",       1, 32, 64, 192, 512, 1, 1, True, True),       # 64 x 16 tiles
    ("past_three_steps",  1, 32, 65, 192, 512, 1, 1, True, True, {"bf16": "conv_igemm bf16"}),       # 65 x 16
    ("seven_steps",       1, 32, 64, 448, 512, 1, 1, False, True),
    ("past_seven_steps",  1, 32, 65, 448, 512, 1, 1, True, False, {"bf16": "conv_igemm bf16"}),
    ("eight_steps",       1, 32, 32, 512, 512, 1, 1, True, True),       # 32 x 16
    ("past_eight_steps",  1, 33, 31, 512, 520, 1, 1, True, False, {"bf16": "gemm_nt bf16 128x128, four slice buffers"}),      # 32 x 17: 1023 pixels, 520 channels
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_lines_match_oracle(torch_mod, case):  # noqa: F811
    layers.test_few_tile_layers_match_oracle(torch_mod, "bf16", case)
