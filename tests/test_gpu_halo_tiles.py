"""The 3x3 layers that keep their input halo in LDS, at both tile heights and every width at which the rule or the number
of halo loads changes, against the CPU oracle with the bound derived beside the helper, which also asserts the kernel."""
import pytest

import test_gpu_small_problems as layers
from test_gpu_parity import torch_mod  # noqa: F401

pytestmark = pytest.mark.gpu

HIGH, LOW = {"bf16": "conv3x3_halo bf16 256x64"}, {"bf16": "conv3x3_halo bf16 128x64"}
CASES = [
    # name           N  H    W   Cin Cout R st relu  res
    ("past_256_w31",      1, 133, 31,  64, 512, 3, 1, True, False, HIGH),      # 17 x 8 workgroups of 256 pixels, the last with 27
    ("past_256_w32",      2, 64,  32, 128, 512, 3, 1, False, True, HIGH),      # 16 x 8: the first that takes 256; two channel blocks
    ("past_256_w63",      1, 66,  63,  64, 512, 3, 1, True, True, HIGH),
    ("past_128_w31",      1, 83,  31,  64, 256, 3, 1, True, True, LOW),       # 21 x 4 workgroups of 128 pixels
    ("past_128_w32",      9, 9,   32, 128, 256, 3, 1, True, False, LOW),
    ("past_128_w63",      1, 41,  63,  64, 256, 3, 1, False, False, LOW),
    # past a whole round of the chip the last tiles go out in pieces of 32, 64 and 128 pixels
    ("pieces_32_w31",     1, 273, 31,  64, 512, 3, 1, True, True, HIGH),      # 34 x 8 workgroups: 16 tiles, half of them with 15 pixels
    ("pieces_32_w62",     1, 146, 62, 128, 512, 3, 1, False, False, HIGH),    # 36 x 8: 32 tiles in eight pieces, the most
    ("pieces_64_w63",     1, 159, 63,  64, 512, 3, 1, True, False, HIGH),     # 40 x 8: 64 tiles in four
    ("pieces_128_w33",    2, 184, 33,  64, 512, 3, 1, True, True, HIGH),      # 48 x 8: 128 tiles in two
    ("whole_again_w33",   1, 373, 33,  64, 512, 3, 1, True, False, HIGH),     # 49 x 8: 136 tiles, whole
    ("past_wide_w64",     1, 65,  64,  64, 512, 3, 1, True, False, LOW),      # enough pixels for 256, rows too long for it
    ("past_wide_w127",    1, 33, 127,  64, 512, 3, 1, True, True, LOW),       # the longest halo
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_halo_tiles_match_oracle(torch_mod, case):  # noqa: F811
    layers.test_few_tile_layers_match_oracle(torch_mod, "bf16", case)
