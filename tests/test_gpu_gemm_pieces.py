"""1x1 layers whose tiles exceed a whole round of the chip by a few, which go out in runs of 64 or 128 rows: against the CPU oracle with the bound
derived beside the helper, which also asserts the kernel.  The last tile holds a few rows, so that pieces of it hold none."""
import pytest

import test_gpu_small_problems as layers
from test_gpu_parity import torch_mod  # noqa: F401

pytestmark = pytest.mark.gpu

GEMM = "gemm_nt bf16 256x%d (64x64 per wave, direct-to-LDS), last tiles in %d pieces"
CASES = [
    # name           N  H    W   Cin Cout R st relu  res
    ("pieces_64",    1, 257, 257, 256, 256,  1, 1, True, True, {"bf16": GEMM % (256, 4)}),      # 259 tiles: 3 in four pieces, the last with one row
    ("pieces_128",   1, 149, 149, 256, 1024, 1, 1, True, False, {"bf16": GEMM % (256, 2)}),     # 87 x 4 tiles: 92 in two
    ("pieces_192",   1, 273, 31,  256, 2048, 1, 1, False, True, {"bf16": GEMM % (192, 2)}),     # 34 x 11, the last columns ragged: 118 in two
    ("strided",      2, 297, 223, 256, 1024, 1, 2, False, False, {"bf16": GEMM % (256, 4)}),    # 131 x 4 of 149 x 112 pixels twice: 12 in four
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_last_tiles_in_pieces_match_oracle(torch_mod, case):  # noqa: F811
    layers.test_few_tile_layers_match_oracle(torch_mod, "bf16", case)
