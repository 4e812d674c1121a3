"""The data gradient of 3x3 stride-2 layers against float64 on the stored operands, at the edges of the one-launch kernel's
tiles and on both sides of each line of its rule; every case names the kernel it expects.

Tolerance: products of two bf16 values are exact in fp32 and at most 4 x 512 of them are summed, with one rounding to bf16
at the end: 2^-8 of the value and 1e-6 of the largest entry."""
import numpy as np
import pytest

import synth
from oracle import numeric as on
from test_gpu_backward import _bits, _dev, _small_ctx, torch_mod  # noqa: F401

pytestmark = pytest.mark.gpu

ONE, TILED, SPLIT = "dgrad3x3_s2", "four classes, conv_igemm", "four classes, conv_splitk"
CASES = [
    # N  H   W  Cin  Cout add mask (kernel, where it is not the one launch)
    (1, 1, 1, 128, 64, 0, 0),          # one pixel, one chunk; no odd row or column
    (1, 2, 2, 128, 64, 1, 1),
    (1, 16, 16, 128, 128, 0, 1),       # exactly one tile of 64 gradient pixels
    (1, 15, 26, 256, 64, 1, 0),        # 104: a full tile and one of 40; odd height; two channel tiles
    (5, 7, 7, 128, 192, 1, 1),         # several images to a tile; odd both ways
    (3, 3, 62, 128, 128, 0, 1),        # 31 columns: the last width with 96 staged rows
    (2, 5, 64, 128, 64, 0, 0),         # 32 columns: 128 staged rows, one workgroup to a CU
    (1, 4, 318, 128, 128, 0, 1),       # 159 columns: the widest it takes
    (1, 4, 320, 128, 64, 0, 1, SPLIT), # one more: class by class
    (2, 9, 8, 64, 128, 1, 1, SPLIT),   # channels not a multiple of 128: class by class
    (2, 13, 20, 128, 256, 1, 1),       # four chunks: the two row buffers and the ring of weights wrap
    (1, 14, 14, 256, 384, 0, 1),       # six; the last count taken with few tiles
    (1, 14, 14, 128, 448, 0, 1, SPLIT),
    (13, 28, 28, 128, 512, 1, 1),      # eight chunks, 40 tiles: the first that takes them
    (12, 28, 28, 128, 512, 0, 0, SPLIT),   # 37 tiles
    (11, 64, 64, 64, 128, 0, 1, TILED),    # class by class with more tiles than the split kernel takes
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "%dx%dx%d_%d_%d_a%d_m%d" % c[:7])
def test_strided_data_gradient_matches_float64(torch_mod, case):  # noqa: F811
    torch = torch_mod
    import paper_2203_15980_amd as dl
    N, H, W, Cin, Cout, add, mask = case[:7]
    print("case", case, flush=True)
    P, Q = (H - 1) // 2 + 1, (W - 1) // 2 + 1
    x, gy, res = _bits(98, 1, (N, H, W, Cin)), _bits(98, 2, (N, P, Q, Cout)), _bits(98, 3, (N, H, W, Cin))
    wt = _bits(98, 4, (Cin, 3, 3, Cout), 0.1)                    # as prepared for the data gradient: taps flipped
    d, put, get = _small_ctx(torch, [x.nbytes, gy.nbytes, gy.nbytes, x.nbytes, x.nbytes])
    put(0, x)
    put(2, gy)
    put(4, res)
    w, one = torch.zeros(Cout * 9 * Cin, dtype=torch.bfloat16, device="cuda:0"), torch.ones(Cout, device="cuda:0")
    wtd = _dev(torch, wt.view(np.uint8).reshape(-1))
    fwd = dl.LayerDesc(x=0, res=dl.NO_TENSOR, y=1, dtype=dl.DTYPE_BF16, w=w.data_ptr(), scale=one.data_ptr(), shift=one.data_ptr(), N=N, H=H, W=W,
                       Cin=Cin, Cout=Cout, R=3, S=3, stride=2, pad=1, relu=0)
    desc = dl.BwdDesc(fwd=fwd, gy=2, gpre=2, gx=3, gx_add=4 if add else dl.NO_TENSOR, mask_gx=mask, wt=wtd.data_ptr(), gw=None,
                      workspace=None, workspace_bytes=0)
    assert (case[7] if len(case) > 7 else ONE) in d.backward_kernel(desc), d.backward_kernel(desc)
    d.backward_segment([desc])
    d.sync()
    got = on.to_f64(get(3, x.shape), "bf16")
    d.close()
    wf, gf = on.to_f64(wt, "bf16"), on.to_f64(gy, "bf16")
    full = np.zeros((N, H + 2, W + 2, Cin))                      # the input with its padding
    for r in range(3):
        for s in range(3):
            full[:, r:r + 2 * P:2, s:s + 2 * Q:2] += gf @ wf[:, 2 - r, 2 - s].T
    ref = full[:, 1:H + 1, 1:W + 1] + (on.to_f64(res, "bf16") if add else 0.0)
    if mask:
        ref = np.where(on.to_f64(x, "bf16") > 0, ref, 0.0)
        assert np.all(got[ref == 0] == 0)
    err = np.abs(got - ref) - np.abs(ref) * 2.0 ** -8
    assert err.max() <= 1e-6 * np.abs(ref).max(), err.max()
