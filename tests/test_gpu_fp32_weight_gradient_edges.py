"""The fp32 weight gradient where its positions wrap: images smaller than a step of four positions, runs that end inside a
round of loads, a wavefront without any.  Reference and bound as in the helper."""
import numpy as np
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


FORMS = [
    # N   H    W    Cin  Cout R stride kernel
    (2,  9,   7,   512, 512, 1, 1, "32x32, 32-bit offsets"),
    (2,  6,   5,   96,  256, 3, 1, "16x16, 32-bit offsets"),        # 216 tiles of 32 x 32: too few
    (2,  6,   5,   128, 256, 3, 1, "32x32, 32-bit offsets"),        # 288
    (1,  7,   7,   512, 512, 1, 1, "32x32, 32-bit offsets"),        # the last three wavefronts have no position
    (1,  33,  31,  512, 512, 1, 1, "32x32, 32-bit offsets"),        # 64 positions each, 63 the last: two rounds, one in each sum
    (1,  25,  41,  256, 1024, 1, 1, "32x32, 32-bit offsets"),       # 68, the last 5: three rounds, the first in its own sum; none for the last
    (1,  41,  53,  128, 256, 3, 1, "32x32, 32-bit offsets"),        # 136: two rounds of five, taps
    (3,  9,   7,   512, 512, 1, 2, "32x32, 64-bit addresses"),
    (2,  8,   11,  64,  48,  1, 3, "16x16, 64-bit addresses"),
    (33, 256, 256, 256, 16,  1, 1, "16x16, 64-bit addresses"),      # x of 2.06 GiB
    (33, 256, 256, 256, 16,  3, 1, "16x16, 64-bit addresses"),
    (33, 256, 256, 256, 128, 3, 1, "32x32, 64-bit addresses"),
]


@pytest.mark.parametrize("case", FORMS, ids=lambda c: "%dx%dx%d_%d_%d_r%d_s%d" % c[:7])
def test_every_form_matches_float64(torch_mod, case):  # noqa: F811
    """Each kernel that the fp32 weight gradient dispatches to, beyond 2 GiB included, against float64 on the GPU (plain products).
    A wavefront adds M / 16 products of unit variance one after the other: its k-th partial sum is about sqrt(k) and rounds by 2^-25 of that, so
    its error is about 2^-25 (M / 16) / sqrt(2); sixteen such errors give 4 times that, against a result of about sqrt(M): 2^-25 * 0.18
    sqrt(M), of which three times are allowed, and 1e-6 for the few roundings beside."""
    torch = torch_mod
    import paper_2203_15980_amd as dl
    N, H, W, Cin, Cout, R, stride, kernel = case
    print("case", case, flush=True)
    P, Q, pad = (H - 1) // stride + 1, (W - 1) // stride + 1, R // 2
    gen = torch.Generator(device="cuda:0").manual_seed(17)
    xbytes, ybytes = N * H * W * Cin * 4, N * P * Q * Cout * 4
    d = layers.make_delta(torch, xbytes + 2 * ybytes + (1 << 20))
    d.bind([xbytes, ybytes, ybytes])
    view = {}
    for t, n, shape in ((0, xbytes, (N, H, W, Cin)), (2, ybytes, (N, P, Q, Cout))):
        d.alloc(t)
        view[t] = d.arena[d.tensor_ptr(t) - d.arena.data_ptr():][:n].view(torch.float32).reshape(shape)
        view[t].normal_(generator=gen)
    scale, zeros = torch.rand(Cout, device="cuda:0", generator=gen) + 0.5, torch.zeros(Cout, device="cuda:0")
    w = torch.zeros(Cout * R * R * Cin, device="cuda:0")
    gw = torch.full((Cout, R, R, Cin), float("nan"), device="cuda:0")
    ws = torch.empty(256, dtype=torch.uint8, device="cuda:0")
    fwd = dl.LayerDesc(x=0, res=dl.NO_TENSOR, y=1, dtype=dl.DTYPE_F32, w=w.data_ptr(), scale=scale.data_ptr(), shift=zeros.data_ptr(), N=N, H=H,
                       W=W, Cin=Cin, Cout=Cout, R=R, S=R, stride=stride, pad=pad, relu=0)
    need = d.backward_workspace(fwd)
    if need > ws.numel():
        ws = torch.empty(need, dtype=torch.uint8, device="cuda:0")
    desc = dl.BwdDesc(fwd=fwd, gy=2, gpre=2, gx=dl.NO_TENSOR, gx_add=dl.NO_TENSOR, gw=gw.data_ptr(), workspace=ws.data_ptr(),
                      workspace_bytes=ws.numel())
    assert kernel in d.backward_kernel(desc), d.backward_kernel(desc)
    torch.cuda.synchronize()
    d.backward_segment([desc])
    d.backward_join()
    d.sync()
    ref = torch.zeros((Cout, R, R, Cin), dtype=torch.float64, device="cuda:0")
    for n in range(N):                                           # an image at a time: the padded float64 copy stays small
        xp = torch.nn.functional.pad(view[0][n].double(), (0, 0, pad, pad, pad, pad))
        gt = view[2][n].double().reshape(P * Q, Cout).t().contiguous()
        for r in range(R):
            for s in range(R):
                ref[:, r, s] += gt @ xp[r:r + stride * (P - 1) + 1:stride, s:s + stride * (Q - 1) + 1:stride].reshape(P * Q, Cin).contiguous()
    ref *= scale.double()[:, None, None, None]
    err = float((gw.double() - ref).abs().max() / ref.abs().max())
    print("  err %.2e" % err, flush=True)
    assert np.isfinite(err) and err <= 1e-6 + 2.0 ** -24 * (N * P * Q) ** 0.5 / 4
    d.close()
