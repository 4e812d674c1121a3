"""The 3 x 3, stride 2 max pool's gradient at the edges of its tiles (8 x 16 pixels, 64 channels), bit for bit.

The incoming gradients are whole numbers up to 8: sums of at most four are exact in bf16, so the result has one right value."""
import numpy as np
import pytest

import synth
from oracle import numeric as on
from test_gpu_backward import _bits, _small_ctx, torch_mod  # noqa: F401

pytestmark = pytest.mark.gpu

CASES = [(1, 1, 1, 8), (3, 2, 2, 64), (2, 7, 15, 72), (2, 8, 16, 64), (1, 9, 17, 136), (2, 16, 31, 8), (1, 25, 33, 64)]


@pytest.mark.parametrize("mask_x", [0, 1])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "%dx%dx%d_%d" % c)
def test_max_pool_gradient_is_exact(torch_mod, case, mask_x):  # noqa: F811
    torch = torch_mod
    import paper_2203_15980_amd as dl
    print("case", case, mask_x, flush=True)
    N, H, W, C = case
    P, Q = (H - 1) // 2 + 1, (W - 1) // 2 + 1
    x = _bits(97, 1, (N, H, W, C))
    pick = _bits(97, 2, x.shape) % 16                                        # ties at zero and at one, both zeros, -inf, NaN of both signs
    for k, v in enumerate([0x0000, 0x8000, 0x3F80, 0xFF80, 0x7F80, 0x7FC1, 0xFFC1, 0x8001, 0x0001]):
        x[pick == k] = v
    x[:, :3, :3, :8] = 0xFF80                                                # whole windows of -inf: nobody receives anything
    gy = synth.f32_to_bf16_bits(np.round(np.clip(synth.normal(97, 3, N * P * Q * C) * 3, -8, 8)).astype(np.float32)).reshape(N, P, Q, C)
    d, put, get = _small_ctx(torch, [x.nbytes, gy.nbytes, gy.nbytes, x.nbytes])
    put(0, x)
    put(2, gy)
    fwd = dl.LayerDesc(x=0, res=dl.NO_TENSOR, y=1, dtype=dl.DTYPE_BF16, w=None, scale=None, shift=None, N=N, H=H, W=W,
                       Cin=C, Cout=C, R=3, S=3, stride=2, pad=1, relu=0, op=dl.OP_MAXPOOL)
    d.backward_segment([dl.BwdDesc(fwd=fwd, gy=2, gpre=2, gx=3, gx_add=dl.NO_TENSOR, mask_gx=mask_x, wt=None, gw=None,
                                   workspace=None, workspace_bytes=0)])
    d.sync()
    got = on.to_f64(get(3, x.shape), "bf16")
    d.close()
    seen = (((x & 0x7FFF) <= 0x7F80) & (x != 0xFF80)).astype(np.uint16)      # neither NaN nor -inf
    xc = np.where(seen, x, 0xFF80).astype(np.uint16)
    live = np.zeros(gy.shape, bool)
    for r in range(3):
        for s in range(3):
            for p in range(P):
                for q in range(Q):
                    h, w = 2 * p + r - 1, 2 * q + s - 1
                    if 0 <= h < H and 0 <= w < W:
                        live[:, p, q] |= seen[:, h, w] != 0
    ref = on.maxpool_bwd(xc, np.where(live, gy, 0).astype(np.uint16), 3, 3, 2, 1, "bf16")
    if mask_x:
        ref = np.where(on.to_f64(xc, "bf16") > 0, ref, 0.0)
    assert np.array_equal(got, ref)
