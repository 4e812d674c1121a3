"""The classifier's two gradients at the edges of their tiles (64 x 128 of gw, 32 x 32 of gx, steps of 16 images and 32 classes), each alone and
both together, against float64 on the stored operands; scale of one, of 24 significant bits and of magnitudes far apart.

dL/dx: bf16 storage, 2^-9 of the element (4e-3 of the maximum); gy * scale is rounded to 32 bits as an fp32 product is, its three parts are exact.
dL/dw and bias: exact products, fp32 sums of at most 520 terms, 1e-5."""
import numpy as np
import pytest

import synth
from oracle import numeric as on
from test_gpu_backward import _bits, _dev, _small_ctx, torch_mod  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["ones", "odd", "apart"])
@pytest.mark.parametrize("N,Cin,Cout", [(1, 64, 8), (16, 64, 72), (17, 128, 1000), (31, 192, 40), (32, 64, 264), (33, 320, 1000), (129, 64, 520), (520, 128, 24),
                                        (577, 960, 24), (578, 960, 40), (545, 960, 120)])      # 570, 570, 540 tiles of gx: 8, 4, 2 to a workgroup
def test_gradients_at_tile_edges(torch_mod, N, Cin, Cout, kind):  # noqa: F811
    torch = torch_mod
    import paper_2203_15980_amd as dl
    x, w, g = _bits(31, 1, (N, 1, 1, Cin)), _bits(31, 2, (Cout, 1, 1, Cin), 0.05), _bits(31, 3, (N, Cout))
    scale = np.ones(Cout, np.float32)
    if kind != "ones":
        scale = (synth.normal(31, 4, Cout) * 0.3 + 1.0).astype(np.float32)
    if kind == "apart":
        scale *= np.float32(2.0) ** ((np.arange(Cout) % 9) * 8 - 32).astype(np.float32)
    d, put, get = _small_ctx(torch, [x.nbytes, g.nbytes, g.nbytes, x.nbytes])
    put(0, x)
    put(2, g)
    wd, sc, bd = _dev(torch, w), _dev(torch, scale), torch.zeros(Cout, device="cuda:0")
    fc = dl.LayerDesc(x=0, res=dl.NO_TENSOR, y=1, dtype=dl.DTYPE_BF16, w=wd.data_ptr(), scale=sc.data_ptr(), shift=bd.data_ptr(), N=N, H=1, W=1,
                      Cin=Cin, Cout=Cout, R=1, S=1, stride=1, pad=0, relu=0)
    xf, wf, gf, s64 = on.to_f64(x, "bf16").reshape(N, Cin), on.to_f64(w, "bf16").reshape(Cout, Cin), on.to_f64(g, "bf16"), scale.astype(np.float64)
    ref = ((gf * s64) @ wf, (gf.T @ xf) * s64[:, None], gf.sum(0))
    outs = []
    for want_gx, want_gw in ((True, True), (True, False), (False, True)):
        gw = torch.full((Cout * Cin + Cout,), float("nan"), device="cuda:0")
        d.backward_segment([dl.BwdDesc(fwd=fc, gy=2, gpre=2, gx=3 if want_gx else dl.NO_TENSOR, gx_add=dl.NO_TENSOR, gw=gw.data_ptr() if want_gw else None)])
        d.backward_join()
        d.sync()
        outs.append((get(3, (N, Cin)).copy() if want_gx else None, gw.cpu().numpy() if want_gw else None))
        if want_gx:
            d.release(3, dl.EV_FREE)
    assert np.array_equal(outs[0][0], outs[1][0]) and np.array_equal(outs[0][1], outs[2][1])
    got = outs[0][1].astype(np.float64)
    gwt = got[:Cout * Cin].reshape(Cout, Cin)
    far = lambda a, b: float(np.max(np.abs(a - b)) / np.max(np.abs(b)))          # noqa: E731
    rows = np.abs(gwt - ref[1]).max(1) / np.abs(ref[1]).max(1)                   # a class at a time: its own scale
    errs = (far(on.to_f64(outs[0][0], "bf16"), ref[0]), float(rows.max()), far(got[Cout * Cin:], ref[2]))
    print(N, Cin, Cout, kind, errs, flush=True)
    assert errs[0] <= 4e-3 and errs[1] <= 1e-5 and errs[2] <= 1e-5
    d.close()


def test_infinite_weights_meet_the_first_part_alone(torch_mod):  # noqa: F811
    """gy * scale in three parts: a part of zero must not make a NaN of an infinite weight.  Even classes' scale is one (their small parts are zeros)."""
    torch = torch_mod
    import paper_2203_15980_amd as dl
    N, Cin, Cout = 33, 64, 72
    x, w, g = _bits(32, 1, (N, 1, 1, Cin)), _bits(32, 2, (Cout, 1, 1, Cin), 0.05), _bits(32, 3, (N, Cout))
    g[(g & 0x7FFF) == 0] = 0x3F80
    scale = np.where(np.arange(Cout) % 2 == 0, 1.0, np.abs(synth.normal(32, 4, Cout)) + 0.5).astype(np.float32)
    for k, c, v in ((0, 3, 0x7F80), (5, 17, 0xFF80), (70, 40, 0x7F80), (71, 63, 0xFF80)):
        w[k, 0, 0, c] = v
    d, put, get = _small_ctx(torch, [x.nbytes, g.nbytes, g.nbytes, x.nbytes])
    put(0, x)
    put(2, g)
    wd, sc, bd = _dev(torch, w), _dev(torch, scale), torch.zeros(Cout, device="cuda:0")
    fc = dl.LayerDesc(x=0, res=dl.NO_TENSOR, y=1, dtype=dl.DTYPE_BF16, w=wd.data_ptr(), scale=sc.data_ptr(), shift=bd.data_ptr(), N=N, H=1, W=1,
                      Cin=Cin, Cout=Cout, R=1, S=1, stride=1, pad=0, relu=0)
    d.backward_segment([dl.BwdDesc(fwd=fc, gy=2, gpre=2, gx=3, gx_add=dl.NO_TENSOR, gw=None)])
    d.sync()
    got = on.to_f64(get(3, (N, Cin)), "bf16")
    ref = (on.to_f64(g, "bf16") * scale.astype(np.float64)) @ on.to_f64(w, "bf16").reshape(Cout, Cin)
    inf = np.isinf(ref)
    assert inf.sum() == 4 * N and not np.isnan(ref).any()
    assert np.array_equal(got[inf], ref[inf])
    assert np.max(np.abs(got[~inf] - ref[~inf])) <= 4e-3 * np.max(np.abs(ref[~inf]))
    d.close()


@pytest.mark.parametrize("N,Cin,Cout", [(1, 64, 8), (33, 64, 72), (17, 128, 1000), (32, 64, 264)])
def test_an_infinite_scale_stays_with_its_class(torch_mod, N, Cin, Cout):  # noqa: F811
    """Lanes whose classes lie past the last read other classes' scale: whatever it is, it must not reach the sums."""
    torch = torch_mod
    import paper_2203_15980_amd as dl
    w, g = _bits(33, 2, (Cout, 1, 1, Cin), 0.05), _bits(33, 3, (N, Cout))
    w[(w & 0x7FFF) == 0] = 0x3D00
    g[(g & 0x7FFF) == 0] = 0x3F80
    scale = np.ones(Cout, np.float32)
    scale[2] = np.inf
    d, put, get = _small_ctx(torch, [N * Cin * 2, g.nbytes, g.nbytes, N * Cin * 2])
    put(2, g)
    wd, sc, bd = _dev(torch, w), _dev(torch, scale), torch.zeros(Cout, device="cuda:0")
    fc = dl.LayerDesc(x=0, res=dl.NO_TENSOR, y=1, dtype=dl.DTYPE_BF16, w=wd.data_ptr(), scale=sc.data_ptr(), shift=bd.data_ptr(), N=N, H=1, W=1,
                      Cin=Cin, Cout=Cout, R=1, S=1, stride=1, pad=0, relu=0)
    d.backward_segment([dl.BwdDesc(fwd=fc, gy=2, gpre=2, gx=3, gx_add=dl.NO_TENSOR, gw=None)])
    d.sync()
    got = on.to_f64(get(3, (N, Cin)), "bf16")
    wf, gf = on.to_f64(w, "bf16").reshape(Cout, Cin), on.to_f64(g, "bf16")
    assert np.array_equal(got, np.sign(gf[:, 2:3]) * np.sign(wf[2])[None] * np.inf)
    d.close()


@pytest.mark.parametrize("N,Cin,Cout", [(128, 64, 8), (129, 64, 8), (192, 128, 72), (255, 320, 40), (520, 64, 56), (4096, 192, 24)])
def test_weight_sums_of_every_eighth_step(torch_mod, N, Cin, Cout):  # noqa: F811
    """Eight sums, of every eighth step of 16 images: 2^24 in one image and -2^24 eight steps on (the last step of its sum, where there is one), a
    single one in each step of the other seven sums.  Exact, as no sum of the tree leaves 24 bits; 2^24 + 1 does, and the ones are lost where sums are
    of every fourth step."""
    torch = torch_mod
    import paper_2203_15980_amd as dl
    n, k = np.arange(N)[:, None], np.arange(Cout)[None]
    g = np.where((n // 16 % 8 != k % 8) & (n % 16 == k % 16), 1.0, 0.0).astype(np.float32)       # class k: 2^24 in sum k % 8
    for c in range(Cout):
        steps = range(16 * (c % 8), N, 128)
        if len(steps) > 1:
            g[steps[0], c], g[steps[-1], c] = 2.0 ** 24, -2.0 ** 24
    x = np.full((N, 1, 1, Cin), 0x3F80, np.uint16)
    g16 = synth.f32_to_bf16_bits(g).reshape(g.shape)
    d, put, get = _small_ctx(torch, [x.nbytes, g16.nbytes, g16.nbytes, x.nbytes])
    put(0, x)
    put(2, g16)
    w, one, gw = torch.zeros(Cout * Cin, dtype=torch.bfloat16, device="cuda:0"), torch.ones(Cout, device="cuda:0"), torch.zeros(Cout * Cin + Cout, device="cuda:0")
    fc = dl.LayerDesc(x=0, res=dl.NO_TENSOR, y=1, dtype=dl.DTYPE_BF16, w=w.data_ptr(), scale=one.data_ptr(), shift=one.data_ptr(), N=N, H=1, W=1,
                      Cin=Cin, Cout=Cout, R=1, S=1, stride=1, pad=0, relu=0)
    d.backward_segment([dl.BwdDesc(fwd=fc, gy=2, gpre=2, gx=dl.NO_TENSOR, gx_add=dl.NO_TENSOR, gw=gw.data_ptr())])
    d.backward_join()
    d.sync()
    got = gw.cpu().numpy()[:Cout * Cin].reshape(Cout, Cin)
    d.close()
    assert np.array_equal(got, np.broadcast_to(g.astype(np.float64).sum(0)[:, None], got.shape)) and got.any()
