"""The head of the network - average pool, loss, and the classifier's and the loss's gradients - at the edges of its
kernels' tiles, against float64 on the stored operands.

Tolerances: bf16 outputs one rounding, 2^-9 of the element and so at most 2^-9 of the maximum (4e-3); fp32 sums of
n terms n * 2^-24 of the sum of magnitudes in the worst order, here at most 1032 terms: 6e-5 (1e-5 for the sums that
MFMAs and wavefronts split)."""
import numpy as np
import pytest

import synth
from oracle import numeric as on
from test_gpu_backward import _bits, _dev, _small_ctx, torch_mod  # noqa: F401

pytestmark = pytest.mark.gpu


def _far(got, ref):
    return float(np.max(np.abs(got - ref)) / max(np.max(np.abs(ref)), 1e-30))


@pytest.mark.parametrize("N,Cin,Cout", [(1, 64, 8), (17, 192, 24), (3, 320, 520), (33, 64, 1000), (2, 64, 1032)])
def test_classifier_gradients_and_loss_at_tile_edges(torch_mod, N, Cin, Cout):  # noqa: F811
    torch = torch_mod
    import paper_2203_15980_amd as dl
    x, w, z = _bits(8, 1, (N, 1, 1, Cin)), _bits(8, 2, (Cout, 1, 1, Cin), 0.05), _bits(8, 4, (N, Cout), 3.0)
    scale = (synth.normal(8, 5, Cout) * 0.3 + 1.0).astype(np.float32)
    labels = synth.make_labels(8, N, Cout)
    d, put, get = _small_ctx(torch, [x.nbytes, z.nbytes, N * 8, 4, z.nbytes, x.nbytes])
    put(0, x)
    put(1, z)
    put(2, labels)
    wd, sc, bd = _dev(torch, w), _dev(torch, scale), torch.zeros(Cout, device="cuda:0")
    fc = dl.LayerDesc(x=0, res=dl.NO_TENSOR, y=1, dtype=dl.DTYPE_BF16, w=wd.data_ptr(), scale=sc.data_ptr(), shift=bd.data_ptr(), N=N,
                      H=1, W=1, Cin=Cin, Cout=Cout, R=1, S=1, stride=1, pad=0, relu=0)
    loss = dl.LayerDesc(x=1, res=2, y=3, dtype=dl.DTYPE_BF16, N=N, H=1, W=1, Cin=Cout, Cout=1, R=1, S=1, stride=1, pad=0, relu=0,
                        op=dl.OP_SOFTMAX_CE)
    gw = torch.full((Cout * Cin + Cout,), float("nan"), device="cuda:0")
    d.recompute_segment([loss])
    d.backward_segment([dl.BwdDesc(fwd=loss, gy=dl.NO_TENSOR, gpre=dl.NO_TENSOR, gx=4, gx_add=dl.NO_TENSOR),
                        dl.BwdDesc(fwd=fc, gy=4, gpre=4, gx=5, gx_add=dl.NO_TENSOR, gw=gw.data_ptr())])
    d.backward_join()
    d.sync()
    zf = on.to_f64(z, "bf16")
    e = np.exp(zf - zf.max(1, keepdims=True))
    soft = e / e.sum(1, keepdims=True)
    got_loss = float(get(3, (1,), np.float32)[0])
    ref_loss = float(np.mean(-np.log(soft[np.arange(N), labels])))
    assert abs(got_loss - ref_loss) <= 1e-5 * abs(ref_loss)
    ref_gz = soft.copy()
    ref_gz[np.arange(N), labels] -= 1
    gz = on.to_f64(get(4, (N, Cout)), "bf16")
    g = gw.cpu().numpy().astype(np.float64)
    xf, wf = on.to_f64(x, "bf16").reshape(N, Cin), on.to_f64(w, "bf16").reshape(Cout, Cin)
    s64 = scale.astype(np.float64)
    errs = (_far(gz, ref_gz / N), _far(on.to_f64(get(5, (N, Cin)), "bf16"), (gz * s64) @ wf),
            _far(g[:Cout * Cin].reshape(Cout, Cin), (gz.T @ xf) * s64[:, None]), _far(g[Cout * Cin:], gz.sum(0)))
    print("N %d Cin %d Cout %d: %s" % (N, Cin, Cout, errs), flush=True)
    assert errs[0] <= 4e-3 and errs[1] <= 4e-3 and errs[2] <= 1e-5 and errs[3] <= 1e-5
    d.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("N,classes", [(1, 1), (33, 256), (33, 257), (1, 1000), (31, 1001), (65, 1024), (3, 1025), (34, 520)])
def test_loss_forms_match_float64(torch_mod, dtype, N, classes):  # noqa: F811
    """Every form of the loss: class counts on both sides of the lines at 256 and 1024, whole 16-byte rows and not, image counts
    that leave wavefronts and their last rounds partly empty.  A label out of range makes the result NaN."""
    torch = torch_mod
    import paper_2203_15980_amd as dl
    z = synth.normal(10, 1, N * classes).astype(np.float32).reshape(N, classes) * 3
    z = z if dtype == "f32" else synth.f32_to_bf16_bits(z).reshape(N, classes)
    labels = synth.make_labels(10, N, classes)
    d, put, get = _small_ctx(torch, [z.nbytes, N * 8, 4])
    put(0, z)
    put(1, labels)
    loss = dl.LayerDesc(x=0, res=1, y=2, dtype=dl.DTYPE_F32 if dtype == "f32" else dl.DTYPE_BF16, N=N, H=1, W=1, Cin=classes, Cout=1, R=1,
                        S=1, stride=1, pad=0, relu=0, op=dl.OP_SOFTMAX_CE)
    d.recompute_segment([loss])
    d.sync()
    got = float(get(2, (1,), np.float32)[0])
    zf = on.to_f64(z, dtype)
    top = zf.max(1)
    ref = float(np.mean(top + np.log(np.exp(zf - top[:, None]).sum(1)) - zf[np.arange(N), labels]))
    print("%s N %d classes %d: %.8g %.8g" % (dtype, N, classes, got, ref), flush=True)
    assert abs(got - ref) <= 1e-5 * max(abs(ref), 1.0)
    bad = labels.copy()
    bad[N // 2] = classes
    d.arena[d.tensor_ptr(1) - d.arena.data_ptr():][:N * 8].copy_(_dev(torch, bad.view(np.uint8)))
    d.recompute_segment([loss])
    d.sync()
    assert np.isnan(get(2, (1,), np.float32)[0])
    d.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("N,H,W,C", [(1, 1, 1, 8), (3, 1, 7, 40), (5, 7, 7, 264), (2, 9, 3, 2048), (513, 1, 1, 8), (130, 4, 4, 40), (19, 1, 17, 264)])
def test_average_pool_at_tile_edges(torch_mod, dtype, N, H, W, C):  # noqa: F811
    torch = torch_mod
    import paper_2203_15980_amd as dl
    x = synth.make_input(9, (N, H, W, C), dtype)
    es = 4 if dtype == "f32" else 2
    d, put, get = _small_ctx(torch, [x.nbytes, N * C * es])
    put(0, x)
    d.recompute_segment([dl.LayerDesc(x=0, res=dl.NO_TENSOR, y=1, dtype=dl.DTYPE_F32 if dtype == "f32" else dl.DTYPE_BF16, N=N, H=H, W=W,
                                      Cin=C, Cout=C, R=H, S=W, stride=1, pad=0, relu=0, op=dl.OP_AVGPOOL)])
    d.sync()
    got = on.to_f64(get(1, (N, C), np.float32 if dtype == "f32" else np.uint16), dtype)
    err = _far(got, on.to_f64(x, dtype).mean((1, 2)))
    print("err %.2e" % err, flush=True)
    assert err <= (1e-6 if dtype == "f32" else 4e-3)
    d.close()
