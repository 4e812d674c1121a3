"""The bf16 weight gradients alone, against float64 on the stored operands, at the edges of their tiles and chunks.

Tolerance: products of two bf16 values are exact in fp32; the sums have at most 6000 terms, split over wavefronts and
workgroups: 1e-5 of the largest entry (about sqrt(6000) * 2^-24, with a margin of two)."""
import numpy as np
import pytest

import synth
from oracle import numeric as on
from test_gpu_backward import _bits, _dev, _small_ctx, torch_mod  # noqa: F401

pytestmark = pytest.mark.gpu

CASES = [
    # N  H   W   Cin  Cout R stride
    (1, 1, 1, 64, 64, 1, 1),          # one pixel; one 64 x 64 tile, eight wavefronts on it
    (1, 9, 15, 128, 64, 1, 1),        # 135 pixels: a full slice of 128 and one of 7
    (2, 8, 8, 256, 64, 1, 1),         # four tiles along the input channels; whole slices
    (1, 5, 13, 64, 128, 1, 1),
    (3, 7, 31, 64, 512, 1, 1),        # four tiles along the output channels, two of those; 651 pixels
    (2, 11, 13, 192, 320, 1, 1),      # neither count a multiple of 128
    (2, 9, 7, 128, 256, 1, 2),        # strided, odd sizes
    (1, 8, 6, 64, 64, 1, 3),
    (1, 1, 1, 64, 64, 3, 1),          # only the centre tap has anything
    (5, 3, 1, 64, 128, 3, 1),         # images one pixel wide: two list pixels to a row
    (3, 7, 7, 128, 64, 3, 1),         # several images to a chunk
    (1, 3, 125, 64, 64, 3, 1),        # the widest row a chunk takes
    (2, 30, 17, 64, 64, 3, 1),        # chunks that end inside an image, a short last one
    (2, 6, 5, 128, 128, 3, 2),        # even height, odd width
    (3, 7, 8, 128, 256, 3, 2),
    (1, 1, 3, 128, 128, 3, 2),        # no odd rows at all
    (1, 9, 79, 128, 128, 3, 2),       # 40 output columns
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "%dx%dx%d_%d_%d_r%d_s%d" % c)
def test_weight_gradient_matches_float64(torch_mod, case):  # noqa: F811
    torch = torch_mod
    import paper_2203_15980_amd as dl
    N, H, W, Cin, Cout, R, stride = case
    print("case", case, flush=True)
    P, Q, pad = (H - 1) // stride + 1, (W - 1) // stride + 1, R // 2
    x, gy = _bits(94, 1, (N, H, W, Cin)), _bits(94, 2, (N, P, Q, Cout))
    scale = (synth.normal(94, 3, Cout) * 0.3 + 1.0).astype(np.float32)
    d, put, get = _small_ctx(torch, [x.nbytes, gy.nbytes, gy.nbytes])
    put(0, x)
    put(2, gy)
    w, sc, sh = torch.zeros(Cout * R * R * Cin, dtype=torch.bfloat16, device="cuda:0"), _dev(torch, scale), torch.zeros(Cout, device="cuda:0")
    fwd = dl.LayerDesc(x=0, res=dl.NO_TENSOR, y=1, dtype=dl.DTYPE_BF16, w=w.data_ptr(), scale=sc.data_ptr(), shift=sh.data_ptr(), N=N, H=H, W=W,
                       Cin=Cin, Cout=Cout, R=R, S=R, stride=stride, pad=pad, relu=0)
    ws = torch.full((max(d.backward_workspace(fwd), 256),), 255, dtype=torch.uint8, device="cuda:0")     # NaN wherever nothing is written
    got = []
    for _ in range(2):
        gw = torch.full((Cout, R, R, Cin), float("nan"), device="cuda:0")
        desc = dl.BwdDesc(fwd=fwd, gy=2, gpre=2, gx=dl.NO_TENSOR, gx_add=dl.NO_TENSOR, gw=gw.data_ptr(), workspace=ws.data_ptr(),
                          workspace_bytes=ws.numel())
        assert d.backward_kernel(desc).startswith("gw: wgrad%dx%d %sbf16" % (R, R, "stride 2 " if R == 3 and stride == 2 else ""))
        d.backward_segment([desc])
        d.backward_join()
        d.sync()
        got.append(gw.cpu().numpy())
    xf, gf = on.to_f64(x, "bf16"), on.to_f64(gy, "bf16")
    xp = np.pad(xf, ((0, 0), (pad, pad), (pad, pad), (0, 0)))
    ref = np.empty((Cout, R, R, Cin))
    for r in range(R):
        for s in range(R):
            ref[:, r, s] = np.tensordot(gf, xp[:, r:r + stride * (P - 1) + 1:stride, s:s + stride * (Q - 1) + 1:stride], ((0, 1, 2), (0, 1, 2)))
    ref *= scale.astype(np.float64)[:, None, None, None]
    err = float(np.max(np.abs(got[0] - ref)) / np.max(np.abs(ref)))
    print("  err %.2e" % err, flush=True)
    assert err <= 1e-5 and np.array_equal(got[0], got[1])
    d.close()


@pytest.mark.parametrize("W", [102, 103, 112, 125, 126])
def test_strided_rows_wider_than_a_chunk(torch_mod, W):  # noqa: F811
    """A 3x3 stride-2 layer's rows of more than 51 output columns (width 103 and up) do not fit the one-launch kernel's chunk: gpre = gy is
    then refused before anything is launched, and a separate gpre at the input's resolution takes the stride-1 kernel up to
    its own width, 125.  Same bound as above."""
    torch = torch_mod
    import paper_2203_15980_amd as dl
    from paper_2203_15980_amd import binding
    N, H, C = 2, 5, 128
    P, Q = (H - 1) // 2 + 1, (W - 1) // 2 + 1
    print("W", W, "Q", Q, flush=True)
    x, gy = _bits(94, 4, (N, H, W, C)), _bits(94, 5, (N, P, Q, C))
    wide = N * H * W * C * 2
    d, put, get = _small_ctx(torch, [x.nbytes, gy.nbytes, gy.nbytes, wide])
    put(0, x)
    put(2, gy)
    w, one = torch.zeros(C * 9 * C, dtype=torch.bfloat16, device="cuda:0"), torch.ones(C, device="cuda:0")
    fwd = dl.LayerDesc(x=0, res=dl.NO_TENSOR, y=1, dtype=dl.DTYPE_BF16, w=w.data_ptr(), scale=one.data_ptr(), shift=one.data_ptr(), N=N, H=H,
                       W=W, Cin=C, Cout=C, R=3, S=3, stride=2, pad=1, relu=0)
    ws = torch.full((max(d.backward_workspace(fwd), 256),), 255, dtype=torch.uint8, device="cuda:0")
    xf, gf = on.to_f64(x, "bf16"), on.to_f64(gy, "bf16")
    xp = np.pad(xf, ((0, 0), (1, 1), (1, 1), (0, 0)))
    ref = np.empty((C, 3, 3, C))
    for r in range(3):
        for s in range(3):
            ref[:, r, s] = np.tensordot(gf, xp[:, r:r + 2 * (P - 1) + 1:2, s:s + 2 * (Q - 1) + 1:2], ((0, 1, 2), (0, 1, 2)))
    for gpre, takes in ((2, Q <= binding.WGRAD_S2_MAX_Q), (3, W <= 125)):
        gw = torch.full((C, 3, 3, C), float("nan"), device="cuda:0")
        desc = dl.BwdDesc(fwd=fwd, gy=2, gpre=gpre, gx=dl.NO_TENSOR, gx_add=dl.NO_TENSOR, gw=gw.data_ptr(), workspace=ws.data_ptr(),
                          workspace_bytes=ws.numel())
        if not takes:
            with pytest.raises(dl.DeltaError) as e:
                d.backward_segment([desc])
            assert e.value.status == dl.ERR_INVALID
            continue
        d.backward_segment([desc])
        d.backward_join()
        d.sync()
        err = float(np.max(np.abs(gw.cpu().numpy() - ref)) / np.max(np.abs(ref)))
        print("  gpre %d err %.2e" % (gpre, err), flush=True)
        assert err <= 1e-5
    d.close()


@pytest.mark.parametrize("W", [102, 112])
def test_network_takes_the_route_its_width_allows(torch_mod, W):  # noqa: F811
    """A strided 3x3 layer between two 1x1 layers: 51 output columns run at the output's resolution, 56 are spread out."""
    torch = torch_mod
    import paper_2203_15980_amd as dl
    from paper_2203_15980_amd.harness import Net
    layers = [synth.LayerSpec("a", "conv", "x0", None, "a", 1, 4, W, 128, 128, index=1),
              synth.LayerSpec("b", "conv", "a", None, "b", 1, 4, W, 128, 128, 3, 3, 2, 1, index=2),
              synth.LayerSpec("c", "conv", "b", None, "c", 1, 2, W // 2, 128, 128, index=3)]
    g = synth.fused_graph(layers, "bf16")
    d = dl.Delta(torch.empty(32 << 20, dtype=torch.uint8, device="cuda:0"), torch.cuda.current_stream().cuda_stream)
    d.bind([t["bytes"] for t in g.tensors])
    net = Net(d, layers, "bf16", synth.master_seed(2))
    net.enable_backward(input_gradient=True)
    net.forward()
    net.backward(keep=True)
    d.sync()
    trace = {t[0]: t for t in net.bwd_trace}
    _, gy_name, gpre_name, gx_name, _, masks_gx = trace["b"]
    assert (gpre_name == gy_name) == (W == 102)
    l, p = layers[1], net.params_np["b"]
    xa = net.read("a")
    ref_gx, ref_gw, _ = on.conv_bn_act_bwd(xa, p["w"], p, net.read("b"), net.read(gy_name), stride=2, pad=1, relu=True, dtype="bf16")
    if masks_gx:
        ref_gx = np.where(on.to_f64(xa, "bf16") > 0, ref_gx, 0.0)
    ex = float(np.max(np.abs(on.to_f64(net.read(gx_name), "bf16") - ref_gx)) / np.max(np.abs(ref_gx)))
    ew = float(np.max(np.abs(net.gw["b"].cpu().numpy().reshape(ref_gw.shape) - ref_gw)) / np.max(np.abs(ref_gw)))
    print("  gx %.2e gw %.2e" % (ex, ew), flush=True)
    assert ex <= 2e-2 and ew <= 2e-4             # the bounds of the layer-by-layer comparisons (weights rounded once more)
    d.close()


def test_a_row_wider_than_a_chunk_is_refused(torch_mod):  # noqa: F811
    torch = torch_mod
    import paper_2203_15980_amd as dl
    nbytes = 3 * 126 * 64 * 2
    d, put, get = _small_ctx(torch, [nbytes, nbytes, nbytes])
    for t in (0, 2):
        d.alloc(t)
    w, one, gw = torch.zeros(64 * 9 * 64, device="cuda:0"), torch.ones(64, device="cuda:0"), torch.empty(64 * 9 * 64, device="cuda:0")
    ws = torch.empty(1 << 20, dtype=torch.uint8, device="cuda:0")
    fwd = dl.LayerDesc(x=0, res=dl.NO_TENSOR, y=1, dtype=dl.DTYPE_BF16, w=w.data_ptr(), scale=one.data_ptr(), shift=one.data_ptr(), N=1, H=3,
                       W=126, Cin=64, Cout=64, R=3, S=3, stride=1, pad=1, relu=0)
    with pytest.raises(dl.DeltaError) as e:
        d.backward_segment([dl.BwdDesc(fwd=fwd, gy=2, gpre=2, gx=dl.NO_TENSOR, gx_add=dl.NO_TENSOR, gw=gw.data_ptr(), workspace=ws.data_ptr(),
                                       workspace_bytes=ws.numel())])
    assert e.value.status == dl.ERR_INVALID
    d.close()


def test_large_and_small_weight_gradients_share_a_workspace(torch_mod):  # noqa: F811
    """A weight gradient of 1 GFLOP runs on the second stream, a smaller one on the compute stream, and all use one workspace:
    the small one that follows has to wait for the large one's sums, the large one that follows for the small one's.  In one segment the
    bits are those of runs with a synchronisation between."""
    torch = torch_mod
    import paper_2203_15980_amd as dl
    shapes = [(8, 32, 32, 256, 256, 1, "second"), (1, 9, 7, 128, 256, 1, "compute"), (32, 14, 14, 128, 128, 3, "second"),
              (2, 7, 7, 128, 64, 3, "compute"), (8, 32, 32, 256, 256, 1, "second")]
    sizes, data = [], []
    for i, (N, H, W, Ci, Co, R, _) in enumerate(shapes):
        data.append((_bits(95, 2 * i, (N, H, W, Ci)), _bits(95, 2 * i + 1, (N, H, W, Co))))
        sizes += [data[i][0].nbytes, data[i][1].nbytes, data[i][1].nbytes]
    d, put, get = _small_ctx(torch, sizes, mb=96)
    w, one = torch.zeros(256 * 256 * 9, device="cuda:0"), torch.ones(256, device="cuda:0")
    fwds, need = [], 0
    for i, (N, H, W, Ci, Co, R, _) in enumerate(shapes):
        put(3 * i, data[i][0])
        put(3 * i + 2, data[i][1])
        fwds.append(dl.LayerDesc(x=3 * i, res=dl.NO_TENSOR, y=3 * i + 1, dtype=dl.DTYPE_BF16, w=w.data_ptr(), scale=one.data_ptr(),
                                 shift=one.data_ptr(), N=N, H=H, W=W, Cin=Ci, Cout=Co, R=R, S=R, stride=1, pad=R // 2, relu=0))
        need = max(need, d.backward_workspace(fwds[i]))
    ws = torch.empty(need, dtype=torch.uint8, device="cuda:0")

    def run(apart):
        gws, descs = [], []
        for i, (N, H, W, Ci, Co, R, stream) in enumerate(shapes):
            gws.append(torch.full((Co * R * R * Ci,), float("nan"), device="cuda:0"))
            descs.append(dl.BwdDesc(fwd=fwds[i], gy=3 * i + 2, gpre=3 * i + 2, gx=dl.NO_TENSOR, gx_add=dl.NO_TENSOR, gw=gws[i].data_ptr(),
                                    workspace=ws.data_ptr(), workspace_bytes=need))
            assert stream + " stream" in d.backward_kernel(descs[i]), d.backward_kernel(descs[i])
        torch.cuda.synchronize()
        for part in ([[x] for x in descs] if apart else [descs]):
            d.backward_segment(part)
            if apart:
                d.backward_join()
                d.sync()
        d.backward_join()
        d.sync()
        return [g.cpu().numpy() for g in gws]
    ref = run(True)
    assert all(np.all(np.isfinite(r)) for r in ref)
    for _ in range(4):
        assert all(np.array_equal(a, b) for a, b in zip(run(False), ref))
    d.close()
