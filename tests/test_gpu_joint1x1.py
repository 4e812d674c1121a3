"""Both gradients of a 1x1 layer in one pass over its tensors: every tile the kernel has (64 KT x 64 CT of gradient and input channels, both chunk
sizes), slices of the input channels, chunks that are whole, one short and one pixel, with and without gx_add and mask.  Reference and bounds as
in the helper (the sums here have up to 25088 terms: 1e-5 is 2^-24 sqrt(25088) with a margin of one)."""
import numpy as np
import pytest

from test_gpu_small_backward import test_both_gradients_match_float64 as both
from test_gpu_parity import make_delta, torch_mod  # noqa: F401

pytestmark = pytest.mark.gpu

JOINT = "joint1x1 bf16, the same launch"
CASES = [
    # dtype  N   H    W   Cin Cout R stride add mask
    ("bf16", 1, 128, 200,  64,  64, 1, 1, True,  True,  JOINT),     # 25600 pixels: whole chunks of 64
    ("bf16", 1, 131, 193,  64,  64, 1, 1, False, True,  JOINT),     # 25283: 3 of the last chunk's 64
    ("bf16", 3,  97,  89, 128,  64, 1, 1, True,  False, JOINT),
    ("bf16", 1, 131, 193, 256,  64, 1, 1, True,  True,  JOINT),     # chunks of 32
    ("bf16", 1, 151, 167, 256,  64, 1, 1, False, False, JOINT),     # 25217: one pixel of the last chunk
    ("bf16", 3,  97,  89, 192,  64, 1, 1, True,  True,  JOINT),     # three slices of 64 input channels
    ("bf16", 1, 131, 193,  64, 128, 1, 1, True,  True,  JOINT),
    ("bf16", 1, 131, 193, 128, 128, 1, 1, False, True,  JOINT),
    ("bf16", 1, 131, 193, 256, 128, 1, 1, True,  True,  JOINT),
    ("bf16", 1, 131, 193, 512, 128, 1, 1, False, True,  JOINT),     # two slices of 256
    ("bf16", 1, 131, 193,  64, 256, 1, 1, False, True,  JOINT),
    ("bf16", 1, 131, 193,  64, 256, 1, 1, True,  True,  JOINT),
    ("bf16", 1, 131, 193, 128, 256, 1, 1, True,  False, JOINT),
    ("bf16", 1, 131, 193,  64, 512, 1, 1, False, True,  JOINT),
    ("bf16", 1, 131, 193, 128, 512, 1, 1, True,  True,  JOINT),     # two slices of 64
    ("bf16", 1,  64,  65,  64,  64, 1, 1, True,  True,  JOINT),     # 65 chunks: 33 workers of two, the last has one
    ("bf16", 1, 131, 193, 320,  64, 1, 1, True,  True,  JOINT),     # five of 64: 48 workers, six to an XCD of 32 CUs
    ("bf16", 1, 131, 193, 768, 256, 1, 1, False, True,  JOINT),     # six of 128: 40 workers
    ("bf16", 1,  97,  89, 448, 256, 1, 1, True,  True,  JOINT),     # seven of 64: 32 workers
    ("bf16", 1,  79,  89, 1024, 256, 1, 1, True, True,  JOINT),     # eight slices of 128; 31 workers, the longest with eight chunks
    ("bf16", 1,  79,  89, 1152, 256, 1, 1, True, True,  "wgrad1x1 bf16, second stream"),      # nine slices
    ("bf16", 1,  95,  95, 128, 512, 1, 1, False, True,  JOINT),     # 9025 pixels
    ("bf16", 1,  95,  94, 128, 512, 1, 1, False, True,  "wgrad1x1 bf16, second stream"),
    ("bf16", 1,  95,  95, 192, 512, 1, 1, False, True,  "wgrad1x1 bf16, second stream"),      # three slices of 64
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "%s_%dx%dx%d_%d_%d_r%d_s%d" % c[:8])
def test_every_tile_matches_float64(torch_mod, case):  # noqa: F811
    both(torch_mod, case)


def test_sums_share_a_workspace_with_the_second_stream(torch_mod):  # noqa: F811
    """A 3x3 weight gradient on the second stream and the one-pass kernel in turn, on a workspace that holds one at a time and on one that
    holds both: the bits are those of runs with a synchronisation between, and a workspace too small for the one-pass kernel's sums takes the two
    kernels."""
    torch = torch_mod
    import paper_2203_15980_amd as dl
    N, H, W, C, K = 16, 56, 56, 64, 256
    sizes = [N * H * W * C * 2, N * H * W * K * 2, N * H * W * K * 2, N * H * W * C * 2, N * H * W * C * 2]       # x, y, gy, gx, 3x3's gy
    d = make_delta(torch, sum(sizes) + N * H * W * C * 4 + (2 << 20))
    d.bind(sizes + [N * H * W * C * 2])                          # 5: the 3x3 layer's gx
    gen = torch.Generator(device="cuda:0").manual_seed(5)
    for t in (0, 2, 4):
        d.alloc(t)
        d.arena[d.tensor_ptr(t) - d.arena.data_ptr():][:sizes[t]].view(torch.bfloat16).normal_(generator=gen)
    d.alloc(1)
    one, w = torch.ones(K, device="cuda:0"), torch.randn(K * C * 9, device="cuda:0", generator=gen).to(torch.bfloat16)
    lay = lambda y, co, R: dl.LayerDesc(x=0, res=dl.NO_TENSOR, y=y, dtype=dl.DTYPE_BF16, w=w.data_ptr(), scale=one.data_ptr(),      # noqa: E731
                                        shift=one.data_ptr(), N=N, H=H, W=W, Cin=C, Cout=co, R=R, S=R, stride=1, pad=R // 2, relu=0)
    f1, f3 = lay(1, K, 1), lay(4, C, 3)
    n1, n3 = d.backward_workspace(f1), d.backward_workspace(f3)

    def run(ws, apart):
        gws = [torch.full((K * C * 9,), float("nan"), device="cuda:0") for _ in range(4)]
        b = lambda f, gy, gx, i: dl.BwdDesc(fwd=f, gy=gy, gpre=gy, gx=gx, gx_add=dl.NO_TENSOR, wt=w.data_ptr(), gw=gws[i].data_ptr(),  # noqa: E731
                                            workspace=ws.data_ptr(), workspace_bytes=ws.numel())
        descs = [b(f3, 4, 5, 0), b(f1, 2, 3, 1), b(f3, 4, 5, 2), b(f1, 2, 3, 3)]
        torch.cuda.synchronize()
        for part in ([[x] for x in descs] if apart else [descs]):
            d.backward_segment(part)
            if apart:
                d.backward_join()
                d.sync()
        d.backward_join()
        d.sync()
        name = d.backward_kernel(descs[1])
        return name, [g.cpu().numpy()[:K * C if i & 1 else C * C * 9] for i, g in enumerate(gws)]
    for nbytes in (max(n1, n3), n1 + n3 + 256):
        ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda:0")
        name, ref = run(ws, True)
        assert name.endswith(JOINT) and all(np.all(np.isfinite(r)) for r in ref)
        assert np.array_equal(ref[0], ref[2]) and np.array_equal(ref[1], ref[3])
        for _ in range(3):
            assert all(np.array_equal(a, b) for a, b in zip(run(ws, False)[1], ref))
    name, small = run(torch.empty(n1 - 256, dtype=torch.uint8, device="cuda:0"), False)
    assert "wgrad1x1" in name
    assert float(np.max(np.abs(small[1] - ref[1])) / np.max(np.abs(ref[1]))) <= 1e-5
    d.close()


@pytest.mark.parametrize("Cin,Cout,H,W,add", [(64, 128, 131, 193, True), (256, 64, 151, 167, False), (128, 512, 95, 95, True)])
def test_infinities_in_the_last_pixel(torch_mod, Cin, Cout, H, W, add):  # noqa: F811
    """The last chunk's rows past the last pixel are fetched from that pixel and cleared: an infinite input and an infinite gradient there reach
    their own column and row of gw and their own pixel of gx, as in float64, and nothing else."""
    torch = torch_mod
    import paper_2203_15980_amd as dl
    M = H * W
    nbytes = [M * Cin * 2, M * Cout * 2, M * Cout * 2, M * Cin * 2, M * Cin * 2]       # x, y, gy, gx, gx_add
    d = make_delta(torch, sum(nbytes) + (2 << 20))
    d.bind(nbytes)
    gen = torch.Generator(device="cuda:0").manual_seed(41)
    view = {}
    for t, C in ((0, Cin), (2, Cout), (4, Cin)):
        d.alloc(t)
        view[t] = d.arena[d.tensor_ptr(t) - d.arena.data_ptr():][:nbytes[t]].view(torch.bfloat16).reshape(M, C)
        view[t].normal_(generator=gen)
        view[t].masked_fill_(view[t] == 0, 0.5)
    d.alloc(1)
    view[0][-1, 3], view[2][-1, 5] = float("inf"), float("-inf")
    wt = torch.randn(Cin, Cout, device="cuda:0", generator=gen).to(torch.bfloat16)
    wt.masked_fill_(wt == 0, 0.5)
    scale = torch.rand(Cout, device="cuda:0", generator=gen) + 0.5
    fwd = dl.LayerDesc(x=0, res=dl.NO_TENSOR, y=1, dtype=dl.DTYPE_BF16, w=wt.data_ptr(), scale=scale.data_ptr(), shift=scale.data_ptr(), N=1, H=H, W=W,
                       Cin=Cin, Cout=Cout, R=1, S=1, stride=1, pad=0, relu=0)
    ws = torch.full((d.backward_workspace(fwd),), 255, dtype=torch.uint8, device="cuda:0")
    gw = torch.full((Cout, Cin), float("nan"), device="cuda:0")
    desc = dl.BwdDesc(fwd=fwd, gy=2, gpre=2, gx=3, gx_add=4 if add else dl.NO_TENSOR, mask_gx=1, wt=wt.data_ptr(), gw=gw.data_ptr(),
                      workspace=ws.data_ptr(), workspace_bytes=ws.numel())
    assert d.backward_kernel(desc).endswith(JOINT)
    torch.cuda.synchronize()
    d.backward_segment([desc])
    d.sync()
    xf, gf = view[0].double(), view[2].double()
    ref_gw = (gf.t().contiguous() @ xf) * scale.double()[:, None]
    ref_gx = gf @ wt.double().t().contiguous() + (view[4].double() if add else 0.0)
    ref_gx = torch.where(xf > 0, ref_gx, torch.zeros_like(ref_gx))
    gx = d.arena[d.tensor_ptr(3) - d.arena.data_ptr():][:nbytes[3]].view(torch.bfloat16).reshape(M, Cin).double()
    for got, ref, most in ((gw.double(), ref_gw, 1e-5), (gx, ref_gx, 4e-3)):
        inf = torch.isinf(ref)
        assert bool(inf.any()) and not bool(torch.isnan(ref).any())
        assert torch.equal(got[inf], ref[inf])
        assert float((got[~inf] - ref[~inf]).abs().max() / ref[~inf].abs().max()) <= most
    d.close()


@pytest.mark.parametrize("Cin,Cout,H,W,add", [(64, 256, 131, 193, False), (64, 256, 97, 89, False), (64, 256, 1, 12545, False), (128, 512, 131, 193, False),
                                              (64, 512, 101, 109, False), (128, 512, 9001, 1, False), (64, 256, 1, 7000, False), (64, 256, 1, 6999, False),
                                              (64, 512, 95, 95, False), (64, 256, 131, 193, True), (128, 256, 131, 193, False), (192, 256, 97, 89, False),
                                              (448, 256, 97, 89, False)])
def test_own_mask_on_the_way(torch_mod, Cin, Cout, H, W, add):  # noqa: F811
    """A layer with a ReLU of its own: gpre and gx carry the bits of the mask's own launch followed by the masked layer, gw its sums in another order
    (bound as in the helper above).  Chunks of 32 pixels, ragged ends, slices; the last six run the mask's launch."""
    torch = torch_mod
    import paper_2203_15980_amd as dl
    M = H * W
    nbytes = [M * Cin * 2, M * Cout * 2, M * Cout * 2, M * Cin * 2, M * Cin * 2, M * Cout * 2, M * Cin * 2]    # x, y, gy, gx, gx_add, gpre, gx apart
    d = make_delta(torch, sum(nbytes) + (2 << 20))
    d.bind(nbytes)
    gen = torch.Generator(device="cuda:0").manual_seed(43)
    view = lambda t, C: d.arena[d.tensor_ptr(t) - d.arena.data_ptr():][:nbytes[t]].view(torch.int16).reshape(M, C)      # noqa: E731
    for t, C in ((0, Cin), (1, Cout), (2, Cout), (4, Cin)):
        d.alloc(t)
        view(t, C).view(torch.bfloat16).normal_(generator=gen)
    y = view(1, Cout)
    y[0, :8] = torch.tensor([0, -32768, 1, 0x7F80, 0x7F81, -128, -1, 0x3F80], dtype=torch.int16, device="cuda:0")      # zeros, infinities, NaN
    wt = torch.randn(Cin, Cout, device="cuda:0", generator=gen).to(torch.bfloat16)
    scale = torch.rand(Cout, device="cuda:0", generator=gen) + 0.5
    fwd = dl.LayerDesc(x=0, res=dl.NO_TENSOR, y=1, dtype=dl.DTYPE_BF16, w=wt.data_ptr(), scale=scale.data_ptr(), shift=scale.data_ptr(), N=1, H=H, W=W,
                       Cin=Cin, Cout=Cout, R=1, S=1, stride=1, pad=0, relu=1)
    ws = torch.full((d.backward_workspace(fwd),), 255, dtype=torch.uint8, device="cuda:0")
    gw = [torch.full((Cout, Cin), float("nan"), device="cuda:0") for _ in range(3)]
    b = lambda gy, gpre, gx, masked, i: dl.BwdDesc(fwd=fwd, gy=gy, gpre=gpre, gx=gx, gx_add=4 if add else dl.NO_TENSOR, mask_gx=1, gy_masked=masked,  # noqa: E731
                                                   wt=wt.data_ptr(), gw=gw[i].data_ptr(), workspace=ws.data_ptr(), workspace_bytes=ws.numel())
    own = b(2, 5, 3, 0, 0)
    assert d.backward_kernel(own).endswith(JOINT)
    assert d.backward_kernel(own).startswith("gpre: joint1x1 bf16; ") == (
        not add and (Cin, Cout, M < {256: 7000, 512: 11000}[Cout]) in ((64, 256, False), (64, 512, False), (128, 512, True), (128, 512, False))), d.backward_kernel(own)
    torch.cuda.synchronize()
    d.backward_segment([own])
    d.sync()
    gpre, gx = view(5, Cout).clone(), view(3, Cin).clone()
    want = torch.where((y > 0) & (y < 0x7F81), view(2, Cout), torch.zeros_like(y))
    assert torch.equal(gpre, want)
    view(5, Cout).fill_(0x7FC1)
    torch.cuda.synchronize()
    d.backward_segment([b(2, 5, 3, 0, 1), b(5, 5, 6, 1, 2)])     # again; and on the gradient as it left it
    d.sync()
    assert torch.equal(view(5, Cout), want) and torch.equal(view(3, Cin), gx) and torch.equal(view(6, Cin), gx)
    assert torch.equal(gw[0], gw[1])
    ref = (gpre.view(torch.bfloat16).double().t().contiguous() @ view(0, Cin).view(torch.bfloat16).double()) * scale.double()[:, None]
    for g in gw:
        assert float((g.double() - ref).abs().max() / ref.abs().max()) <= 1e-5
    d.close()


def test_own_mask_without_room_for_gx(torch_mod):  # noqa: F811
    """The arena holds gpre and not gx: the call says so, and gpre, resident from then on, is gy * [y > 0] and not what its memory held."""
    torch = torch_mod
    import paper_2203_15980_amd as dl
    H, W, Cin, Cout = 131, 193, 64, 256
    M = H * W
    nbytes = [M * Cin * 2, M * Cout * 2, M * Cout * 2, M * Cin * 2, M * Cout * 2]      # x, y, gy, gx, gpre
    arena = torch.full((sum(nbytes) - nbytes[3] // 2,), 0x5A, dtype=torch.uint8, device="cuda:0")
    d = dl.Delta(arena, torch.cuda.current_stream().cuda_stream)
    d.bind(nbytes)
    gen = torch.Generator(device="cuda:0").manual_seed(47)
    view = lambda t: d.arena[d.tensor_ptr(t) - d.arena.data_ptr():][:nbytes[t]].view(torch.int16).reshape(M, -1)      # noqa: E731
    for t in (0, 1, 2):
        d.alloc(t)
        view(t).view(torch.bfloat16).normal_(generator=gen)
    w, one, gw = torch.zeros(Cin, Cout, dtype=torch.bfloat16, device="cuda:0"), torch.ones(Cout, device="cuda:0"), torch.zeros(Cout, Cin, device="cuda:0")
    fwd = dl.LayerDesc(x=0, res=dl.NO_TENSOR, y=1, dtype=dl.DTYPE_BF16, w=w.data_ptr(), scale=one.data_ptr(), shift=one.data_ptr(), N=1, H=H, W=W,
                       Cin=Cin, Cout=Cout, R=1, S=1, stride=1, pad=0, relu=1)
    ws = torch.zeros(d.backward_workspace(fwd), dtype=torch.uint8, device="cuda:0")
    desc = dl.BwdDesc(fwd=fwd, gy=2, gpre=4, gx=3, gx_add=dl.NO_TENSOR, mask_gx=1, wt=w.data_ptr(), gw=gw.data_ptr(), workspace=ws.data_ptr(),
                      workspace_bytes=ws.numel())
    assert d.backward_kernel(desc).endswith(JOINT)
    torch.cuda.synchronize()
    with pytest.raises(dl.DeltaError) as e:
        d.backward_segment([desc])
    d.sync()
    assert e.value.status == dl.ERR_OOM_ARENA
    assert torch.equal(view(4), torch.where(view(1) > 0, view(2), torch.zeros_like(view(2))))
    d.close()
