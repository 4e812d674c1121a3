"""Both gradients of a layer in one launch, against float64 on the stored operands (products on the GPU, no kernel of the library): edges of
the tiles and steps, every form of the layer, and both sides of the dispatch's lines.

Tolerances, of the largest entry: dL/dx in bf16 one rounding, 2^-9, 4e-3 with the fp32 sums' share; in fp32 sums of at most 2304 products, split over
wavefronts, 1e-5; dL/dw exact products summed in fp32 over at most 8200 terms in runs of an eighth, 1e-5 (about sqrt(8200) * 2^-24 with a
margin of two)."""
import numpy as np
import pytest

from test_gpu_parity import make_delta, torch_mod  # noqa: F401

pytestmark = pytest.mark.gpu

SAME, CLASS, OWN = "the same launch", "the launch of one class", "small_backward bf16, compute stream"
CASES = [
    # dtype  N   H    W   Cin Cout R stride  add mask  what the weight gradient's part of the kernel's name ends with
    ("bf16", 1,  1,   1,   64,  64, 1, 1, False, False, SAME),       # one position, one step of one wavefront
    ("bf16", 1,  3,  11,   64, 128, 1, 1, True,  True,  SAME),       # 33 positions: a second step of one row
    ("bf16", 2,  8,  16,   64,  64, 1, 1, False, True,  SAME),       # 256 positions: exactly one step each
    ("bf16", 1,  19, 27,  192, 320, 1, 1, True,  False, SAME),       # 513: a second round of one position; odd counts of tiles
    ("bf16", 2,  5,   7,  512, 1024, 1, 1, True, True,  SAME),       # the wider tile of gw, steps of 16 positions, five rounds
    ("bf16", 1,  1,   1,   64,  64, 3, 1, True,  True,  SAME),       # only the centre tap
    ("bf16", 5,  3,   1,   64, 128, 3, 1, False, True,  SAME),       # images one pixel wide
    ("bf16", 3,  7,   7,  256, 256, 3, 1, True,  True,  SAME),       # the wider tile with taps
    ("bf16", 2,  9,  11,  128,  64, 3, 1, True,  False, SAME),
    ("bf16", 3,  12, 10,   64, 128, 3, 1, False, False, SAME),
    ("bf16", 2,  9,  13,  128,  64, 1, 2, True,  True,  SAME),       # strided 1x1: positions pick their pixels
    ("bf16", 1,  7,   8,   64,  64, 1, 3, False, False, SAME),
    ("bf16", 2,  9,  12,   64, 128, 3, 2, True,  True,  CLASS),      # strided 3x3, class by class
    ("bf16", 1,  2,   2,   64,  64, 3, 2, False, False, CLASS),
    ("bf16", 2,  9,  12,  128, 128, 3, 2, True,  True,  OWN),        # its data gradient in one launch
    ("bf16", 1,  64, 64,   64,  64, 1, 1, False, True,  SAME),       # 4096 positions: the last that go this way with few tiles of gw
    ("bf16", 1,  64, 65,   64,  64, 1, 1, False, True,  "joint1x1 bf16, the same launch"),
    ("bf16", 1,  64, 100, 256, 256, 1, 1, False, True,  SAME),       # 6400: the last with 64
    ("bf16", 1,  40, 40, 1024, 512, 1, 1, True,  True,  SAME),       # eight steps: 1600 tiles of gx are the last
    ("bf16", 1,   1, 1601, 1024, 512, 1, 1, True, True, "wgrad1x1 bf16, second stream"),
    ("bf16", 1,  79, 80, 1024, 512, 1, 2, False, True,  SAME),
    ("bf16", 1,   1, 3201, 1024, 512, 1, 2, False, True, "wgrad1x1 bf16, second stream"),
    ("bf16", 1,  64, 64, 1024,  64, 1, 1, False, True,  SAME),       # one step: 4096
    ("bf16", 1,  17, 241, 1024, 64, 1, 1, False, True,  "joint1x1 bf16, the same launch"),
    ("bf16", 1,  64, 80,  512,  64, 3, 1, False, True,  SAME),       # nine: 2560
    ("bf16", 1, 197,  26,  512,  64, 3, 1, False, True, "wgrad3x3 bf16, second stream"),         # 2576
    ("bf16", 1,  58, 64,  512, 128, 3, 1, True,  True,  SAME),       # 1856 tiles, 34988 by the sum
    ("bf16", 1,  47, 79,  512, 128, 3, 1, True,  True,  "wgrad3x3 bf16, second stream"),        # 1872, 35157
    ("bf16", 10, 14, 14,  256, 256, 3, 1, True,  True,  SAME),       # 1960 pixels: the wider tile of gw
    ("bf16", 16, 14, 14,  256, 256, 3, 1, True,  True,  SAME),       # 3136: the narrow one, 576 of them; 3.7 GFLOP
    ("bf16", 1,  56, 56,  256,  64, 1, 1, True,  True,  SAME),
    ("f32",  1,  1,   1,   32,  64, 1, 1, True,  True,  SAME),
    ("f32",  1,  3,  11,   96,  32, 1, 1, False, True,  SAME),       # 33 positions: 8 to a wavefront, the fifth has one
    ("f32",  2,  7,  13,   64,  96, 3, 1, True,  True,  SAME),
    ("f32",  5,  1,   2,   32,  32, 3, 1, False, False, SAME),       # two images to a step of four positions
    ("f32",  1,  33, 31,   64,  32, 1, 1, True,  False, SAME),       # 128 to a wavefront: one round and a half
    ("f32",  2,  6,  11,  256, 128, 3, 1, True,  True,  SAME),       # 32 x 32 tiles
    ("f32",  1,  64, 128,  32,  32, 1, 1, False, True,  SAME),       # 8192 positions: the last that go this way
    ("f32",  1,  64, 129,  32,  32, 1, 1, False, True,  "wgrad_f32 16x16, 32-bit offsets, compute stream"),
    ("f32",  1,  48,  32, 2048, 64, 1, 1, True,  True,  SAME),       # two steps: no line for the tiles of gx, 3072 here
    ("f32",  1,  64,  32, 1024, 128, 1, 1, False, True, SAME),       # four steps: 2048 tiles are the last
    ("f32",  1,   3, 683, 1024, 128, 1, 1, False, True, "wgrad_f32 16x16, 32-bit offsets, compute stream"),
    ("f32",  1,  48,  32, 1024, 256, 1, 1, True,  True, SAME),       # eight: 1536
    ("f32",  1,  29,  53, 1024, 256, 1, 1, True,  True, "wgrad_f32 32x32, 32-bit offsets, compute stream"),
    ("f32",  1,  64,  64, 512, 512, 1, 1, False,  True, SAME),       # sixteen: 2048
    ("f32",  1,  17, 241, 512, 512, 1, 1, False,  True, "wgrad_f32 32x32, 32-bit offsets, second stream"),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "%s_%dx%dx%d_%d_%d_r%d_s%d" % c[:8])
def test_both_gradients_match_float64(torch_mod, case):  # noqa: F811
    torch = torch_mod
    import paper_2203_15980_amd as dl
    dtype, N, H, W, Cin, Cout, R, stride, add, mask, ends = case
    print("case", case, flush=True)
    t, code, es = (torch.float32, dl.DTYPE_F32, 4) if dtype == "f32" else (torch.bfloat16, dl.DTYPE_BF16, 2)
    P, Q, pad = (H - 1) // stride + 1, (W - 1) // stride + 1, R // 2
    xb, yb = N * H * W * Cin * es, N * P * Q * Cout * es
    # tensors: 0 x, 1 y, 2 gy, 3 gx, 4 gx_add, 5 gpre at the input's resolution (a strided 3x3 layer that has to spread its gradient)
    nbytes = [xb, yb, yb, xb, xb, N * H * W * Cout * es]
    d = make_delta(torch, sum(nbytes) + (2 << 20))
    d.bind(nbytes)
    gen = torch.Generator(device="cuda:0").manual_seed(23)
    view = {}
    for i, shape in ((0, (N, H, W, Cin)), (2, (N, P, Q, Cout)), (4, (N, H, W, Cin))):
        d.alloc(i)
        view[i] = d.arena[d.tensor_ptr(i) - d.arena.data_ptr():][:nbytes[i]].view(t).reshape(shape)
        view[i].normal_(generator=gen)
    rnd = lambda *s: torch.randn(*s, device="cuda:0", generator=gen)            # noqa: E731
    w, scale, zeros = rnd(Cout, R, R, Cin).to(t), rnd(Cout) * 0.3 + 1.0, torch.zeros(Cout, device="cuda:0")
    fwd = dl.LayerDesc(x=0, res=dl.NO_TENSOR, y=1, dtype=code, w=w.data_ptr(), scale=scale.data_ptr(), shift=zeros.data_ptr(), N=N, H=H, W=W,
                       Cin=Cin, Cout=Cout, R=R, S=R, stride=stride, pad=pad, relu=0)
    wt = torch.empty(Cin, R, R, Cout, dtype=t, device="cuda:0")
    d.bwd_weights(fwd, wt.data_ptr())
    ws = torch.full((max(d.backward_workspace(fwd), 256),), 255, dtype=torch.uint8, device="cuda:0")      # NaN wherever nothing is written
    spread = stride > 1 and R == 3 and (Cin % 128 or Cout % 128)
    gx, gw = [], []
    for _ in range(2):
        out = torch.full((Cout, R, R, Cin), float("nan"), device="cuda:0")
        desc = dl.BwdDesc(fwd=fwd, gy=2, gpre=5 if spread else 2, gx=3, gx_add=4 if add else dl.NO_TENSOR, mask_gx=int(mask), wt=wt.data_ptr(),
                          gw=out.data_ptr(), workspace=ws.data_ptr(), workspace_bytes=ws.numel())
        assert d.backward_kernel(desc).endswith(ends), d.backward_kernel(desc)
        torch.cuda.synchronize()
        d.backward_segment([desc])
        d.backward_join()
        d.sync()
        gw.append(out.clone())
        gx.append(d.arena[d.tensor_ptr(3) - d.arena.data_ptr():][:xb].view(t).reshape(N, H, W, Cin).clone())
    xf, gf, wf = view[0].double(), view[2].double().reshape(N * P * Q, Cout), wt.double()
    xp = torch.nn.functional.pad(xf, (0, 0, pad, pad, pad, pad))
    ref_gw, gp = torch.empty(Cout, R, R, Cin, dtype=torch.float64, device="cuda:0"), torch.zeros_like(xp)
    for r in range(R):
        for s in range(R):
            at = (slice(None), slice(r, r + stride * (P - 1) + 1, stride), slice(s, s + stride * (Q - 1) + 1, stride))
            ref_gw[:, r, s] = gf.t().contiguous() @ xp[at].reshape(N * P * Q, Cin).contiguous()
            gp[at] += (gf @ wf[:, R - 1 - r, R - 1 - s].t().contiguous()).reshape(N, P, Q, Cin)
    ref_gw *= scale.double()[:, None, None, None]
    ref_gx = gp[:, pad:pad + H, pad:pad + W]
    if R == 1 and stride > 1 and dtype == "bf16":                                # stored once before it is spread out
        ref_gx = ref_gx.to(t).double()
    if add:
        ref_gx = ref_gx + view[4].double()
    if mask:
        ref_gx = ref_gx * (xf > 0)
    rel = lambda a, b: float((a.double() - b).abs().max() / b.abs().max())       # noqa: E731
    ex, ew = rel(gx[0], ref_gx), rel(gw[0], ref_gw)
    print("  gx %.2e gw %.2e" % (ex, ew), flush=True)
    assert np.isfinite(ew) and ew <= 1e-5 and np.isfinite(ex) and ex <= (1e-5 if dtype == "f32" else 4e-3)
    assert torch.equal(gx[0], gx[1]) and torch.equal(gw[0], gw[1])
    d.close()


def test_padding_spreads_no_infinity(torch_mod):  # noqa: F811
    """A pixel outside the image meets the gradient nowhere: an infinite gradient in the first row and column reaches the taps that read pixels
    for it, and leaves the tap that looks up and left from there finite."""
    torch = torch_mod
    import paper_2203_15980_amd as dl
    N, H, W, C = 1, 5, 6, 64
    nbytes = [N * H * W * C * 2] * 4
    d = make_delta(torch, sum(nbytes) + (1 << 20))
    d.bind(nbytes)
    view = {}
    for i in (0, 2):
        d.alloc(i)
        view[i] = d.arena[d.tensor_ptr(i) - d.arena.data_ptr():][:nbytes[i]].view(torch.bfloat16).reshape(N, H, W, C)
        view[i].fill_(1.0)
    view[2][0, 0, :, 0] = view[2][0, :, 0, 0] = float("inf")
    w, one = torch.zeros(C * 9 * C, dtype=torch.bfloat16, device="cuda:0"), torch.ones(C, device="cuda:0")
    fwd = dl.LayerDesc(x=0, res=dl.NO_TENSOR, y=1, dtype=dl.DTYPE_BF16, w=w.data_ptr(), scale=one.data_ptr(), shift=one.data_ptr(), N=N, H=H, W=W,
                       Cin=C, Cout=C, R=3, S=3, stride=1, pad=1, relu=0)
    ws = torch.empty(max(d.backward_workspace(fwd), 256), dtype=torch.uint8, device="cuda:0")
    gw = torch.empty(C, 3, 3, C, device="cuda:0")
    torch.cuda.synchronize()
    d.backward_segment([dl.BwdDesc(fwd=fwd, gy=2, gpre=2, gx=3, gx_add=dl.NO_TENSOR, wt=w.data_ptr(), gw=gw.data_ptr(), workspace=ws.data_ptr(),
                                   workspace_bytes=ws.numel())])
    d.sync()
    assert bool((gw[0, 0, 0] == (H - 1) * (W - 1)).all()) and bool(torch.isinf(gw[0, 1, 1]).all()) and bool(torch.isfinite(gw[1:]).all())
    d.close()


@pytest.mark.parametrize("form", [(64, 64, 1, 1, False), (64, 128, 3, 1, False), (128, 64, 1, 2, False), (64, 64, 3, 2, True), (128, 128, 3, 2, True)],
                         ids=lambda f: "%d_%d_r%d_s%d_relu%d" % f)
def test_both_gradients_count_the_work_of_either(torch_mod, form):  # noqa: F811
    """recompute_flops counts the work as launched: for both gradients together what they count one by one (a strided 3x3 layer with a ReLU mask of
    its own runs both on the spread gradient, at the input's resolution)."""
    torch = torch_mod
    import paper_2203_15980_amd as dl
    Cin, Cout, R, stride, relu = form
    N, H, W = 2, 9, 12
    P, Q = (H - 1) // stride + 1, (W - 1) // stride + 1
    xb, yb = N * H * W * Cin * 2, N * P * Q * Cout * 2
    nbytes = [xb, yb, yb, xb, N * H * W * Cout * 2]
    d = make_delta(torch, sum(nbytes) + (2 << 20))
    d.bind(nbytes)
    for t in (0, 1, 2):
        d.alloc(t)
        d.arena[d.tensor_ptr(t) - d.arena.data_ptr():][:nbytes[t]].view(torch.bfloat16).normal_()
    w, one = torch.randn(Cout * R * R * Cin, device="cuda:0").bfloat16(), torch.ones(max(Cin, Cout), device="cuda:0")
    fwd = dl.LayerDesc(x=0, res=dl.NO_TENSOR, y=1, dtype=dl.DTYPE_BF16, w=w.data_ptr(), scale=one.data_ptr(), shift=one.data_ptr(), N=N, H=H, W=W,
                       Cin=Cin, Cout=Cout, R=R, S=R, stride=stride, pad=R // 2, relu=int(relu))
    ws, gw = torch.empty(max(d.backward_workspace(fwd), 256), dtype=torch.uint8, device="cuda:0"), torch.empty(Cout * R * R * Cin, device="cuda:0")
    count = {}
    for what in ("both", "gx", "gw"):
        desc = dl.BwdDesc(fwd=fwd, gy=2, gpre=4 if relu else 2, gx=dl.NO_TENSOR if what == "gw" else 3, gx_add=dl.NO_TENSOR, wt=w.data_ptr(),
                          gw=None if what == "gx" else gw.data_ptr(), workspace=ws.data_ptr(), workspace_bytes=ws.numel())
        if what == "both":
            assert d.backward_kernel(desc).endswith(SAME), d.backward_kernel(desc)
        before = d.stats()["recompute_flops"]
        torch.cuda.synchronize()
        d.backward_segment([desc])
        d.sync()
        count[what] = d.stats()["recompute_flops"] - before
    assert count["both"] == count["gx"] + count["gw"], count
    d.close()
