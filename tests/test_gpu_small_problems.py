"""Layers that cannot fill the chip: the split-reduction convolution kernel and the fp32 weight gradient against the
CPU oracle, at the edges of their tiles and of the range that the dispatch gives them.

Tolerances: bf16 one rounding of the output, half an ulp = 2^-9 of the element, of which the maximum is at most
2^-9 of the tensor's maximum (4e-3 leaves the fp32 sums their share); fp32 sums of up to 2304 products of
unit-scale operands, at most 2304 * 2^-24 = 1.4e-4 relative in the worst order, 1e-5 for sums split over
wavefronts (about the square root of that)."""
import numpy as np
import pytest

import synth
from oracle import numeric as on
from test_gpu_parity import make_delta, rel_err, single, torch_mod  # noqa: F401

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-5, "bf16": 4e-3}

CASES = [
    # name              N   H   W  Cin Cout R st relu  res  (kernel, where it is not the split-reduction one: by type)
    ("one_tile",        1,  4,  8, 128,  32, 1, 1, True, False),     # exactly 32 pixels x 32 channels, one or two steps
    ("ragged_tile",     1,  3, 11, 192,  40, 1, 1, True, True),      # 33 pixels, 40 channels
    ("one_pixel",       1,  1,  1, 256,   8, 3, 1, False, False),    # only the centre tap; 8 channels
    ("odd_steps",       2,  5,  7, 320, 136, 1, 1, False, True),     # five steps: not every wavefront has one
    ("pad_s2",          2,  9, 12, 128, 128, 3, 2, True, False),
    ("long",            1,  7,  9, 256,  64, 3, 1, True, True),
    ("5x5",             1,  6,  5,  64,  72, 5, 1, True, False),
    ("at_the_line",     1, 64, 80, 128, 128, 1, 1, True, False),     # 160 x 4 tiles: the last of the short reductions
    ("past_the_line",   1, 64, 81, 128, 128, 1, 1, True, False, {"f32": "conv_igemm f32", "bf16": "conv1x1_stream"}),    # 162 x 4: the kernel for larger layers
    ("halo_past_the_line", 3, 75, 73, 192, 64, 3, 1, True, True, {"f32": "conv_igemm f32", "bf16": "conv3x3_halo bf16 128x64"}),    # 514 x 2 tiles of 27 steps, ragged, odd width
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_few_tile_layers_match_oracle(torch_mod, dtype, case):  # noqa: F811
    torch = torch_mod
    import paper_2203_15980_amd as dl
    name, N, H, W, Cin, Cout, R, stride, relu, res = case[:10]
    kernel = case[10][dtype] if len(case) > 10 else "conv_splitk"
    print("case", name, dtype, flush=True)
    l = single(name, N, H, W, Cin, Cout, R, stride, R // 2, relu, res)
    es, master = (4 if dtype == "f32" else 2), 79
    x, p = synth.make_input(master, (N, H, W, Cin), dtype), synth.make_params(master, l, dtype)
    yshape = (N, l.P, l.Q, Cout)
    r = None
    if res:
        r = synth.normal(master, 999, int(np.prod(yshape))).astype(np.float32).reshape(yshape)
        r = r if dtype == "f32" else synth.f32_to_bf16_bits(r).reshape(yshape)
    ref = on.conv_bn_act(x, p["w"], p, res=r, stride=stride, pad=R // 2, relu=relu, dtype=dtype)
    nbytes = [x.nbytes, int(np.prod(yshape)) * es, int(np.prod(yshape)) * es]
    d = make_delta(torch, sum(nbytes) + (1 << 20))
    d.bind(nbytes)
    base = d.arena.data_ptr()
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")       # noqa: E731
    at = lambda t: d.arena[d.tensor_ptr(t) - base:][:nbytes[t]]                  # noqa: E731
    for t, a in ((0, x), (1, r)):
        if a is not None:
            d.alloc(t)
            at(t).copy_(dev(a.view(np.uint8).reshape(-1)))
    w, bn = dev(p["w"]), [dev(p[k]) for k in ("gamma", "beta", "mean", "var")]
    scale, shift = torch.empty(Cout, device="cuda:0"), torch.empty(Cout, device="cuda:0")
    d.bn_fold(*[b.data_ptr() for b in bn], float(p["eps"]), Cout, scale.data_ptr(), shift.data_ptr())
    desc = dl.LayerDesc(x=0, res=1 if res else dl.NO_TENSOR, y=2, dtype=dl.DTYPE_F32 if dtype == "f32" else dl.DTYPE_BF16,
                        w=w.data_ptr(), scale=scale.data_ptr(), shift=shift.data_ptr(), N=N, H=H, W=W, Cin=Cin, Cout=Cout, R=R,
                        S=R, stride=stride, pad=R // 2, relu=1 if relu else 0)
    assert kernel in d.layer_kernel(desc), d.layer_kernel(desc)
    got = []
    for _ in range(2):                                                          # the same bits both times
        d.recompute_segment([desc])
        d.sync()
        got.append(at(2).cpu().numpy().view(np.float32 if dtype == "f32" else np.uint16).reshape(yshape).copy())
    err = rel_err(got[0], ref, dtype)
    print("  err %.2e" % err, flush=True)
    assert err <= TOL[dtype] and np.array_equal(got[0], got[1])
    d.close()


@pytest.mark.parametrize("case", [("one_chunk", 1, 1, 3, 32, 16, 1), ("ragged", 1, 9, 13, 96, 48, 3), ("narrow_image", 2, 7, 1, 32, 32, 3),
                                  ("wide_tiles", 2, 6, 11, 256, 128, 3), ("odd_tiles", 1, 12, 17, 160, 48, 1)], ids=lambda c: c[0])
def test_fp32_weight_gradient_matches_float64(torch_mod, case):  # noqa: F811
    """The weight gradient alone (x and gy as they are): both tile sizes, fewer positions than wavefronts, images
    narrower than one step."""
    torch = torch_mod
    import paper_2203_15980_amd as dl
    name, N, H, W, Cin, Cout, R = case
    print("case", name, flush=True)
    rnd = lambda aid, shape: synth.normal(93, aid, int(np.prod(shape))).astype(np.float32).reshape(shape)   # noqa: E731
    x, gy, scale = rnd(1, (N, H, W, Cin)), rnd(2, (N, H, W, Cout)), rnd(3, (Cout,)) + 2.0
    nbytes = [x.nbytes, gy.nbytes, gy.nbytes]
    d = make_delta(torch, sum(nbytes) + (1 << 20))
    d.bind(nbytes)
    base = d.arena.data_ptr()
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")       # noqa: E731
    for t, a in ((0, x), (2, gy)):
        d.alloc(t)
        d.arena[d.tensor_ptr(t) - base:][:nbytes[t]].copy_(dev(a.view(np.uint8).reshape(-1)))
    sc, zeros, w = dev(scale), torch.zeros(Cout, device="cuda:0"), torch.zeros(Cout * R * R * Cin, device="cuda:0")
    ws = torch.empty(256, dtype=torch.uint8, device="cuda:0")
    gw = torch.full((Cout, R, R, Cin), float("nan"), device="cuda:0")
    fwd = dl.LayerDesc(x=0, res=dl.NO_TENSOR, y=1, dtype=dl.DTYPE_F32, w=w.data_ptr(), scale=sc.data_ptr(), shift=zeros.data_ptr(), N=N,
                       H=H, W=W, Cin=Cin, Cout=Cout, R=R, S=R, stride=1, pad=R // 2, relu=0)
    desc = dl.BwdDesc(fwd=fwd, gy=2, gpre=2, gx=dl.NO_TENSOR, gx_add=dl.NO_TENSOR, gw=gw.data_ptr(), workspace=ws.data_ptr(),
                      workspace_bytes=256)
    d.backward_segment([desc])
    d.sync()
    pad = R // 2
    xp = np.pad(x.astype(np.float64), ((0, 0), (pad, pad), (pad, pad), (0, 0)))
    ref = np.empty((Cout, R, R, Cin))
    for r in range(R):
        for s in range(R):
            ref[:, r, s] = np.einsum("nhwk,nhwc->kc", gy.astype(np.float64), xp[:, r:r + H, s:s + W])
    ref *= scale.astype(np.float64)[:, None, None, None]
    err = float(np.max(np.abs(gw.cpu().numpy() - ref)) / np.max(np.abs(ref)))
    print("  err %.2e" % err, flush=True)
    assert err <= TOL["f32"]
    d.close()
