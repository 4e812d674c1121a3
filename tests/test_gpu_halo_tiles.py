"""The 3x3 layers that keep their input halo in LDS, at both tile heights and every width at which the rule or the number
of halo loads changes, against the CPU oracle with the bound derived beside the helper, which also asserts the kernel."""
import pytest

import test_gpu_small_problems as layers
from test_gpu_parity import make_delta, torch_mod  # noqa: F401

pytestmark = pytest.mark.gpu

HIGH, LOW = {"bf16": "conv3x3_halo bf16 256x64"}, {"bf16": "conv3x3_halo bf16 128x64"}
PIECES = {n: {"bf16": "conv3x3_halo bf16 256x64 (8x1 waves), last tiles in %d pieces" % n} for n in (2, 4, 8)}
CASES = [
    # name           N  H    W   Cin Cout R st relu  res
    ("past_256_w31",      1, 133, 31,  64, 512, 3, 1, True, False, HIGH),      # 17 x 8 workgroups of 256 pixels, the last with 27
    ("past_256_w32",      2, 64,  32, 128, 512, 3, 1, False, True, HIGH),      # 16 x 8: the first that takes 256; two channel blocks
    ("past_256_w63",      1, 66,  63,  64, 512, 3, 1, True, True, HIGH),
    ("past_128_w31",      1, 83,  31,  64, 256, 3, 1, True, True, LOW),       # 21 x 4 workgroups of 128 pixels
    ("past_128_w32",      9, 9,   32, 128, 256, 3, 1, True, False, LOW),
    ("past_128_w63",      1, 41,  63,  64, 256, 3, 1, False, False, LOW),
    # past a whole round of the chip the last tiles go out in pieces of 32, 64 and 128 pixels
    ("pieces_32_w31",     1, 273, 31,  64, 512, 3, 1, True, True, PIECES[8]),      # 34 x 8 workgroups: 16 tiles, half of them with 15 pixels
    ("pieces_32_w62",     1, 146, 62, 128, 512, 3, 1, False, False, PIECES[8]),    # 36 x 8: 32 tiles in eight pieces, the most
    ("pieces_64_w63",     1, 159, 63,  64, 512, 3, 1, True, False, PIECES[4]),     # 40 x 8: 64 tiles in four
    ("pieces_128_w33",    2, 184, 33,  64, 512, 3, 1, True, True, PIECES[2]),      # 48 x 8: 128 tiles in two
    ("whole_again_w33",   1, 373, 33,  64, 512, 3, 1, True, False, HIGH),     # 49 x 8: 136 tiles, whole
    ("past_wide_w64",     1, 65,  64,  64, 512, 3, 1, True, False, LOW),      # enough pixels for 256, rows too long for it
    ("past_wide_w127",    1, 33, 127,  64, 512, 3, 1, True, True, LOW),       # the longest halo
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_halo_tiles_match_oracle(torch_mod, case):  # noqa: F811
    layers.test_few_tile_layers_match_oracle(torch_mod, "bf16", case)


@pytest.mark.parametrize("H,W,Cin,Cout,R,name", [(256, 32, 64, 512, 3, "conv3x3_halo bf16 256x64 (8x1 waves)"),                    # 32 x 8 workgroups: one round
                                                 (257, 32, 64, 512, 3, "conv3x3_halo bf16 256x64 (8x1 waves), last tiles in 8 pieces"),
                                                 (373, 33, 64, 512, 3, "conv3x3_halo bf16 256x64 (8x1 waves)"),                    # 136 tiles past a round
                                                 (149, 149, 256, 1024, 1, "gemm_nt bf16 256x256 (64x64 per wave, direct-to-LDS), last tiles in 2 pieces"),
                                                 (197, 149, 256, 1024, 1, "gemm_nt bf16 256x256 (64x64 per wave, direct-to-LDS)")])     # 115 x 4: 204 past a round
def test_pieces_are_named_where_tiles_are_cut(torch_mod, H, W, Cin, Cout, R, name):  # noqa: F811
    import paper_2203_15980_amd as dl
    d, one = make_delta(torch_mod, 1 << 20), torch_mod.ones(16, device="cuda:0")
    d.bind([H * W * Cin * 2, H * W * Cout * 2])
    got = d.layer_kernel(dl.LayerDesc(x=0, res=dl.NO_TENSOR, y=1, dtype=dl.DTYPE_BF16, w=one.data_ptr(), scale=one.data_ptr(), shift=one.data_ptr(), N=1,
                                      H=H, W=W, Cin=Cin, Cout=Cout, R=R, S=R, stride=1, pad=R // 2, relu=0))
    d.close()
    assert got == name


def test_tiles_go_out_whole_beside_the_second_stream(torch_mod):  # noqa: F811
    """A data gradient without a mask whose layer's weight gradient, or an earlier one, is on the second stream, and a forward launch beside one: whole
    tiles.  Alone, and after the join: pieces.  The same bits all ways."""
    torch = torch_mod
    import paper_2203_15980_amd as dl
    N, H, W, C = 2, 273, 33, 256                                 # 71 x 4 workgroups: 28 past a round
    n = N * H * W * C * 2
    d = make_delta(torch, 8 * n)
    d.bind([n] * 6)                                              # x, y, gy, gx (beside its own), gx (alone), y of the forward launch
    gen = torch.Generator(device="cuda:0").manual_seed(61)
    view = lambda t: d.arena[d.tensor_ptr(t) - d.arena.data_ptr():][:n]                          # noqa: E731
    for t in (0, 1, 2):
        d.alloc(t)
        view(t).view(torch.bfloat16).normal_(generator=gen)
    w = torch.randn(C * 9 * C, device="cuda:0", generator=gen).to(torch.bfloat16)
    one, gw = torch.ones(C, device="cuda:0"), torch.zeros(C * 9 * C, device="cuda:0")
    lay = lambda y: dl.LayerDesc(x=0, res=dl.NO_TENSOR, y=y, dtype=dl.DTYPE_BF16, w=w.data_ptr(), scale=one.data_ptr(), shift=one.data_ptr(), N=N, H=H,   # noqa: E731
                                 W=W, Cin=C, Cout=C, R=3, S=3, stride=1, pad=1, relu=0)
    ws = torch.empty(d.backward_workspace(lay(1)), dtype=torch.uint8, device="cuda:0")
    back = lambda gx, with_gw: dl.BwdDesc(fwd=lay(1), gy=2, gpre=2, gx=gx, gx_add=dl.NO_TENSOR, wt=w.data_ptr(), gw=gw.data_ptr() if with_gw else None,    # noqa: E731
                                          workspace=ws.data_ptr(), workspace_bytes=ws.numel())
    whole = "conv3x3_halo bf16 256x64 (8x1 waves)"
    cut = whole + ", last tiles in 8 pieces"
    torch.cuda.synchronize()
    assert d.backward_kernel(back(3, True)).startswith("gx: %s; gw: " % whole) and "second stream" in d.backward_kernel(back(3, True))
    assert d.backward_kernel(back(4, False)) == "gx: " + cut and d.layer_kernel(lay(5)) == cut
    d.backward_segment([back(3, True)])
    assert d.backward_kernel(back(4, False)) == "gx: " + whole and d.layer_kernel(lay(5)) == whole
    d.recompute_segment([lay(5)])
    d.backward_join()
    assert d.backward_kernel(back(4, False)) == "gx: " + cut and d.layer_kernel(lay(5)) == cut
    d.backward_segment([back(4, False)])
    d.sync()
    beside = view(5).clone()
    assert torch.equal(view(3), view(4)) and view(3).any()
    torch.cuda.synchronize()
    d.recompute_segment([lay(5)])
    d.sync()
    assert torch.equal(view(5), beside)
    d.close()
