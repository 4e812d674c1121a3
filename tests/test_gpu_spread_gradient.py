"""The data gradient of a strided 1x1 layer stored straight to its pixels of gx, zeros between: the bits of the same layer at stride 1, spread
out on the host.  Odd sizes, strides 2 and 3, every tile of the kernels that store so, its ragged edges, and the routes that still take two launches."""
import numpy as np
import pytest

import synth
from test_gpu_backward import _bits, _dev, _small_ctx, torch_mod  # noqa: F401

pytestmark = pytest.mark.gpu

CASES = [
    # N   H   W  Cin  Cout s  both  kernel
    (1, 1, 1, 256, 512, 2, 0, "conv_splitk bf16 32x32"),
    (3, 13, 17, 512, 1024, 2, 0, "conv_splitk bf16 32x32"),
    (2, 14, 15, 256, 512, 3, 0, "conv_splitk bf16 32x32"),     # blocks of 3 x 3, cut short below and at the right
    (3, 13, 17, 512, 1024, 2, 1, "small_backward bf16"),
    (1, 28, 28, 256, 512, 2, 1, "small_backward bf16"),
    (11, 55, 56, 256, 512, 2, 0, "gemm_nt bf16 128x128, four", "+ spread_add"),   # half a chip of tiles: two launches
    (6, 55, 56, 256, 512, 2, 0, "gemm_nt bf16 128x128 ("),
    (46, 27, 28, 512, 1024, 2, 0, "gemm_nt bf16 128x128 ("),
    (47, 56, 55, 256, 512, 2, 0, "gemm_nt bf16 128x256"),      # 47 x 28 x 28 rows: the last tile ragged
    (21, 56, 56, 512, 256, 2, 0, "gemm_nt bf16 256x"),
    (31, 27, 29, 1536, 512, 2, 0, "gemm_nt bf16 256x"),
    (41, 29, 29, 832, 512, 2, 0, "gemm_nt bf16 256x"),         # channels that end inside a tile
    (20, 13, 13, 512, 1024, 3, 0, "conv_splitk bf16 32x32"),
    (2, 13, 12, 64, 128, 2, 0, "conv_splitk f32 32x32"),
    (2, 16, 15, 64, 64, 2, 0, "conv1x1_stream", "+ spread_add"),    # a kernel without the form
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "%dx%dx%d_%d_%d_s%d_b%d" % c[:7])
def test_spread_gradient_carries_the_bits_of_the_layer_at_stride_1(torch_mod, case):  # noqa: F811
    torch = torch_mod
    import paper_2203_15980_amd as dl
    N, H, W, Cin, Cout, s, both, name = case[:8]
    print("case", case, flush=True)
    P, Q = (H - 1) // s + 1, (W - 1) // s + 1
    f32 = "f32" in name
    bits = (lambda m, i, shape, k=1.0: (synth.normal(m, i, int(np.prod(shape))) * k).astype(np.float32).reshape(shape)) if f32 else _bits
    t = np.float32 if f32 else np.uint16
    x, gy = bits(131, 1, (N, H, W, Cin)) if both else np.zeros((N, H, W, Cin), t), bits(131, 2, (N, P, Q, Cout))
    wtd = _dev(torch, bits(131, 4, (Cin, Cout), 0.1).view(np.uint8).reshape(-1))
    small = N * P * Q * Cin * x.itemsize
    d, put, get = _small_ctx(torch, [x.nbytes, gy.nbytes, gy.nbytes, x.nbytes, small, small],
                             mb=2 + (2 * x.nbytes + 2 * gy.nbytes + 2 * small >> 20))
    put(0, x)
    put(2, gy)
    put(3, np.full_like(x, 12345))                              # what no pixel may keep
    w, one = torch.zeros(Cout * Cin, dtype=torch.float32 if f32 else torch.bfloat16, device="cuda:0"), torch.ones(Cout, device="cuda:0")
    gw = torch.zeros(Cout, Cin, device="cuda:0")

    def desc(xid, gx, h, v, stride, gw_ptr):
        fwd = dl.LayerDesc(x=xid, res=dl.NO_TENSOR, y=1, dtype=dl.DTYPE_F32 if f32 else dl.DTYPE_BF16, w=w.data_ptr(), scale=one.data_ptr(), shift=one.data_ptr(), N=N, H=h,
                           W=v, Cin=Cin, Cout=Cout, R=1, S=1, stride=stride, pad=0, relu=0)
        work = torch.empty(max(256, d.backward_workspace(fwd)), dtype=torch.uint8, device="cuda:0")
        return work, dl.BwdDesc(fwd=fwd, gy=2, gpre=2, gx=gx, gx_add=dl.NO_TENSOR, mask_gx=0, wt=wtd.data_ptr(), gw=gw_ptr,
                                workspace=work.data_ptr(), workspace_bytes=work.numel())

    keep1, strided = desc(0, 3, H, W, s, gw.data_ptr() if both else None)
    keep2, plain = desc(4, 5, P, Q, 1, None)
    kernel = d.backward_kernel(strided)
    assert name in kernel and (case[8] if len(case) > 8 else ", spread") in kernel, kernel
    d.backward_segment([strided, plain])
    d.backward_join()
    d.sync()
    got, want = get(3, x.shape, t), np.zeros_like(x)
    want[:, ::s, ::s] = get(5, (N, P, Q, Cin), t)
    d.close()
    assert np.array_equal(got, want)
    assert want.any()


@pytest.mark.parametrize("case", [(61, 57, 58, 128, 0, 1), (25, 8001, 1, 128, 0, 1), (98305, 1, 2, 128, 0, 1), (61, 57, 58, 64, 0, 1), (3, 257, 257, 64, 0, 1),
                                  (62, 57, 57, 128, 1, 0), (60, 56, 55, 128, 0, 0), (60, 56, 55, 64, 0, 0)], ids=lambda c: "%dx%dx%d_%d_%d_%d" % c)
def test_a_gradient_with_known_zeros_is_added_as_if_all_of_it_were_read(torch_mod, case):  # noqa: F811
    """The strided layer's gx added by the layer that runs next (256 -> 128 or 64 channels, both gradients in one pass): in one call, where its zeros are
    known (the last flag, by the kernel that ran), the bits of one call per layer.  The flag before: a third layer overwrites the tensor in between.
    (60 x 56 x 55 lies below the line.)"""
    torch = torch_mod
    import paper_2203_15980_amd as dl
    N, H, W, C, between, known = case
    print("case", case, flush=True)
    P, Q, rng = (H - 1) // 2 + 1, (W - 1) // 2 + 1, np.random.default_rng(7)
    bits = lambda *shape: ((rng.integers(0, 1 << 16, shape, np.uint16) & 0x80FF) | 0x3F00).astype(np.uint16)     # noqa: E731  # +-[0.5, 2)
    x, g512, gc = bits(N, H, W, 256), bits(N, P, Q, 512), bits(N, H, W, C)
    dev = lambda *shape: _dev(torch, bits(*shape).view(np.uint8).reshape(-1))                                    # noqa: E731
    d, put, get = _small_ctx(torch, [x.nbytes, g512.nbytes, gc.nbytes, x.nbytes, x.nbytes, g512.nbytes, gc.nbytes],
                             mb=4 + (3 * x.nbytes + 2 * g512.nbytes + 2 * gc.nbytes >> 20))
    put(0, x), put(1, g512), put(2, gc)
    put(3, np.full_like(x, 12345))
    one, keep = torch.ones(512, device="cuda:0"), []

    def desc(gy, y, gx, add, cout, stride, gw):
        w, wt, out = torch.zeros(cout * 256, dtype=torch.bfloat16, device="cuda:0"), dev(256, cout), torch.zeros(cout, 256, device="cuda:0")
        fwd = dl.LayerDesc(x=0, res=dl.NO_TENSOR, y=y, dtype=dl.DTYPE_BF16, w=w.data_ptr(), scale=one.data_ptr(), shift=one.data_ptr(), N=N, H=H, W=W,
                           Cin=256, Cout=cout, R=1, S=1, stride=stride, pad=0, relu=0)
        work = torch.empty(max(256, d.backward_workspace(fwd)), dtype=torch.uint8, device="cuda:0")
        keep.extend([w, wt, out, work])
        return dl.BwdDesc(fwd=fwd, gy=gy, gpre=gy, gx=gx, gx_add=add, mask_gx=int(add != dl.NO_TENSOR), wt=wt.data_ptr(), gw=out.data_ptr() if gw else None,
                          workspace=work.data_ptr(), workspace_bytes=work.numel())

    chain = [desc(1, 5, 3, dl.NO_TENSOR, 512, 2, False)]
    if between:
        chain.append(desc(2, 6, 3, dl.NO_TENSOR, C, 1, False))
    chain.append(desc(2, 6, 4, 3, C, 1, True))
    assert ", spread" in d.backward_kernel(chain[0]) and "joint1x1" in d.backward_kernel(chain[-1]), [d.backward_kernel(k) for k in chain]
    outs, even = [], []
    for calls in ([chain], [[k] for k in chain]):
        with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as prof:
            for call in calls:
                d.backward_segment(call)
            d.backward_join()
            d.sync()
        ran = [e.name for e in prof.events() if "joint1x1_kernel" in e.name]
        even += [n.split("<")[1].split(">")[0].split(", ")[2] for n in ran]       # 0: nothing added, 1: a tensor, 2: one with known zeros
        outs.append((get(4, x.shape, np.uint16).copy(), keep[-2].cpu().numpy().copy()))
        d.release(4, dl.EV_FREE)
        put(4, np.zeros_like(x))
    d.close()
    assert np.array_equal(outs[0][0], outs[1][0]) and np.array_equal(outs[0][1], outs[1][1])
    assert outs[0][0].any()
    if not even:
        pytest.skip("the profiler saw no kernels here")
    assert even == ["2" if known else "1", "1"], even
