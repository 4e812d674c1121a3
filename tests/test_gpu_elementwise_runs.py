"""Batch normalisation, add and ReLU that follow each other in a segment run as one pass, ReLU's and batch normalisation's backward as one
launch less: the bits are those of the operators one by one (a segment each), for every run there is, ragged sizes included, and where
something in the run is used twice the operators go one by one."""
import numpy as np
import pytest

import synth
from test_gpu_backward import _bits, _dev, _small_ctx, torch_mod  # noqa: F401

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1, 1, 8), (1, 3, 5, 24), (2, 7, 9, 64), (1, 13, 11, 2056), (4, 28, 28, 512), (3, 57, 31, 256)]      # pieces of 16 bytes: odd counts, one, 1.3 M


def _ops(torch, dl, shape):
    """Tensors 0 x, 1 res, 2 bn, 3 add, 4 relu, 5 gy, 6 g, 7 gx; the layers and what they keep alive."""
    N, H, W, C = shape
    d, put, get = _small_ctx(torch, [N * H * W * C * 2] * 8, mb=256)
    data = {t: _bits(71, t, shape) for t in (0, 1, 5)}
    data[1].reshape(-1)[:min(7, data[1].size)] = np.array([0x8000, 0x7FC0, 0xFFC1, 0x7F80, 0xFF80, 0x0001, 0x8001], np.uint16)[:data[1].size]
    gamma, beta = _dev(torch, synth.normal(71, 11, C).astype(np.float32)), _dev(torch, synth.normal(71, 12, C).astype(np.float32))
    same = dict(dtype=dl.DTYPE_BF16, N=N, H=H, W=W, Cin=C, Cout=C, R=1, S=1, stride=1, pad=0, relu=0)
    bn = lambda x=0, y=2: dl.LayerDesc(x=x, res=dl.NO_TENSOR, y=y, scale=gamma.data_ptr(), shift=beta.data_ptr(), op=dl.OP_BATCHNORM,      # noqa: E731
                                       eps=1e-5, **same)
    add = lambda x=2, res=1, y=3: dl.LayerDesc(x=x, res=res, y=y, op=dl.OP_ADD, **same)                                                    # noqa: E731
    relu = lambda x=3, y=4: dl.LayerDesc(x=x, res=dl.NO_TENSOR, y=y, op=dl.OP_RELU, **same)                                               # noqa: E731
    return d, put, get, data, bn, add, relu, (gamma, beta)


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_runs_carry_the_bits_of_single_operators(torch_mod, shape):  # noqa: F811
    torch = torch_mod
    import paper_2203_15980_amd as dl
    d, put, get, data, bn, add, relu, keep = _ops(torch, dl, shape)
    runs = [[bn(), add(), relu()], [bn(), add()], [bn(), relu(x=2)], [add(x=0), relu()], [bn(), add(), relu(), bn(x=4, y=6)],
            [bn(), relu(x=2), add(x=4), relu(x=3, y=6)],
            # not one pass: the add reads the normalisation twice, takes it as its second operand, writes over the input; the ReLU over the residual
            [bn(), add(res=2), relu()], [bn(), add(x=1, res=2), relu()], [bn(), add(y=0), relu(x=0)], [bn(), add(), relu(y=1)]]
    for k, run in enumerate(runs):
        print("shape", shape, "run", k, flush=True)
        outs = sorted({l.y for l in run})
        got = []
        for together in (False, True):
            d.bind([data[0].nbytes] * 8)                         # nothing is resident
            put(0, data[0])
            put(1, data[1])
            for part in ([run] if together else [[l] for l in run]):
                d.recompute_segment(part)
            d.sync()
            got.append([get(t, shape).copy() for t in outs])
        assert all(np.array_equal(a, b) for a, b in zip(*got)), k
    d.close()


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_masked_gradient_and_normalisation_backward(torch_mod, shape):  # noqa: F811
    torch = torch_mod
    import paper_2203_15980_amd as dl
    d, put, get, data, bn, add, relu, keep = _ops(torch, dl, shape)
    put(0, data[0])
    put(4, data[1])                                              # the stored ReLU output: signs, zeros, NaN, infinities
    put(5, data[5])
    C = shape[-1]
    got = []
    for together in (False, True):
        gw = torch.full((2 * C,), float("nan"), device="cuda:0")
        b = lambda fwd, gy, gx, g=None: dl.BwdDesc(fwd=fwd, gy=gy, gpre=gy, gx=gx, gx_add=dl.NO_TENSOR, gw=g)      # noqa: E731
        descs = [b(relu(), 5, 6), b(bn(), 6, 7, gw.data_ptr())]
        if not together:
            d.alloc(2), d.alloc(3)                               # the forward outputs that the layers name
        before = d.stats()["recompute_launches"]
        for part in ([descs] if together else [[x] for x in descs]):
            d.backward_segment(part)
        d.sync()
        assert d.stats()["recompute_launches"] - before == 2
        got.append([get(6, shape).copy(), get(7, shape).copy(), gw.cpu().numpy().view(np.uint32)])
        for t in (6, 7):
            d.release(t, dl.EV_FREE)
    assert all(np.array_equal(a, b) for a, b in zip(*got))
    d.close()


def test_a_run_without_room_goes_as_far_as_it_can(torch_mod):  # noqa: F811
    """The arena holds the inputs and one output: the normalisation is there and whole, the status says that the add has no room."""
    torch = torch_mod
    import paper_2203_15980_amd as dl
    N, H, W, C = 1, 16, 16, 512
    n = N * H * W * C * 2
    d = dl.Delta(torch.empty(3 * n + n // 2, dtype=torch.uint8, device="cuda:0"), torch.cuda.current_stream().cuda_stream)
    d.bind([n] * 5)
    x, res = _bits(71, 0, (N, H, W, C)), _bits(71, 1, (N, H, W, C))
    at = lambda t: d.arena[d.tensor_ptr(t) - d.arena.data_ptr():][:n]            # noqa: E731
    for t, a in ((0, x), (1, res)):
        d.alloc(t)
        at(t).copy_(_dev(torch, a.view(np.uint8).reshape(-1)))
    one = torch.ones(C, device="cuda:0")
    same = dict(dtype=dl.DTYPE_BF16, N=N, H=H, W=W, Cin=C, Cout=C, R=1, S=1, stride=1, pad=0, relu=0)
    bn = dl.LayerDesc(x=0, res=dl.NO_TENSOR, y=2, scale=one.data_ptr(), shift=one.data_ptr(), op=dl.OP_BATCHNORM, eps=1e-5, **same)
    add = dl.LayerDesc(x=2, res=1, y=3, op=dl.OP_ADD, **same)
    with pytest.raises(dl.DeltaError):
        d.recompute_segment([bn, add])
    d.sync()
    first = at(2).cpu().numpy().copy()
    d.release(2, dl.EV_FREE)
    d.recompute_segment([bn])
    d.sync()
    assert np.array_equal(first, at(2).cpu().numpy())
    d.close()


def test_a_masked_gradient_without_room_behind_it_is_stored_and_counted(torch_mod):  # noqa: F811
    """The arena holds the ReLU's gradient and not the normalisation's: as one by one, the first is made and counted, the status says that
    the second has no room."""
    torch = torch_mod
    import paper_2203_15980_amd as dl
    N, H, W, C = 1, 16, 16, 512
    n = N * H * W * C * 2
    one = torch.ones(C, device="cuda:0")
    same = dict(dtype=dl.DTYPE_BF16, N=N, H=H, W=W, Cin=C, Cout=C, R=1, S=1, stride=1, pad=0, relu=0)
    bn = dl.LayerDesc(x=0, res=dl.NO_TENSOR, y=1, scale=one.data_ptr(), shift=one.data_ptr(), op=dl.OP_BATCHNORM, eps=1e-5, **same)
    relu = dl.LayerDesc(x=1, res=dl.NO_TENSOR, y=2, op=dl.OP_RELU, **same)
    descs = [dl.BwdDesc(fwd=relu, gy=3, gpre=3, gx=4, gx_add=dl.NO_TENSOR), dl.BwdDesc(fwd=bn, gy=4, gpre=4, gx=5, gx_add=dl.NO_TENSOR)]
    got = []
    for together in (False, True):
        d = dl.Delta(torch.empty(4 * n + n // 2, dtype=torch.uint8, device="cuda:0"), torch.cuda.current_stream().cuda_stream)
        d.bind([n] * 6)
        at = lambda t: d.arena[d.tensor_ptr(t) - d.arena.data_ptr():][:n]        # noqa: E731
        for t in (0, 2, 3):
            d.alloc(t)
            at(t).copy_(_dev(torch, _bits(71, t, (N, H, W, C)).view(np.uint8).reshape(-1)))
        with pytest.raises(dl.DeltaError) as e:
            for part in ([descs] if together else [[x] for x in descs]):
                d.backward_segment(part)
        d.sync()
        got.append((e.value.status, d.stats()["recompute_launches"], at(4).cpu().numpy().copy()))
        d.close()
    assert got[0][0] == got[1][0] == dl.ERR_OOM_ARENA and got[0][1] == got[1][1] == 1
    assert np.array_equal(got[0][2], got[1][2])


def test_statistics_do_not_wait_for_the_residual(torch_mod):  # noqa: F811
    """Normalisation and add in one pass while the residual is still being reloaded: the statistics need x alone and run beside the copy, only
    the pass over the elements waits for it.  128 MB over the host link take milliseconds, the statistics a fraction of one."""
    torch = torch_mod
    import paper_2203_15980_amd as dl
    N, H, W, C = 32, 64, 64, 512
    n = N * H * W * C * 2
    d = dl.Delta(torch.empty(5 * n, dtype=torch.uint8, device="cuda:0"), torch.cuda.current_stream().cuda_stream)
    d.bind([n] * 4)
    one = torch.ones(C, device="cuda:0")
    same = dict(dtype=dl.DTYPE_BF16, N=N, H=H, W=W, Cin=C, Cout=C, R=1, S=1, stride=1, pad=0, relu=0)
    bn = dl.LayerDesc(x=0, res=dl.NO_TENSOR, y=2, scale=one.data_ptr(), shift=one.data_ptr(), op=dl.OP_BATCHNORM, eps=1e-5, **same)
    add = dl.LayerDesc(x=2, res=1, y=3, op=dl.OP_ADD, **same)
    for t in (0, 1):
        d.alloc(t)
        d.arena[d.tensor_ptr(t) - d.arena.data_ptr():][:n].view(torch.bfloat16).normal_()
    for t in (2, 3):
        d.alloc(t)
    d.recompute_segment([bn, add])                               # whatever is allocated on first use
    d.sync()
    d.release(1, dl.EV_OFFLOAD)
    d.sync()
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CPU, torch.profiler.ProfilerActivity.CUDA]) as prof:
        d.prefetch(1)
        d.recompute_segment([bn, add])
        d.sync()
        torch.cuda.synchronize()
    spans = {}
    for e in prof.events():
        for key in ("HtoD", "bn_stats_kernel", "bn_finalize_kernel", "bn_tail_kernel"):
            if key in e.name and e.device_type == torch.autograd.DeviceType.CUDA:
                spans[key] = (e.time_range.start, e.time_range.end)
    print(spans, flush=True)
    if len(spans) < 4:
        pytest.skip("the profiler saw no kernels here: %s" % sorted({e.name for e in prof.events()})[:20])
    assert spans["bn_finalize_kernel"][1] < spans["HtoD"][1] <= spans["bn_tail_kernel"][0]
    d.close()
