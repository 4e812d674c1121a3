"""The loss over several workgroups: image counts around its lines (32 images, the scratch's 16384) and its workgroups of four, launches
that follow each other without a synchronisation, two contexts in turn.  Sums of N fp32 losses in 1024 chains and a tree: N / 1024 + 10
roundings of 2^-24, at 16384 images 1.6e-6 in the worst order; 1e-5 as for the other forms."""
import numpy as np
import pytest

import synth
from oracle import numeric as on
from test_gpu_backward import _small_ctx, torch_mod  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,classes", [(32, 1000), (33, 1000), (35, 8), (64, 512), (129, 520), (257, 1024), (16384, 16), (16385, 16)])
def test_loss_over_workgroups(torch_mod, N, classes):  # noqa: F811
    import paper_2203_15980_amd as dl
    rows = [synth.f32_to_bf16_bits(synth.normal(12, k, N * classes).astype(np.float32) * 3).reshape(N, classes) for k in (1, 2)]
    labels = [synth.make_labels(12 + k, N, classes) for k in (0, 1)]
    loss = dl.LayerDesc(x=0, res=1, y=2, dtype=dl.DTYPE_BF16, N=N, H=1, W=1, Cin=classes, Cout=1, R=1, S=1, stride=1, pad=0, relu=0,
                        op=dl.OP_SOFTMAX_CE)
    ctx = []
    for z, lab in zip(rows, labels):
        d, put, get = _small_ctx(torch_mod, [z.nbytes, N * 8, 4])
        put(0, z)
        put(1, lab)
        ctx.append((d, get))
    for k in range(6):                                           # every launch leaves the counter as it found it
        ctx[k % 2][0].recompute_segment([loss] * (1 + k))
    for (d, get), z, lab in zip(ctx, rows, labels):
        d.sync()
        zf = on.to_f64(z, "bf16")
        top = zf.max(1)
        ref = float(np.mean(top + np.log(np.exp(zf - top[:, None]).sum(1)) - zf[np.arange(N), lab]))
        first = get(2, (1,), np.float32).copy()
        print("N %d classes %d: %.8g %.8g" % (N, classes, first[0], ref), flush=True)
        assert abs(float(first[0]) - ref) <= 1e-5 * max(abs(ref), 1.0)
        d.recompute_segment([loss])
        d.sync()
        assert np.array_equal(first, get(2, (1,), np.float32))
        d.close()


def test_more_contexts_than_slots(torch_mod):  # noqa: F811
    """Contexts beyond those that find a slot for their losses take one workgroup; a slot given back is taken again."""
    import paper_2203_15980_amd as dl
    N, classes = 64, 1000
    z, lab = synth.f32_to_bf16_bits(synth.normal(12, 1, N * classes).astype(np.float32) * 3).reshape(N, classes), synth.make_labels(12, N, classes)
    loss = dl.LayerDesc(x=0, res=1, y=2, dtype=dl.DTYPE_BF16, N=N, H=1, W=1, Cin=classes, Cout=1, R=1, S=1, stride=1, pad=0, relu=0,
                        op=dl.OP_SOFTMAX_CE)
    got = []
    for count in (67, 3):
        ctx = [_small_ctx(torch_mod, [z.nbytes, N * 8, 4], mb=1) for _ in range(count)]
        for d, put, get in ctx:
            put(0, z)
            put(1, lab)
            d.recompute_segment([loss])
        for d, put, get in ctx:
            d.sync()
            got.append(float(get(2, (1,), np.float32)[0]))
            d.close()
    assert max(got) - min(got) <= 1e-5 * max(got) and got[0] == got[67]


def test_captured_losses_keep_off_the_contexts_scratch(torch_mod):  # noqa: F811
    """A graph that holds a loss is replayed on one stream while its context computes losses on another, and again after that context is
    closed and another one has its place: every result is the one computed alone."""
    torch = torch_mod
    import paper_2203_15980_amd as dl
    N, classes = 129, 1000
    z, lab = synth.f32_to_bf16_bits(synth.normal(13, 1, N * classes).astype(np.float32) * 3).reshape(N, classes), synth.make_labels(13, N, classes)
    zf = on.to_f64(z, "bf16")
    top = zf.max(1)
    ref = float(np.mean(top + np.log(np.exp(zf - top[:, None]).sum(1)) - zf[np.arange(N), lab]))
    near = lambda v: abs(v - ref) <= 1e-5 * max(abs(ref), 1.0)                   # noqa: E731
    loss = lambda y: dl.LayerDesc(x=0, res=1, y=y, dtype=dl.DTYPE_BF16, N=N, H=1, W=1, Cin=classes, Cout=1, R=1, S=1, stride=1, pad=0,      # noqa: E731
                                  relu=0, op=dl.OP_SOFTMAX_CE)
    main, side, keep = torch.cuda.Stream(), torch.cuda.Stream(), []

    def context():
        arena = torch.empty(1 << 20, dtype=torch.uint8, device="cuda:0")
        keep.append(arena)                                       # the graph's tensors outlive the context
        d = dl.Delta(arena, main.cuda_stream)
        d.bind([z.nbytes, N * 8, 4, 4])
        view = [arena[d.alloc(t) - arena.data_ptr():][:n] for t, n in enumerate((z.nbytes, N * 8, 4, 4))]
        view[0].copy_(torch.from_numpy(z.view(np.uint8).reshape(-1)))
        view[1].copy_(torch.from_numpy(lab.view(np.uint8).reshape(-1)))
        torch.cuda.synchronize()
        return d, view[2].view(torch.float32), view[3].view(torch.float32)
    d, eager, held = context()
    d.recompute_segment([loss(2)])
    torch.cuda.synchronize()
    alone = float(eager[0])
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=main):
        d.recompute_segment([loss(3)])
    graph.replay()
    torch.cuda.synchronize()
    replayed = float(held[0])
    assert near(alone) and near(replayed)
    for second in (False, True):
        if second:
            d.close()
            d, eager, _ = context()
        for _ in range(5):
            held.fill_(float("nan"))
            eager.fill_(float("nan"))
            torch.cuda.synchronize()
            with torch.cuda.stream(side):
                for _ in range(4):
                    graph.replay()
            d.recompute_segment([loss(2)] * 16)
            torch.cuda.synchronize()
            assert float(eager[0]) == alone and float(held[0]) == replayed
    d.close()
