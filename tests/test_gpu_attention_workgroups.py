"""Attention with 2, 4 and 8 wavefronts to a workgroup, at the edges of a wavefront's 32 queries, of a block of 64 keys and of each workgroup's queries.

An image's result does not depend on how many queries share a workgroup: the images of a large batch carry the bits of that image alone.  The image alone is
held against float64: 2^-9 from the stored result, 2^-9 from the probabilities (a mean of v with relative errors of that size), below 1e-2 of the maximum."""
import numpy as np
import pytest

from oracle import transformer as ot
from test_gpu_transformer import _bits, _ctx, torch_mod  # noqa: F401

pytestmark = pytest.mark.gpu


def _run(torch, dl, qkv, heads, waves):
    N, S, H = qkv.shape[0], qkv.shape[1], heads * 64
    d, put, get = _ctx(torch, [qkv.nbytes, N * S * H * 2], 96)
    put(0, qkv)
    desc = dl.LayerDesc(x=0, res=dl.NO_TENSOR, y=1, dtype=dl.DTYPE_BF16, w=None, scale=None, shift=None,
                        N=N, H=S, W=1, Cin=3 * H, Cout=H, R=heads, S=1, stride=1, pad=0, relu=0, op=dl.OP_ATTENTION)
    assert "%d waves" % waves in d.layer_kernel(desc)
    d.recompute_segment([desc])
    d.sync()
    out = get(1, (N, S, H)).copy()
    d.close()
    return out


# S, then (images, wavefronts) of two batches with 2 heads; the last image is compared with float64
@pytest.mark.parametrize("S,one,many", [(1, (1, 2), (130, 4)), (31, (1, 2), (129, 4)), (33, (1, 2), (129, 4)), (64, (1, 2), (129, 4)), (65, (1, 2), (65, 4)),
                                        (127, (2, 2), (65, 4)), (128, (2, 2), (65, 4)), (129, (1, 2), (64, 4)), (129, (1, 2), (65, 8)), (192, (1, 2), (65, 8)),
                                        (193, (1, 2), (65, 8)), (256, (32, 2), (65, 8)), (257, (1, 2), (50, 8)), (257, (1, 2), (86, 4)), (384, (1, 2), (43, 8)),
                                        (385, (1, 4), (40, 8)), (513, (1, 4), (26, 8))])
def test_images_do_not_depend_on_the_workgroup(torch_mod, S, one, many):  # noqa: F811
    torch = torch_mod
    import paper_2203_15980_amd as dl
    heads = 2
    qkv = _bits(66, S, (many[0], S, 3 * heads * 64))
    a = _run(torch, dl, qkv[:one[0]], heads, one[1])
    b = _run(torch, dl, qkv, heads, many[1])
    assert np.array_equal(a, b[:one[0]])
    ref = ot.attention_f64(qkv[-1:], heads, "bf16")
    err = float(np.max(np.abs(ot.to_f64(b[-1:], "bf16") - ref)) / np.max(np.abs(ref)))
    print(S, one, many, "%.2e" % err, flush=True)
    assert err <= 1e-2
