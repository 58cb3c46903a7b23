"""Dense bf16 layers on the direct-to-LDS kernels (igemm_dma_kernel, wgrad_dma_kernel) where their loads' addresses can go wrong: the masks of rows
and columns at the edges of odd images, for filters of 1 to 49 taps in both directions; backward-data of stride 2 by parity class and by
pixel; images of one and of two rows; reductions of fewer steps than the ring has stages; every tile width and both K steps under a filter; row,
column and pixel tails; the weight gradient's pixels over images of more and of less than a step of 32.  Every operation of the block against
the plain fp64 oracle primitives on the tensors that the library read, at the bounds of local_parity.py (a wrong tap or pixel is off by the
size of the result).  The profile classes say which kernels ran, on a chip of 256 compute units."""
import pytest
import torch

import local_parity
import parity
from paper_2301_12443_amd import workloads as W

pytestmark = pytest.mark.gpu

# (batch, h, w, channels of the layer's input, of its output, k, stride), tiles of the forward, backward-data and weight-gradient launch
# (None: too few for these kernels)
CASES = [
    ((20, 21, 20, 64, 512, 3, 1), "256x64x32", None, "256x256"),           # weight gradient: the last column tile a quarter full
    ((9, 33, 31, 96, 384, 3, 1), "256x64x32", None, "192x256"),
    ((30, 39, 41, 64, 64, 5, 1), "256x64x32", "256x64x32", None),          # 25 taps
    ((30, 39, 40, 64, 64, 6, 1), "256x64x32", "256x64x32", None),          # 36, an even filter
    ((30, 39, 40, 64, 64, 7, 1), "256x64x32", "256x64x32", None),          # 49
    ((30, 39, 41, 64, 256, 3, 1), "256x256x64", "256x64x32", "256x256"),
    ((30, 39, 41, 192, 64, 3, 1), "256x64x32", "256x192x64", None),
    ((30, 39, 41, 128, 128, 3, 1), "256x128x64", "256x128x64", None),
    ((30, 39, 41, 96, 96, 3, 1), "256x96x32", "256x96x32", None),
    ((12, 62, 64, 64, 256, 3, 2), "256x64x32", "256x64x32", "256x256"),    # parity classes
    ((12, 62, 64, 64, 64, 5, 2), None, "256x64x32", None),
    ((12, 62, 64, 64, 64, 7, 2), None, "256x64x32", None),
    ((12, 62, 64, 96, 192, 3, 2), None, "256x96x32", "192x256"),
    ((12, 62, 64, 64, 512, 1, 2), "256x64x32", "256x64x32", None),         # classes that no tap reaches
    ((12, 63, 61, 64, 256, 3, 2), "256x64x32", "256x64x32", "256x256"),    # an odd image: in pixel order
    ((12, 63, 61, 64, 64, 5, 2), None, "256x64x32", None),
    ((20, 21, 20, 64, 768, 1, 1), "256x64x32", None, None),                # two steps
    ((20, 21, 20, 128, 512, 1, 1), "256x64x32", None, None),               # four
    ((33, 65, 63, 64, 512, 1, 1), "256x256x64", "256x64x32", None),               # one
    ((2000, 5, 5, 64, 64, 3, 1), "256x64x32", "256x64x32", None),          # ten images a tile
    ((360, 5, 5, 64, 512, 3, 1), "256x64x32", None, "256x256"),            # more than an image a step of the weight gradient
    ((180, 7, 7, 64, 384, 3, 1), "256x64x32", None, "192x256"),
    # one row: two of three filter rows lie outside, and beyond the end of the tensor
    ((1, 1, 8200, 64, 512, 3, 1), "256x64x32", None, "256x256"),
    ((1, 1, 46000, 64, 64, 3, 1), "256x64x32", "256x64x32", None),
    ((1, 1, 46000, 64, 64, 3, 2), None, "256x64x32", None),
    ((1, 2, 23100, 64, 64, 5, 1), "256x64x32", "256x64x32", None),
    # 1 x 1 weight gradients on 192 x 256, 256 x 192 and 256 x 256 tiles, a ragged last step
    ((73, 61, 59, 256, 192, 1, 1), "256x192x64", "256x256x64", "192x256"),
    ((33, 65, 63, 192, 512, 1, 1), "256x256x64", "256x192x64", "256x192"),
    ((33, 65, 63, 256, 512, 1, 1), "256x256x64", "256x256x64", "256x256"),
]


def _layer(n, h, w, ci, co, k, s, twice=False):
    t, b = W.Block(), W.Block()
    t.cba(0, co, k, s, act=W.ACT_NONE)
    v = b.cba(0, ci, 1, act=W.ACT_RELU)
    u = b.cba(v, co, k, s, act=W.ACT_NONE)
    if twice:
        b.add(u, b.cba(v, co, k, s, act=W.ACT_NONE))
    return W.Workload("dense_ring", n, (ci, h, w), [t], [b], "bf16", lr=0.05)


def _check(wl):
    worst = local_parity.run_and_check(wl, wl.batch)
    print(", ".join(f"{key} {e:.1e}" for key, e in sorted(worst.items())), flush=True)


def _classes(wl, op=1):
    """The profile classes of the student layer's launches."""
    d = parity.make_distiller(wl, wl.batch, "bf16")
    d.teacher_relay(torch.from_numpy(W.make_input(wl)).cuda())
    d.set_profile(True)
    d.student_step(1, wl.lr)
    return [p["name"] for p in d.get_profile() if p["op"] == op]


@pytest.mark.parametrize("shape,fwd,dgrad,wgrad", CASES)
def test_addresses_of_the_direct_to_lds_kernels(shape, fwd, dgrad, wgrad):
    wl = _layer(*shape)
    names = _classes(wl)
    ran = [[n for n in names if n.startswith(kind) and n[len(kind):].startswith(tiles)]
           for kind, tiles in (("igemm_fwd_", "256x"), ("igemm_dgrad_", "256x"), ("wgrad_", ("192x", "256x")))]
    assert ran == [[f"igemm_fwd_{fwd}_store"] if fwd else [], [f"igemm_dgrad_{dgrad}_store"] if dgrad else [], [f"wgrad_{wgrad}"] if wgrad else []], names
    _check(wl)


@pytest.mark.parametrize("shape", [(30, 39, 41, 64, 64, 3, 1), (12, 62, 64, 64, 64, 5, 2)])
def test_backward_data_that_adds_to_a_gradient(shape):
    wl = _layer(*shape, twice=True)
    assert "igemm_dgrad_256x64x32_store" in _classes(wl, 2) and "igemm_dgrad_256x64x32_accum" in _classes(wl, 1)
    _check(wl)
