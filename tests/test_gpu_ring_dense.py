"""Dense bf16 layers on the direct-to-LDS kernels (igemm_dma_kernel, wgrad_dma_kernel) where their loads' addresses can go wrong: the tap mask
at the edges of odd images, at 25 taps, and beyond its 32 bits (49 taps: the 128-row kernel takes the layer); backward-data of stride 2 by
parity class and by pixel; reductions of fewer steps than the ring has stages; row, column and pixel tails; the weight gradient's pixels over
images of more and of less than a step of 32.  Every operation of the block against the plain fp64 oracle primitives on the tensors that the
library read, at the bounds of local_parity.py (a wrong tap or pixel is off by the size of the result)."""
import pytest
import torch

import local_parity
import parity
from paper_2301_12443_amd import workloads as W

pytestmark = pytest.mark.gpu

# (batch, h, w, channels of the layer's input, of its output, k, stride)
CASES = [
    (20, 21, 20, 64, 512, 3, 1),         # 8400 rows; weight gradient on 256 x 256 tiles, the last column tile a quarter full
    (9, 33, 31, 96, 384, 3, 1),          # K step 32; 192 x 256 tiles
    (6, 37, 39, 64, 256, 5, 1),          # 25 taps
    (6, 37, 39, 32, 256, 7, 1),          # 49 taps
    (20, 40, 42, 64, 256, 3, 2),         # parity classes
    (20, 41, 43, 64, 256, 3, 2),         # an odd image: in pixel order
    (20, 40, 42, 64, 512, 1, 2),         # classes that no tap reaches
    (20, 21, 20, 64, 768, 1, 1),         # one step
    (20, 21, 20, 128, 512, 1, 1),        # two
    (360, 5, 5, 64, 512, 3, 1),          # more than an image a step of the weight gradient
    (180, 7, 7, 64, 384, 3, 1),
    (1, 1, 8200, 64, 512, 3, 1),         # one row: two of three filter rows lie outside, and beyond the end of the tensor
    (1, 2, 4200, 64, 256, 5, 1),
    # 1 x 1 weight gradients on 192 x 256, 256 x 192 and 256 x 256 tiles, a ragged last step
    (73, 61, 59, 256, 192, 1, 1),
    (33, 65, 63, 192, 512, 1, 1),
    (33, 65, 63, 256, 512, 1, 1),
]


def _layer(n, h, w, ci, co, k, s):
    t, b = W.Block(), W.Block()
    t.cba(0, co, k, s, act=W.ACT_NONE)
    v = b.cba(0, ci, 1, act=W.ACT_RELU)
    b.cba(v, co, k, s, act=W.ACT_NONE)
    return W.Workload("dense_ring", n, (ci, h, w), [t], [b], "bf16", lr=0.05)


def _check(wl):
    worst = local_parity.run_and_check(wl, wl.batch)
    print(", ".join(f"{key} {e:.1e}" for key, e in sorted(worst.items())), flush=True)


def _classes(wl):
    """The profile classes of the layer's launches, student and teacher."""
    d = parity.make_distiller(wl, wl.batch, "bf16")
    x = torch.from_numpy(W.make_input(wl)).cuda()
    d.set_profile(True)
    d.teacher_relay(x)
    d.student_step(1, wl.lr)
    return [p["name"] for p in d.get_profile() if (p["net"], p["op"]) in ((1, 1), (0, 0))]


@pytest.mark.parametrize("n,h,w,ci,co,k,s", CASES)
def test_addresses_of_the_direct_to_lds_kernels(n, h, w, ci, co, k, s):
    _check(_layer(n, h, w, ci, co, k, s))


@pytest.mark.parametrize("k", [6, 7])
def test_filters_of_more_taps_than_a_word_has_bits(k):
    wl = _layer(30, 39, 40, 64, 64, k, 1)
    assert {"igemm_fwd_256x64x32_store", "igemm_fwd_256x64x32_affine", "igemm_dgrad_256x64x32_store"} <= set(_classes(wl))
    _check(wl)
