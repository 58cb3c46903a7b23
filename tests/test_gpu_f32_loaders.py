"""float32 dense convolutions whose operands loader waves bring (conv_f32_kernels.h), where the loaders' short cuts begin and end: stages
inside one tap (channels in multiples of 64 on 16-wide tiles, of 32 on 32-wide ones) at stride 1 and 2, weight gradients over images of
whole rows a stage, of whole images a stage and of neither, and as many stages as the ring has slots, one more and one less.  Bit for bit
against the direct kernels (force_direct), whose order of summation they keep: a wrong index, mask or stage changes the result.  The profile
classes say which tile and ring ran, on a chip of 256 compute units (igemm_f32_fwd_32r3: 32 x 32 results, a ring of three stages)."""
import numpy as np
import pytest
import torch

import parity
from paper_2301_12443_amd import workloads as W
from test_gpu_conv_f32 import _everything, _workload

pytestmark = pytest.mark.gpu

# (batch, h, w, channels of the block's input, of the layer's input, of its output, k, stride)
SHAPES = [
    (9, 16, 16, 16, 64, 128, 3, 2),      # a stage inside one tap, stride 2 both ways, whole rows of dy a stage
    (3, 7, 9, 16, 128, 64, 3, 1),        # ... on odd images
    (16, 32, 32, 16, 64, 72, 3, 1),      # 32-wide tiles, a stage inside one tap
    (16, 33, 32, 16, 96, 64, 3, 1),      # ... 33 rows of 32 pixels: no whole stages an image
    (24, 4, 4, 16, 128, 136, 3, 1),      # four images a stage of the weight gradient
    (70, 2, 2, 16, 64, 72, 3, 1),        # sixteen
    (5, 1, 1, 64, 320, 64, 1, 1),        # five, six and seven stages, one pixel an image
    (5, 1, 1, 64, 384, 64, 1, 1),
    (5, 1, 1, 64, 448, 64, 1, 1),
    (6, 3, 4, 16, 24, 48, 3, 1),         # rows of 4 pixels, 3 rows an image
    (3, 8, 64, 8, 16, 24, 5, 1),         # one row of 64 pixels a stage
    (2, 128, 128, 8, 8, 16, 3, 1),       # half a row
]


@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_same_bits_as_the_direct_kernels(shape):
    wl = _workload(*shape)
    ref, got = _everything(wl, True, 2), _everything(wl, False, 2)
    for name in ref:
        np.testing.assert_array_equal(got[name], ref[name], err_msg=name)


# ... and the launches of the layer
MANY = [
    # 16-wide tiles with more than one workgroup a unit: a ring of three stages, reductions of 1, 3, 14 and 18 stages
    ((16, 14, 14, 16, 64, 256, 1, 1), ("igemm_f32_fwd_32r3", "igemm_f32_dgrad_32r6", "wgrad_f32_32r6")),
    ((9, 14, 14, 16, 192, 256, 1, 1), ("igemm_f32_fwd_32r3", "igemm_f32_dgrad_32r3", "wgrad_f32_32r6")),
    ((7, 13, 13, 16, 128, 320, 3, 1), ("igemm_f32_fwd_32r3", "igemm_f32_dgrad_32r6", "wgrad_f32_32r3")),
    ((8, 14, 14, 16, 256, 96, 3, 1), ("igemm_f32_fwd_32r6", "igemm_f32_dgrad_32r3", "wgrad_f32_32r6")),
    ((8, 14, 14, 16, 256, 128, 3, 2), ("igemm_f32_fwd_32r6", "igemm_f32_dgrad_32r3", "wgrad_f32_32r3")),
    # weight gradients of one, two, three and five stages
    ((1, 7, 7, 16, 768, 768, 1, 1), ("wgrad_f32_32r3",)),
    ((5, 5, 5, 16, 384, 768, 1, 1), ("wgrad_f32_32r3",)),
    ((3, 8, 8, 16, 64, 512, 3, 1), ("wgrad_f32_32r3",)),
    ((9, 5, 6, 16, 64, 520, 3, 1), ("wgrad_f32_32r3",)),
    # 32-wide tiles
    ((16, 33, 32, 16, 96, 64, 3, 1), ("igemm_f32_fwd_64r3", "igemm_f32_dgrad_64r3", "wgrad_f32_32r6")),
]


@pytest.mark.parametrize("shape,classes", MANY, ids=str)
def test_same_bits_on_either_ring(shape, classes):
    wl = _workload(*shape)
    d = parity.make_distiller(wl)
    d.teacher_relay(torch.from_numpy(W.make_input(wl)).cuda())
    d.set_profile(True)
    d.student_step(1, wl.lr)
    # (a weight gradient goes out with others of its kernel, under the name of the first)
    names = {p["name"] for p in d.get_profile() if p["op"] == 1 or p["name"].startswith("wgrad")}
    assert names >= set(classes), names
    ref, got = _everything(wl, True, 2), _everything(wl, False, 2)
    for name in ref:
        np.testing.assert_array_equal(got[name], ref[name], err_msg=name)
