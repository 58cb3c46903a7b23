"""float32 dense convolutions whose operands loader waves bring (conv_f32_kernels.h), where the loaders' short cuts begin and end: stages
inside one tap (channels in multiples of 64 on 16-wide tiles, of 32 on 32-wide ones) at stride 1 and 2, weight gradients over images of
whole rows a stage, of whole images a stage and of neither, and as many stages as the ring has slots, one more and one less.  Bit for bit
against the direct kernels (force_direct), whose order of summation they keep: a wrong index, mask or stage changes the result."""
import numpy as np
import pytest

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
