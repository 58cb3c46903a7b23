"""float32 dense convolutions (igemm_f32_kernel, wgrad_f32_kernel) at the edges of their tiles and of their launch
rules: every operation of a one-block step against the plain fp64 oracle primitives, elementwise (local_parity.py).
Its 1e-4 is far above what these layers can show: a sum of n float32 products is off by at most n 2^-24 of the sum of
their magnitudes, 3e-6 of the largest result at n = 576 (and by a fraction of it in practice); a wrong index, mask or
partial tile is off by the size of the result."""
import pytest

import local_parity
from paper_2301_12443_amd import workloads as W

pytestmark = pytest.mark.gpu

# (batch, h, w, channels of the block's input, of the layer's input, of its output, k, stride)
SHAPES = [
    (1, 5, 7, 8, 8, 8, 1, 1),            # one run of eight channels, a ragged 35-row tile, 8 of 32 columns
    (3, 9, 11, 8, 40, 72, 3, 1),         # columns 72 = 32 + 32 + 8, five runs a tap
    # images of one pixel: eight of nine taps are padding.  (Not a batch of 2: over two values x-hat is +-1 whatever they
    # are, the gradient behind the normalisation is exactly 0 and all that is left of it is rounding.)
    (40, 1, 1, 16, 16, 24, 3, 1),
    (2, 13, 10, 8, 24, 48, 3, 2),        # stride 2 on an odd image: backward-data by parity
    (2, 12, 14, 8, 16, 40, 7, 2),        # long filter rows
    (4, 8, 8, 16, 256, 64, 3, 1),        # reduction cut over eight waves
    (5, 65, 63, 8, 16, 72, 1, 1),        # 64 x 64 tiles, ragged both ways (20475 rows)
    (4, 64, 64, 8, 8, 64, 3, 1),         # 64 x 64 tiles whose reduction has an odd number of runs (9)
    (1, 6, 6, 8, 136, 200, 1, 1),        # a weight gradient of one split, ragged tiles
]


@pytest.mark.parametrize("n,h,w,c0,ci,co,k,s", SHAPES)
def test_every_operation_of_a_small_block(n, h, w, c0, ci, co, k, s):
    t, b = W.Block(), W.Block()
    t.cba(0, co, k, s, act=W.ACT_NONE)
    v = b.cba(0, ci, 1, act=W.ACT_NONE)
    # two readers of v: the second backward-data launch adds onto the first one's result
    a = b.cba(v, co, k, s, act=W.ACT_NONE)
    c = b.cba(v, co, 1, s, act=W.ACT_NONE)
    b.add(a, c)
    wl = W.Workload("f32_conv", n, (c0, h, w), [t], [b], "f32", lr=0.05)
    worst = local_parity.run_and_check(wl, n, precision="f32")
    print(", ".join(f"{key} {e:.1e}" for key, e in sorted(worst.items())), flush=True)
