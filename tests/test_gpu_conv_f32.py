"""float32 dense convolutions (igemm_f32_kernel, wgrad_f32_kernel) at the edges of their tiles and of their launch
rules: every operation of a one-block step against the plain fp64 oracle primitives, elementwise (local_parity.py), and
bit for bit against the direct kernels (force_direct), whose order of summation they keep.
The first's 1e-4 is far above what these layers can show: a sum of n float32 products is off by at most n 2^-24 of the sum of
their magnitudes, 3e-6 of the largest result at n = 576 (and by a fraction of it in practice); a wrong index, mask or
partial tile is off by the size of the result."""
import numpy as np
import pytest

import local_parity
import parity
from paper_2301_12443_amd import pbd, workloads as W

pytestmark = pytest.mark.gpu

# (batch, h, w, channels of the block's input, of the layer's input, of its output, k, stride)
SHAPES = [
    (1, 5, 7, 8, 8, 8, 1, 1),            # one run of eight channels, a ragged 35-row tile, 8 of 16 columns
    (3, 9, 11, 8, 40, 72, 3, 1),         # columns 72 = 4 x 16 + 8, five runs a tap
    # images of one pixel: eight of nine taps are padding.  (Not a batch of 2: over two values x-hat is +-1 whatever they
    # are, the gradient behind the normalisation is exactly 0 and all that is left of it is rounding.)
    (40, 1, 1, 16, 16, 24, 3, 1),
    (2, 13, 10, 8, 24, 48, 3, 2),        # stride 2 on an odd image: backward-data by parity
    (2, 12, 14, 8, 16, 40, 7, 2),        # long filter rows
    (4, 8, 8, 16, 256, 64, 3, 1),        # a long chain
    (5, 65, 63, 8, 16, 72, 1, 1),        # 32 x 32 tiles, ragged both ways (20475 rows)
    (4, 64, 64, 8, 8, 64, 3, 1),         # 16384 rows whose reduction has an odd number of runs (9)
    (1, 6, 6, 8, 136, 200, 1, 1),        # a weight gradient of one stage, ragged tiles
    (17, 65, 63, 8, 8, 40, 3, 1),        # 64 x 64 tiles, ragged both ways (69615 rows), 40 of 64 columns
    (2, 9, 8, 16, 112, 1040, 3, 1),      # weight gradient on 64 x 64 tiles (17 x 16 of them, ragged both ways)
]


def _workload(n, h, w, c0, ci, co, k, s):
    t, b = W.Block(), W.Block()
    t.cba(0, co, k, s, act=W.ACT_NONE)
    v = b.cba(0, ci, 1, act=W.ACT_NONE)
    # two readers of v: the second backward-data launch adds onto the first one's result
    a = b.cba(v, co, k, s, act=W.ACT_NONE)
    c = b.cba(v, co, 1, s, act=W.ACT_NONE)
    b.add(a, c)
    return W.Workload("f32_conv", n, (c0, h, w), [t], [b], "f32", lr=0.05)


@pytest.mark.parametrize("n,h,w,c0,ci,co,k,s", SHAPES)
def test_every_operation_of_a_small_block(n, h, w, c0, ci, co, k, s):
    worst = local_parity.run_and_check(_workload(n, h, w, c0, ci, co, k, s), n, precision="f32")
    print(", ".join(f"{key} {e:.1e}" for key, e in sorted(worst.items())), flush=True)


def _everything(wl, force_direct, steps, loaded=()):
    """All that `steps` steps leave behind, by name."""
    import torch
    d = parity.make_distiller(wl, force_direct=force_direct)
    for net, b, j, arr in loaded:
        d.load_param(net, b, j, W.P_WEIGHT, arr)
    out = {}
    for step in range(steps):
        d.teacher_relay(torch.from_numpy(W.make_input(wl, step=step)).cuda())
        for b in range(wl.B):
            d.student_step(b + 1, wl.lr)
        d.sync()
    for b in range(wl.B):
        out[f"A_{b + 1}"] = d.read_act(b + 1)
        for (j, slot), shape in W.param_shapes(wl, W.NET_STUDENT, b).items():
            out[f"param{b}.{j}.{slot}"] = d.read_tensor(pbd.PBD_PARAM, 1, b, j, slot, shape)
            if slot <= W.P_BETA:
                out[f"grad{b}.{j}.{slot}"] = d.read_tensor(pbd.PBD_GRAD, 1, b, j, slot, shape)
    out["losses"] = d.losses.cpu().numpy()
    return out


@pytest.mark.parametrize("wl,steps", [(_workload(*s), 2) for s in SHAPES] + [(W.tiny_cnn(8), 4)],
                         ids=[str(s) for s in SHAPES] + ["tiny_cnn"])
def test_same_bits_as_the_direct_kernels(wl, steps):
    ref, got = _everything(wl, True, steps), _everything(wl, False, steps)
    for name in ref:
        np.testing.assert_array_equal(got[name], ref[name], err_msg=name)


def test_non_finite_weights_stay_where_the_direct_kernels_leave_them():
    """An infinity and a NaN in the teacher's and the student's filters: taps outside the image are left out, not
    multiplied by zero."""
    wl = _workload(2, 13, 10, 8, 24, 48, 3, 2)
    wt = W.make_param(wl, W.NET_TEACHER, 0, 0, W.P_WEIGHT, (48, 8, 3, 3)).copy()
    ws = W.make_param(wl, W.NET_STUDENT, 0, 1, W.P_WEIGHT, (48, 24, 3, 3)).copy()
    wt[5, 3, 0, 0], wt[6, 1, 2, 2], ws[7, 9, 0, 2] = np.inf, np.nan, -np.inf
    loaded = [(W.NET_TEACHER, 0, 0, wt), (W.NET_STUDENT, 0, 1, ws)]
    ref, got = _everything(wl, True, 1, loaded), _everything(wl, False, 1, loaded)
    assert np.isfinite(ref["A_1"][:, 5]).any() and not np.isfinite(ref["A_1"][:, 5]).all()
    for name in ref:
        np.testing.assert_array_equal(got[name], ref[name], err_msg=name)
