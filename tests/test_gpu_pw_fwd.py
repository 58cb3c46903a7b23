"""The forward pass of an expand layer (dense 1 x 1, at most 32 inputs, 33 to 192 outputs) in a kernel of its own (pw_fwd_kernel): the
student's with its batch norm, the frozen teacher's with the folded one, against the plain fp64 oracle primitives at the bounds of
local_parity.py; the batch statistics also where every channel lies far from zero, and where the first pixel lies far from all others (a workgroup's sums are
shifted by its first pixel).  One to three
groups of 64 channels, partly filled ones, one to four groups of inputs, three inputs padded to eight, a last tile of one to 31 pixels, fewer
tiles than waves and more than two a wave."""
import numpy as np
import pytest
import torch

import local_parity
import parity
from oracle import pbd_oracle as orc
from paper_2301_12443_amd import pbd, workloads as W

pytestmark = pytest.mark.gpu

# (batch, h, w, inputs, outputs, activation)
CASES = [
    (16, 32, 32, 16, 96, W.ACT_RELU6),             # the fewest pixels
    (17, 31, 32, 32, 192, W.ACT_RELU6),
    (21, 29, 29, 24, 144, W.ACT_RELU),             # the last tile holds 29 pixels
    (75, 31, 31, 8, 40, W.ACT_NONE),               # the last of 7
    (75, 31, 31, 3, 72, W.ACT_RELU6),
    (1, 129, 129, 16, 64, W.ACT_RELU),             # one pixel in the last tile
    (60, 57, 57, 32, 160, W.ACT_RELU6),            # 6092 tiles: six a wave
]


def _workload(n, h, w, c_in, c, act):
    t, b = W.Block(), W.Block()
    t.cba(t.cba(0, c, 1, act=act), 16, 3, act=W.ACT_NONE)
    b.cba(b.cba(0, c, 1, act=act), 16, 3, act=W.ACT_NONE)
    return W.Workload("pw_fwd", n, (c_in, h, w), [t], [b], "bf16", lr=0.05)


@pytest.mark.parametrize("n,h,w,c_in,c,act", CASES)
def test_expand_layer(n, h, w, c_in, c, act):
    wl = _workload(n, h, w, c_in, c, act)
    worst = local_parity.run_and_check(wl, n, {0: ({0}, set())})
    print(", ".join(f"{key} {e:.1e}" for key, e in sorted(worst.items())), flush=True)
    d = parity.make_distiller(wl, n, "bf16")
    d.set_profile(True)
    d.teacher_relay(torch.from_numpy(W.make_input(wl, batch=n)).cuda())
    d.student_step(1, wl.lr)
    names = [p["name"] for p in d.get_profile()]
    assert names.count("pw_fwd_affine") == 1 and names.count("pw_fwd_store") == 1, names
    err = local_parity.teacher_block_error(d, wl, 0, (0, n // 2, n - 1))
    assert err < local_parity.TOL_BF16, err


def test_statistics_far_from_zero():
    """Images with an offset of 30 standard deviations, filters of one sign: means far above the deviations."""
    n, h, w, c_in, c = 16, 33, 32, 16, 96
    wl = _workload(n, h, w, c_in, c, W.ACT_RELU)
    d = parity.make_distiller(wl, n, "bf16")
    (j, slot), shape = next((k, s) for k, s in W.param_shapes(wl, W.NET_STUDENT, 0).items() if k == (0, W.P_WEIGHT))
    d.load_param(W.NET_STUDENT, 0, j, slot, np.abs(W.make_param(wl, W.NET_STUDENT, 0, j, slot, shape)) + 0.05)
    d.teacher_relay(torch.from_numpy(W.make_input(wl, batch=n) + 30.0).cuda())
    d.student_step(1, wl.lr)
    d.sync()
    y = d.read_conv_out(0, 0).astype(np.float64)
    mean, var = y.mean(axis=(0, 2, 3)), y.var(axis=(0, 2, 3))
    assert (np.abs(mean) > 10 * np.sqrt(var)).all()
    mg, ig = d.read_batch_stats(0, 0)
    # chains of at most 16 additions a lane and 8 + 4 across: 28 roundings of 2^-24, of the deviations from a first pixel (within 6 of them)
    assert np.abs(mg - mean).max() / np.sqrt(var).min() < 1e-3 and np.abs((mg - mean) / mean).max() < 2.0 ** -23
    assert np.abs(ig * np.sqrt(var + 1e-5) - 1.0).max() < 28 * 2.0 ** -24 * 37


@pytest.mark.parametrize("n,h,w,c_in,c", [(64, 64, 64, 16, 96), (17, 31, 32, 32, 192), (75, 31, 31, 8, 40)])
def test_statistics_with_a_first_pixel_far_from_the_others(n, h, w, c_in, c):
    """Blank images but for the very first pixel: every other difference from it is the same number, whose square's rounding adds up."""
    wl = _workload(n, h, w, c_in, c, W.ACT_RELU)
    x = np.ones((n, c_in, h, w), dtype=np.float32)
    x[0, :, 0, 0] = W.make_input(wl, batch=1)[0, :, 0, 0] * 300.0
    d = parity.make_distiller(wl, n, "bf16")
    d.teacher_relay(torch.from_numpy(x).cuda())
    d.student_step(1, wl.lr)
    d.sync()
    y = d.read_conv_out(0, 0).astype(np.float64)
    mean, var = y.mean(axis=(0, 2, 3)), y.var(axis=(0, 2, 3))
    far = var > 100 * 1e-5                       # (where the epsilon does not hide the variance)
    assert far.sum() > c // 2
    mg, ig = d.read_batch_stats(0, 0)
    # M var = D^2 (M - 1) / M; the first workgroup's `own` pixels have a sum of squares of (own - 1) D^2: chains of at most 24 additions a lane
    # and 8 + 4 across, 36 roundings of 2^-24 of it, half of that in the inverse root (own: 8 rounds of 4 waves with 32 pixels at most)
    own = 4 * 32 * max(1, -(-n * h * w // (768 // -(-c // 64) * 128)))
    err = np.abs(ig * np.sqrt(var + 1e-5) - 1.0)[far].max()
    print(f"{own} pixels: {err:.2e}, mean {np.abs(mg - mean).max():.2e}", flush=True)
    assert err < 18 * 2.0 ** -24 * own
    # (the mean: the first workgroup's is D off its first pixel, D = sqrt(M var), and weighs own / M)
    assert (np.abs(mg - mean) < 36 * 2.0 ** -24 * (np.abs(mean) + np.sqrt(var) * max(1.0, own / np.sqrt(n * h * w)))).all()
