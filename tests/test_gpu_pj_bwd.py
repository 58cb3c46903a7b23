"""Backward-data and the weight gradient of a projection that normalises the layer in front itself, and that layer's batch-norm sums, in one
kernel (pj_bwd_kernel): every operation of such a block against the plain fp64 oracle primitives on the tensors that the library read, at the
bounds of local_parity.py, the weight gradient at that of a float32 sum (as in test_gpu_dense_fold.py: chains of at most 256 pixels a wave and
516 additions of the waves' and workgroups' sums at these sizes, 3e-3 of the largest component).  One to four groups of outputs, one to
twelve 64-channel groups, partly filled ones, a last tile of one and of 31 pixels, fewer tiles than waves and more than two a wave."""
import numpy as np
import pytest
import torch

import local_parity
import parity
from paper_2301_12443_amd import pbd, workloads as W

pytestmark = pytest.mark.gpu

TOL_DW = 3e-3

# (batch, h, w, channels, outputs, activation, kernel size of the layer in front: 1 dense, else depthwise)
CASES = [
    (16, 32, 32, 96, 16, W.ACT_RELU6, 3),          # the fewest pixels
    (17, 31, 32, 192, 32, W.ACT_RELU6, 5),
    (21, 29, 29, 144, 24, W.ACT_RELU, 7),          # the last tile holds 29 pixels
    (75, 31, 31, 40, 8, W.ACT_RELU6, 3),           # the last of 7
    (1, 129, 129, 64, 16, W.ACT_RELU, 1),          # one pixel in the last tile; a dense layer in front
    (19, 31, 29, 576, 24, W.ACT_RELU6, 3),         # nine groups of channels
    (16, 33, 33, 768, 32, W.ACT_RELU, 1),          # twelve: 42 ranges of pixels, three to four tiles a wave
]


def _classes(d, wl):
    d.set_profile(True)
    d.student_step(1, wl.lr)
    names = [p["name"] for p in d.get_profile()]
    d.set_profile(False)
    return names


@pytest.mark.parametrize("n,h,w,c,out,act,k", CASES)
def test_projection(n, h, w, c, out, act, k):
    t, b = W.Block(), W.Block()
    t.cba(0, 16, 1, act=W.ACT_NONE)
    v = b.cba(0, c, 1, act=act)
    if k > 1:
        v = b.cba(v, c, k, groups=c, act=act)
    u = b.cba(v, out, 1, act=W.ACT_RELU)
    b.cba(u, 16, 3, act=W.ACT_NONE)
    wl = W.Workload("pj_bwd", n, (8, h, w), [t], [b], "bf16", lr=0.05)
    worst = local_parity.run_and_check(wl, n, tol_dw=TOL_DW)
    print(", ".join(f"{key} {e:.1e}" for key, e in sorted(worst.items())), flush=True)
    d = parity.make_distiller(wl, n, "bf16")
    d.teacher_relay(torch.from_numpy(W.make_input(wl, batch=n)).cuda())
    assert _classes(d, wl).count("pj_bwd_bn") == 1


def test_other_layers_keep_the_separate_passes():
    def fused(n, c, out, k, stride):
        t, b = W.Block(), W.Block()
        t.cba(0, 16, 1, stride, act=W.ACT_NONE)
        v = b.cba(0, c, 1, act=W.ACT_RELU6)
        v = b.cba(v, out, k, stride, act=W.ACT_NONE)
        b.cba(v, 16, 1, act=W.ACT_NONE)
        wl = W.Workload("pj_bwd", n, (8, 32, 32), [t], [b], "bf16", lr=0.05)
        d = parity.make_distiller(wl, n, "bf16")
        d.teacher_relay(torch.from_numpy(W.make_input(wl, batch=n)).cuda())
        return "pj_bwd_bn" in _classes(d, wl)
    assert fused(16, 96, 32, 1, 1)
    for other in ((15, 96, 32, 1, 1), (16, 96, 40, 1, 1), (16, 96, 32, 3, 1), (64, 96, 32, 1, 2), (16, 1032, 32, 1, 1)):
        assert not fused(*other), other


def test_architecture_round_forms_the_same_gradients():
    """With the same parameters the architecture round (no weight gradients) and the weight round leave the same gradient of what the
    projections of the second mixed layer read and of the first one's output."""
    n = 17
    b = W.Block()
    v = b.cba(0, 24, 1, act=W.ACT_NONE)
    seen = []
    for layer in range(2):
        outs = []
        for k, e in ((3, 3), (5, 6), (3, 6)):
            u = b.cba(v, 24 * e, 1, act=W.ACT_RELU6)
            u = b.cba(u, 24 * e, k, groups=24 * e, act=W.ACT_RELU6)
            if layer:
                seen.append(u)
            outs.append(b.cba(u, 24, 1, act=W.ACT_NONE))
        v = b.mix(outs, [1.0 / 3] * 3)
        if not layer:
            seen.append(v)
    t = W.Block()
    t.cba(0, 24, 1, act=W.ACT_NONE)
    wl = W.Workload("pj_bwd", n, (8, 31, 32), [t], [b], "bf16", lr=0.05)
    grads = []
    for arch in (True, False):
        d = parity.make_distiller(wl, n, "bf16")
        d.teacher_relay(torch.from_numpy(W.make_input(wl, batch=n)).cuda())
        d.set_profile(True)
        d.arch_step(1, 0.01) if arch else d.student_step(1, wl.lr)
        names = [p["name"] for p in d.get_profile()]
        # the three candidates of a layer in one launch (of the first layer the architecture round takes nothing)
        assert names.count("pj_dgrad_bn" if arch else "pj_bwd_bn") == (1 if arch else 2), names
        grads.append([d.read_grad_value(0, u) for u in seen])
    for got, ref in zip(*grads):
        assert np.abs(ref).max() > 0
        # (other orders of summation in the batch norms' backward pass: the odd value rounds to the next bfloat16 code)
        assert np.abs(got - ref).max() <= 2.0 ** -7 * np.abs(ref).max()
