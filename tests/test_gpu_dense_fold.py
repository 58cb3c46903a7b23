"""A layer whose only reader is a dense 1 x 1 layer of at most 32 outputs leaves its normalisation to it (igemm_kernel and
wgrad_tr_kernel, FOLD): every operation of such a block against the plain fp64 oracle primitives on the tensors that the library read, at
the bounds of local_parity.py, the weight gradient at that of a float32 sum (as in test_gpu_dw_mfma.py: chains of at most 400 + pixels /
splits additions, 3e-3 of the largest component at these sizes).  Channel counts on each of the three ways the reduction is walked, tiles
of 64 and 128 rows, ragged rows and columns, the last channel group of a step half empty."""
import pytest

import local_parity
import parity
from paper_2301_12443_amd import pbd, workloads as W

pytestmark = pytest.mark.gpu

TOL_DW = 3e-3

# (batch, h, w, channels, outputs, activation)
CASES = [
    (6, 33, 31, 192, 16, W.ACT_RELU6),     # 64-row tiles; K step 64
    (5, 29, 30, 96, 32, W.ACT_RELU),       # K step 32, exactly 32 columns
    (9, 23, 21, 72, 24, W.ACT_RELU6),      # a step across the end of the channels
    (17, 16, 16, 8, 8, W.ACT_RELU),        # one vector of channels, one of outputs
    (5, 31, 27, 576, 24, W.ACT_RELU6),     # nine steps
    (70, 31, 31, 64, 16, W.ACT_RELU),      # 128-row tiles
    (70, 31, 31, 96, 24, W.ACT_RELU6),
    (70, 31, 31, 40, 32, W.ACT_RELU6),
    (70, 31, 31, 144, 8, W.ACT_RELU),
]


@pytest.mark.parametrize("n,h,w,c,out,act", CASES)
def test_normalisation_in_the_dense_reader(n, h, w, c, out, act):
    t, b = W.Block(), W.Block()
    t.cba(0, 16, 1, act=W.ACT_NONE)
    v = b.cba(0, c, 1, act=act)
    v = b.cba(v, out, 1, act=W.ACT_RELU)
    b.cba(v, 16, 3, act=W.ACT_NONE)
    wl = W.Workload("dense_fold", n, (8, h, w), [t], [b], "bf16", lr=0.05)
    worst = local_parity.run_and_check(wl, n, tol_dw=TOL_DW)
    print(", ".join(f"{key} {e:.1e}" for key, e in sorted(worst.items())), flush=True)


def test_what_is_folded():
    import torch
    def names(c, out, k, stride, readers):
        t, b = W.Block(), W.Block()
        t.cba(0, 16, 1, stride, act=W.ACT_NONE)
        v = b.cba(0, c, 1, act=W.ACT_RELU6)
        u = b.cba(v, out, k, stride, act=W.ACT_NONE)
        if readers == 2:
            u = b.add(u, b.cba(v, out, 1, stride, act=W.ACT_NONE))
        b.cba(u, 16, 1, act=W.ACT_NONE)
        wl = W.Workload("dense_fold", 6, (8, 33, 31), [t], [b], "bf16", lr=0.05)
        d = parity.make_distiller(wl, 6, "bf16")
        d.teacher_relay(torch.from_numpy(W.make_input(wl, batch=6)).cuda())
        d.set_profile(True)
        d.student_step(1, wl.lr)
        return {p["name"] for p in d.get_profile() if p["net"] == pbd.PBD_STUDENT and p["op"] <= 1}
    assert any("bn_store" in x for x in names(96, 32, 1, 1, 1))
    for other in ((96, 40, 1, 1, 1), (96, 32, 3, 1, 1), (96, 32, 1, 2, 1), (96, 32, 1, 1, 2), (1032, 32, 1, 1, 1)):
        assert not any("bn_store" in x for x in names(*other)), other
