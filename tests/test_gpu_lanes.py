"""The candidates of a mixed layer go out together, launches of one kernel in one grid (many_kernel): the same kernels with the same
arguments as one candidate after the other, so every bit is the same.  pbd_student_step_static, whose scratch has no room for several
candidates at a time, is the one-by-one form.  Kernels that only some candidates use, several mixed layers on top of each other, chains of
one to three layers, a candidate that is the input itself, and sizes on every path of the batch norms and of the kernels that take an
expand or projection layer whole (their weight-gradient sums lie in the lane's scratch, and the candidates' gradients of the shared input are
added in order)."""
import numpy as np
import pytest
import torch

import parity
from paper_2301_12443_amd import pbd, workloads as W

pytestmark = pytest.mark.gpu


def _mbconv(b, v, c_in, c, k, e, s):
    v = b.cba(v, c_in * e, 1, act=W.ACT_RELU6)
    v = b.cba(v, c_in * e, k, s, groups=c_in * e, act=W.ACT_RELU6)
    return b.cba(v, c, 1, act=W.ACT_NONE)


# (batch, h, w, stride, (kernel, expansion) of each candidate, further candidates)
CASES = [
    (3, 19, 23, 1, [(3, 3), (5, 6), (7, 3)], "none"),                                     # short columns
    (6, 33, 31, 1, [(3, 3), (3, 6), (5, 3), (5, 6), (7, 3), (7, 6)], "none"),             # the backward pass in one kernel
    (5, 31, 34, 2, [(3, 6), (5, 3), (7, 6)], "none"),
    (70, 9, 8, 1, [(5, 3), (3, 3), (5, 5)], "dense"),                                     # a dense 3 x 3, a single 1 x 1
    (20, 16, 16, 1, [(3, 3), (5, 3)], "identity"),
    (7, 28, 28, 1, [(3, 6), (5, 6), (7, 6), (3, 3), (5, 3), (7, 3), (3, 2), (5, 2)], "none"),   # as many as one launch takes
    (17, 31, 32, 1, [(3, 3), (5, 6), (7, 3), (3, 6), (5, 3), (7, 6)], "none"),            # expand and projection layers in kernels of their own
    (72, 31, 33, 2, [(3, 6), (5, 3), (7, 6)], "identity"),                                # ... behind a stride-2 layer, and beside the input itself
]


@pytest.mark.parametrize("n,h,w,stride,candidates,more", CASES)
def test_candidates_together_and_one_by_one(n, h, w, stride, candidates, more):
    t, b = W.Block(), W.Block()
    t.cba(0, 24, 3, stride, act=W.ACT_NONE)
    v = b.cba(0, 16, 1, act=W.ACT_RELU6)
    for layer, s in enumerate((stride, 1)):
        c_in = 24 if layer else 16
        outs = [_mbconv(b, v, c_in, 24, k, e, s) for k, e in candidates]
        if more == "dense":
            outs += [b.cba(v, 24, 3, act=W.ACT_RELU), b.cba(v, 24, 1, act=W.ACT_NONE)]
        if more == "identity" and layer:
            outs.append(v)
        m = b.mix(outs, [1.0 / len(outs)] * len(outs))
        v = b.add(v, m) if layer else m
    wl = W.Workload("lanes", n, (8, h, w), [t], [b], "bf16", lr=0.05)
    x = torch.from_numpy(W.make_input(wl, batch=n)).cuda()
    a, o = parity.make_distiller(wl, n, "bf16"), parity.make_distiller(wl, n, "bf16")
    for d in (a, o):
        d.teacher_relay(x)
    for step in range(2):
        a.student_step(1, wl.lr)
        o.student_step_static(1, wl.lr)
        a.sync(); o.sync()
        assert np.isfinite(a.losses[0].item()) and a.losses[0].item() == o.losses[0].item()
        for (j, slot), shape in W.param_shapes(wl, W.NET_STUDENT, 0).items():
            for kind in (pbd.PBD_PARAM,) + ((pbd.PBD_GRAD, pbd.PBD_MOMENTUM) if slot <= W.P_BETA else ()):
                np.testing.assert_array_equal(a.read_tensor(kind, 1, 0, j, slot, shape), o.read_tensor(kind, 1, 0, j, slot, shape),
                                              err_msg=f"step {step}, op {j}, slot {slot}, kind {kind}")
        for i in range(1, len(b.ops) + 1):
            np.testing.assert_array_equal(a.read_grad_value(0, i), o.read_grad_value(0, i))
    a.set_profile(True)
    a.student_step(1, wl.lr)
    entries = a.get_profile()
    a.set_profile(False)
    # the six 1 x 1 layers in front and behind alone would be two launches a candidate and mixed layer
    assert sum(p["name"].startswith("igemm_fwd") for p in entries) < 2 * 2 * len(candidates)
    if n * h * w >= 16384:
        names = [p["name"] for p in entries]
        assert {"pw_fwd_store", "pw_bwd_bn", "pj_bwd_bn"} <= set(names), names
        assert names.count("pw_bwd_bn") >= len(candidates) > names.count("pw_fwd_store")      # one after the other, and together
