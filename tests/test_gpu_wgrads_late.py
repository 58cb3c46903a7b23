"""A block's small weight gradients go out together at its end, those of one kernel in one grid of up to eight (find_late, flush_late).
pbd_student_step_static sends every one out by itself and adds its partial sums at once: every bit of a step is the same.  More than eight layers of one kernel, tiles of every width, kernels that are alone, depthwise layers of both
strides, one tile without partial sums; and against the plain fp64 oracle primitives at the bounds of local_parity.py."""
import numpy as np
import pytest
import torch

import local_parity
import parity
from paper_2301_12443_amd import pbd, workloads as W

pytestmark = pytest.mark.gpu


def _chain(widths):
    def build(b):
        v = 0
        for c in widths:
            v = b.cba(v, c, 1, act=W.ACT_RELU)
        return v
    return build


def _depthwise(b):
    v = b.cba(0, 72, 1, act=W.ACT_NONE)
    for k, s in ((3, 1), (5, 1), (7, 1), (3, 2), (5, 1), (3, 1)):
        v = b.cba(v, 72, k, s, groups=72, act=W.ACT_RELU)
        v = b.cba(v, 72, 1, act=W.ACT_NONE)
    return v


CASES = [
    (5, 13, 11, _chain([136] * 10), 1),                       # ten of one kernel, ragged pixels
    (7, 12, 12, _chain([40, 136, 40, 72, 136, 200, 56]), 1),  # 64 and 128 wide tiles
    (30, 17, 16, _depthwise, 2),
    (1, 3, 3, _chain([24, 40, 24]), 1),                       # fewer pixels than a step: no partial sums
]


def _workload(n, h, w, build, stride, precision):
    t, b = W.Block(), W.Block()
    t.cba(0, 48, 1, stride, act=W.ACT_NONE)
    b.cba(build(b), 48, 3, act=W.ACT_NONE)
    return W.Workload("late", n, (16, h, w), [t], [b], precision, lr=0.05)


@pytest.mark.parametrize("precision", ["bf16", "f32"])
@pytest.mark.parametrize("n,h,w,build,stride", CASES)
def test_together_and_one_by_one(n, h, w, build, stride, precision):
    wl = _workload(n, h, w, build, stride, precision)
    x = torch.from_numpy(W.make_input(wl, batch=n)).cuda()
    a, o = parity.make_distiller(wl, n, precision), parity.make_distiller(wl, n, precision)
    for d in (a, o):
        d.teacher_relay(x)
    for step in range(2):
        a.student_step(1, wl.lr)
        o.student_step_static(1, wl.lr)
        a.sync(); o.sync()
        assert np.isfinite(a.losses[0].item()) and a.losses[0].item() == o.losses[0].item()
        for (j, slot), shape in W.param_shapes(wl, W.NET_STUDENT, 0).items():
            kinds = [pbd.PBD_PARAM] + ([pbd.PBD_GRAD, pbd.PBD_MOMENTUM] if slot <= W.P_BETA else [])
            for kind in kinds:
                np.testing.assert_array_equal(a.read_tensor(kind, 1, 0, j, slot, shape), o.read_tensor(kind, 1, 0, j, slot, shape),
                                              err_msg=f"step {step}, op {j}, slot {slot}, kind {kind}")


@pytest.mark.parametrize("precision", ["bf16", "f32"])
@pytest.mark.parametrize("n,h,w,build,stride", CASES)
def test_fewer_launches_than_layers(n, h, w, build, stride, precision):
    wl = _workload(n, h, w, build, stride, precision)
    d = parity.make_distiller(wl, n, precision)
    d.teacher_relay(torch.from_numpy(W.make_input(wl, batch=n)).cuda())
    d.set_profile(True)
    d.student_step(1, wl.lr)
    launches = [p["name"] for p in d.get_profile() if p["name"].startswith("wgrad_")]
    assert len(launches) < sum(op.type == W.OP_CBA and op.groups == 1 for op in wl.student[0].ops), launches


@pytest.mark.parametrize("n,h,w,build,stride", CASES[:3])
def test_against_the_oracle(n, h, w, build, stride):
    wl = _workload(n, h, w, build, stride, "bf16")
    worst = local_parity.run_and_check(wl, n)
    print(", ".join(f"{key} {e:.1e}" for key, e in sorted(worst.items())), flush=True)
