"""The backward pass of an expand layer (dense 1 x 1, at most 32 inputs and 192 outputs, behind it a batch norm) in one kernel
(pw_bwd_kernel): every operation of such a block against the plain fp64 oracle primitives on the tensors that the library read, at the
bounds of local_parity.py, the weight gradient at that of a float32 sum (as in test_gpu_dense_fold.py: chains of at most 256 pixels a wave and
264 additions of the waves' and workgroups' sums at these sizes, 3e-3 of the largest component).  Every number of 32-channel chunks, partly
filled ones, one to four groups of inputs, three inputs padded to eight, a last tile of one and of 31 pixels, fewer and more tiles than waves."""
import numpy as np
import pytest
import torch

import local_parity
import parity
from paper_2301_12443_amd import pbd, workloads as W

pytestmark = pytest.mark.gpu

TOL_DW = 3e-3

# (batch, h, w, inputs, outputs, activation, kernel size and stride of the depthwise layer behind)
CASES = [
    (17, 31, 32, 32, 192, W.ACT_RELU6, 3, 1),      # 16864 pixels: 527 tiles for 528 waves
    (16, 32, 32, 16, 96, W.ACT_RELU6, 5, 2),       # the fewest pixels
    (21, 29, 29, 24, 144, W.ACT_RELU, 7, 1),       # the last tile holds 29 pixels; half a chunk
    (75, 31, 31, 8, 40, W.ACT_RELU6, 3, 1),        # more tiles than waves, the last of 7 pixels
    (73, 33, 31, 24, 128, W.ACT_RELU, 3, 2),
    (67, 33, 31, 32, 104, W.ACT_RELU6, 5, 1),
    (1, 129, 129, 16, 64, W.ACT_NONE, 3, 1),       # one pixel in the last tile; no rectifier
]


def _block(c_in, c, act, k, stride, first):
    b = W.Block()
    v = 0 if first else b.cba(0, c_in, 1, act=W.ACT_NONE)
    u = b.cba(v, c, 1, act=act)
    u = b.cba(u, c, k, stride, groups=c, act=W.ACT_RELU6)
    u = b.cba(u, c_in, 1, act=W.ACT_NONE)
    if stride == 1 and not first:
        u = b.add(v, u)                            # the input's gradient is there already
        u = b.cba(u, c_in, 1, act=W.ACT_NONE)
    return b


def _classes(d, wl):
    d.set_profile(True)
    d.student_step(1, wl.lr)
    names = [p["name"] for p in d.get_profile()]
    d.set_profile(False)
    return names


@pytest.mark.parametrize("first", [False, True])
@pytest.mark.parametrize("n,h,w,c_in,c,act,k,stride", CASES)
def test_expand_layer(n, h, w, c_in, c, act, k, stride, first):
    t = W.Block()
    t.cba(0, c_in, 1, stride, act=W.ACT_NONE)
    wl = W.Workload("pw_bwd", n, (c_in if first and c_in > 8 else 3 if first else 8, h, w), [t], [_block(c_in, c, act, k, stride, first)], "bf16", lr=0.05)
    worst = local_parity.run_and_check(wl, n, tol_dw=TOL_DW)
    print(", ".join(f"{key} {e:.1e}" for key, e in sorted(worst.items())), flush=True)
    d = parity.make_distiller(wl, n, "bf16")
    d.teacher_relay(torch.from_numpy(W.make_input(wl, batch=n)).cuda())
    assert _classes(d, wl).count("pw_bwd_bn") == 1
    # the gradient of the convolution output is formed on request: each time the same
    v = 1 if first else 2
    np.testing.assert_array_equal(d.read_grad_value(0, v), d.read_grad_value(0, v))


@pytest.mark.parametrize("c,act", [(96, W.ACT_RELU6), (144, W.ACT_RELU), (40, W.ACT_NONE)])
@pytest.mark.parametrize("last", [False, True])
def test_the_gradient_read_is_the_one_the_kernel_used(c, act, last):
    """A filter that copies 16 of the outputs' channels' gradients to the inputs (one weight of one a row and column): backward-data then
    hands out the gradient of the convolution output as the kernel formed it, every bit.  The value in front is a max-pool's, whose
    gradient is kept as it arrives."""
    n, c_in = 16, 16
    t, b = W.Block(), W.Block()
    t.cba(0, 16, 3, 2, act=W.ACT_NONE)
    e = b.cba(b.pool(0, 2, 2), c, 1, act=act)
    b.cba(e, 16, 1, act=W.ACT_NONE)
    wl = W.Workload("pw_bwd", n, (c_in, 64, 64), [t], [b], "bf16", lr=0.05)
    first = c - c_in if last else 0
    w = np.zeros((c, c_in, 1, 1), dtype=np.float32)
    w[first:first + c_in, :, 0, 0] = np.eye(c_in)
    d = parity.make_distiller(wl, n, "bf16")
    d.load_param(W.NET_STUDENT, 0, e - 1, W.P_WEIGHT, w)
    d.teacher_relay(torch.from_numpy(W.make_input(wl, batch=n)).cuda())
    d.set_profile(True)
    d.student_step(1, wl.lr)
    assert "pw_bwd_bn" in {p["name"] for p in d.get_profile()}
    dy = d.read_grad_value(0, e)[:, first:first + c_in]
    assert np.count_nonzero(dy) > dy.size // 2
    np.testing.assert_array_equal(d.read_grad_value(0, e - 1), dy)


def _beside_the_default_stream(make, busy):
    """A distiller whose stream does not share a hardware queue with the legacy default stream: streams are dealt out to a few queues in the
    order in which the process made them, and what waits in one queue runs in order whatever its stream.  make() brings a new one on a stream of its own,
    busy() keeps the default stream at work for a while."""
    made = []
    for _ in range(8):
        d = make()
        made.append(d)
        one = torch.zeros(1, device="cuda")
        torch.cuda.synchronize()
        busy()
        end, done = torch.cuda.Event(), torch.cuda.Event()
        end.record()
        with torch.cuda.stream(d._stream):
            one.add_(1)
            done.record()
        done.synchronize()
        beside = not end.query()
        torch.cuda.synchronize()
        if beside:
            return d
    pytest.fail("every stream shares the default stream's hardware queue")


def test_reading_a_gradient_waits_for_the_bound_stream_alone():
    """read_grad_value of an expand layer and of a depthwise one, whose gradient is formed on request, while another stream (the legacy
    default one) is busy for some hundred times as long as the read takes."""
    n, h, w = 16, 32, 32
    t = W.Block()
    t.cba(0, 16, 1, act=W.ACT_NONE)
    wl = W.Workload("pw_bwd", n, (16, h, w), [t], [_block(16, 96, W.ACT_RELU6, 3, 1, True)], "bf16", lr=0.05)
    a = torch.randn(8192, 8192, device="cuda", dtype=torch.bfloat16)
    out = a @ a
    torch.cuda.synchronize()

    def keep_busy(products):
        for _ in range(products):
            torch.matmul(a, a, out=out)
    d = _beside_the_default_stream(lambda: parity.make_distiller(wl, n, "bf16"), lambda: keep_busy(60))
    d.teacher_relay(torch.from_numpy(W.make_input(wl, batch=n)).cuda())
    assert {"pw_bwd_bn", "dw_wgrad_mfma_bn_k3"} <= set(_classes(d, wl))
    d.sync()
    for v in (1, 2):
        want = d.read_grad_value(0, v)
        keep_busy(600)                                 # 0.4 s and more
        end = torch.cuda.Event()
        end.record()
        got = d.read_grad_value(0, v)
        busy = not end.query()
        torch.cuda.synchronize()
        assert busy, f"value {v}"
        np.testing.assert_array_equal(got, want)


def test_other_layers_keep_the_separate_passes():
    def fused(n, c_in, c, k, stride, residual=False):
        b = W.Block()
        v = b.cba(0, c_in, 1, act=W.ACT_NONE)
        if residual:
            b.add(b.cba(0, c, 1, act=W.ACT_NONE), b.cba(v, c, 1, act=W.ACT_NONE))
        else:
            b.cba(v, c, k, stride, act=W.ACT_RELU)
        b.cba(len(b.ops), 8, 1, act=W.ACT_NONE)
        t = W.Block()
        t.cba(0, 8, 1, stride, act=W.ACT_NONE)
        wl = W.Workload("pw_bwd", n, (40, 32, 32), [t], [b], "bf16", lr=0.05)
        d = parity.make_distiller(wl, n, "bf16")
        d.teacher_relay(torch.from_numpy(W.make_input(wl, batch=n)).cuda())
        return "pw_bwd_bn" in _classes(d, wl)
    assert fused(16, 16, 64, 1, 1)
    for other in ((15, 16, 64, 1, 1), (16, 40, 64, 1, 1), (16, 16, 200, 1, 1), (16, 16, 32, 1, 1), (16, 16, 64, 3, 1), (64, 16, 64, 1, 2),
                  (16, 16, 64, 1, 1, True)):
        assert not fused(*other), other


def test_architecture_round_forms_the_same_input_gradients():
    """With the same parameters the architecture round (no weight gradients) and the weight round leave the same gradient of the first mixed
    layer's output, which six expand layers add to."""
    n = 17
    b = W.Block()
    v = b.cba(0, 24, 1, act=W.ACT_NONE)
    for layer in range(2):
        outs = []
        for k, e in ((3, 3), (5, 6), (3, 6)):
            u = b.cba(v, 24 * e, 1, act=W.ACT_RELU6)
            u = b.cba(u, 24 * e, k, groups=24 * e, act=W.ACT_RELU6)
            outs.append(b.cba(u, 24, 1, act=W.ACT_NONE))
        v = b.mix(outs, [1.0 / 3] * 3)
        first = v if layer == 0 else first
    t = W.Block()
    t.cba(0, 24, 1, act=W.ACT_NONE)
    wl = W.Workload("pw_bwd", n, (8, 31, 32), [t], [b], "bf16", lr=0.05)
    grads = []
    for arch in (True, False):
        d = parity.make_distiller(wl, n, "bf16")
        d.teacher_relay(torch.from_numpy(W.make_input(wl, batch=n)).cuda())
        d.set_profile(True)
        d.arch_step(1, 0.01) if arch else d.student_step(1, wl.lr)
        names = {p["name"] for p in d.get_profile()}
        assert ("pw_dgrad_bn" if arch else "pw_bwd_bn") in names, names
        grads.append(d.read_grad_value(0, first))
    assert np.abs(grads[1]).max() > 0
    # (sums of other groups of pixels go into the batch norms' backward pass: the odd value rounds to the next bfloat16 code)
    assert np.abs(grads[0] - grads[1]).max() <= 2.0 ** -7 * np.abs(grads[1]).max()
