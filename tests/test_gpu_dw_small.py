"""3 x 3 depthwise layers of short columns, which take the batch norms around them along (dw_small_fwd_kernel, dw_small_bwd_kernel), at the
edges: images of two pixels, of one row and of one column, rows around a whole number of waves and of 512, the most rows that take
the fused kernels and one image more, few channels, every rectifier; a layer that reads the block's input, one behind a dense layer,
one behind a depthwise layer, and one whose input has another reader.  Every operation of a one-block step against the plain fp64 oracle
primitives on the tensors that the library read, at the bounds of local_parity.py; and bit for bit against the separate launches."""
import numpy as np
import pytest
import torch

import local_parity
from paper_2301_12443_amd import pbd, workloads as W

pytestmark = pytest.mark.gpu

# (batch, h, w, channels, rectifier)
SHAPES = [
    (40, 1, 2, 8, W.ACT_RELU),
    (40, 1, 5, 24, W.ACT_RELU6),
    (37, 7, 1, 40, W.ACT_NONE),
    (64, 2, 4, 64, W.ACT_RELU),           # 512 rows
    (33, 4, 4, 96, W.ACT_RELU),           # 528
    (85, 4, 4, 136, W.ACT_RELU6),         # 1360
    (128, 4, 4, 32, W.ACT_RELU),          # 2048: the most ...
    (129, 4, 4, 32, W.ACT_RELU),          # ... and one image more
]


@pytest.mark.parametrize("precision", ["bf16", "f32"])
@pytest.mark.parametrize("n,h,w,c,act", SHAPES)
def test_every_operation_of_a_small_block(n, h, w, c, act, precision):
    t, b = W.Block(), W.Block()
    t.cba(0, c, 1, act=W.ACT_NONE)
    v = b.cba(0, 16, 3, groups=16, act=act)
    v = b.cba(v, c, 1, act=act)
    v = b.cba(v, c, 3, groups=c, act=act)
    v = b.cba(v, c, 3, groups=c, act=act)
    v = b.cba(v, c, 1, act=act)
    b.add(v, b.cba(v, c, 3, groups=c, act=W.ACT_NONE))
    worst = local_parity.run_and_check(W.Workload("dw_small", n, (16, h, w), [t], [b], precision, lr=0.05), n, precision=precision)
    print(", ".join(f"{key} {e:.1e}" for key, e in sorted(worst.items())), flush=True)


@pytest.mark.parametrize("precision", ["bf16", "f32"])
@pytest.mark.parametrize("n,h,w,c,act", [x for x in SHAPES if x[0] != 129])
def test_same_bits_as_the_separate_launches(n, h, w, c, act, precision):
    """bfloat16: the layers with zeros added to what comes out of them, by one more layer whose weights are zeros or by a mixed layer of two.
    float32: force_direct, whose kernels add in the same order."""
    def run(separate):
        mixed = separate and precision == "bf16"
        t, b = W.Block(), W.Block()
        t.cba(0, c, 1, act=W.ACT_NONE)
        v = b.cba(0, 16, 3, groups=16, act=act)
        v = b.cba(v, c, 1, act=act)
        v = b.cba(v, c, 3, groups=c, act=act)
        v = b.cba(v, c, 3, groups=c, act=act)
        chain = b.cba(v, c, 1, act=act)
        z = [b.cba(0, c, 1, act=W.ACT_NONE) for _ in range(1 + mixed)]
        b.add(chain, b.mix(z, (0.5, 0.5)) if mixed else z[0])
        wl = W.Workload("dw_small_bits", n, (16, h, w), [t], [b], precision, lr=0.05)
        d = pbd.Distiller(wl, force_direct=separate and not mixed)
        d.bind("cuda:0")
        d.load_params()
        for v in z:
            d.load_param(W.NET_STUDENT, 0, v - 1, W.P_WEIGHT, np.zeros((c, 16, 1, 1), dtype=np.float32))
        d.teacher_relay(torch.from_numpy(W.make_input(wl)).cuda())
        d.set_profile(True)
        d.student_step(1, wl.lr)
        d.sync()
        names = {p["name"] for p in d.get_profile() if p["name"].startswith("dw_small")}
        assert names == (set() if separate else {"dw_small_fwd", "dw_small_fwd_bn", "dw_small_bwd", "dw_small_bwd_bn"}), names
        got = {"loss": d.losses.cpu().numpy()}
        shapes = W.param_shapes(wl, W.NET_STUDENT, 0)
        for j in range(chain):
            got[f"conv{j}"], got[f"value{j}"], got[f"grad{j}"] = d.read_conv_out(0, j), d.read_value(0, j + 1), d.read_grad_value(0, j + 1)
            got[f"mean{j}"], got[f"invstd{j}"] = d.read_batch_stats(0, j)
            for slot in (W.P_WEIGHT, W.P_GAMMA, W.P_BETA):
                got[f"grad{j}.{slot}"] = d.read_tensor(pbd.PBD_GRAD, 1, 0, j, slot, shapes[(j, slot)])
            for slot in range(W.P_RVAR + 1):
                got[f"param{j}.{slot}"] = d.read_tensor(pbd.PBD_PARAM, 1, 0, j, slot, shapes[(j, slot)])
        return got
    ref, got = run(True), run(False)
    for name in ref:
        np.testing.assert_array_equal(got[name], ref[name], err_msg=name)
