"""The small-tile implicit GEMM with its operands in a ring of LDS stages (igemm_kernel, RING) and the tile that such a launch takes
(free_tile), at the edges: fewer and more reduction steps than stages, K steps of 64 and 32, a reduction cut in two, ragged rows and
columns, every tile shape with every depth of the ring that the dispatch gives it, stride 2 both ways, images smaller than the filter, and launches
that add to a gradient.  Every operation of a one-block step against the plain fp64 oracle primitives on the tensors that the library read, at the
bf16 bound of local_parity.py: one rounding to bfloat16 separates the two sides (2^-9 of a value, up to twice that where two are added), a
wrong index, mask or stage is off by the size of the result.  The profile classes say which tile and ring ran, on a chip of 256 compute
units.  And bit for bit against the kernel that stages through registers, which layers of 48 channels take: the same layers with zeros
for channels 48 to 63 or 95 go through the ring."""
import numpy as np
import pytest
import torch

import local_parity
import parity
from paper_2301_12443_amd import pbd, workloads as W

pytestmark = pytest.mark.gpu

# (batch, h, w, channels of the block's input, of the layer's input, of its output, k, stride)
SHAPES = [
    (1, 9, 7, 64, 64, 64, 1, 1),         # one step, 63 rows: a ragged tile of 64 x 64
    (5, 4, 4, 64, 128, 72, 1, 1),        # two steps of three stages, 72 of 128 columns
    (3, 5, 5, 64, 192, 512, 1, 1),       # three steps
    (85, 2, 2, 64, 512, 512, 1, 1),      # 340 rows, eight steps
    (9, 2, 2, 64, 256, 512, 3, 1),       # images smaller than the filter, 36 rows, the reduction cut in two
    (13, 7, 7, 64, 320, 1024, 1, 1),     # 637 rows, five steps
    (64, 7, 7, 64, 192, 2048, 1, 1),     # 128 x 128 tiles, ragged rows (3136)
    (20, 14, 14, 64, 64, 128, 3, 1),     # 3920 rows
    (6, 13, 13, 64, 128, 192, 3, 2),     # stride 2 on an odd image: backward-data by parity
    (6, 12, 12, 64, 96, 160, 3, 1),      # K step 32
    (33, 7, 7, 32, 160, 96, 1, 1),       # ... five steps, 96 columns
    (30, 13, 13, 64, 384, 64, 1, 1),     # 5070 rows: batch-norm sums in the store
    (40, 12, 12, 32, 96, 32, 1, 1),      # ... 32 columns
]


def _workload(n, h, w, c0, ci, co, k, s):
    t, b = W.Block(), W.Block()
    t.cba(0, co, k, s, act=W.ACT_NONE)
    v = b.cba(0, ci, 1, act=W.ACT_NONE)
    # two readers of v: the second backward-data launch adds onto the first one's result
    a = b.cba(v, co, k, s, act=W.ACT_NONE)
    c = b.cba(v, co, 1, s, act=W.ACT_NONE)
    b.add(a, c)
    return W.Workload("ring_small", n, (c0, h, w), [t], [b], "bf16", lr=0.05)


@pytest.mark.parametrize("n,h,w,c0,ci,co,k,s", SHAPES)
def test_every_operation_of_a_small_block(n, h, w, c0, ci, co, k, s):
    worst = local_parity.run_and_check(_workload(n, h, w, c0, ci, co, k, s), n, precision="bf16")
    print(", ".join(f"{key} {e:.1e}" for key, e in sorted(worst.items())), flush=True)


# (batch, h, w, channels of the layer's input, of its output, k), of the layer's launches: forward, backward-data, backward-data that adds (None: not
# looked at).  128x64r2: a tile of 128 x 64 with a ring of two stages.
RINGS = [
    # K step 64
    ((32, 7, 7, 256, 2560, 1), "64x128r3_store", None, None),              # 500 tiles: two a unit; four steps
    ((32, 7, 7, 2560, 256, 1), None, "64x128r3_store", "64x128r3_accum"),
    ((1, 9, 7, 512, 2048, 5), "64x128r3_partial", None, None),
    ((1, 9, 7, 2048, 512, 5), None, "64x128r3_partial", "64x128r3_partial"),
    ((43, 7, 7, 320, 2048, 1), "64x128r2_store", None, None),              # 528 tiles: three a unit; five steps
    ((43, 7, 7, 2048, 320, 1), None, "64x128r2_store", "64x128r2_accum"),
    ((60, 13, 13, 256, 160, 2), "64x128r2_partial", None, None),
    ((20, 7, 7, 768, 768, 2), "64x128r2_partial", "64x128r2_partial", "64x128r2_partial"),
    ((64, 7, 7, 256, 2048, 1), "128x128r2_store", None, None),             # 400 tiles; four steps
    ((64, 7, 7, 2048, 256, 1), None, "128x128r2_store", "128x128r2_accum"),
    ((64, 7, 7, 256, 1024, 1), "64x128r3_store", None, None),              # (200 of them: one a unit)
    ((80, 7, 7, 256, 640, 2), "128x128r2_partial", None, None),
    ((64, 7, 7, 1024, 256, 2), None, "128x128r2_partial", "128x128r2_partial"),
    ((1, 9, 7, 256, 256, 2), "64x64r3_partial", "64x64r3_partial", "64x64r3_partial"),
    ((1, 9, 7, 64, 64, 3), "64x64r3_store", "64x64r3_store", "64x64r3_accum"),
    ((2, 9, 7, 64, 32, 3), "64x32r3_store", None, None),                   # (wave pairs that only load)
    ((2, 9, 7, 32, 64, 3), None, "64x32r3_store", "64x32r3_accum"),
    ((1, 9, 7, 32, 256, 2), None, "64x32r3_partial", "64x32r3_partial"),
    ((40, 41, 40, 64, 48, 2), "128x64r2_store", None, None),               # batch-norm sums in the store
    ((40, 41, 40, 64, 32, 2), "128x32r2_store", None, None),
    ((40, 41, 40, 32, 64, 2), "128x64r3_store", "128x32r2_store", "128x32r2_accum"),
    # K step 32
    ((2, 9, 7, 96, 160, 3), "64x128r3_store", "64x64r3_partial", "64x64r3_partial"),
    ((2, 9, 7, 160, 32, 3), "64x32r3_partial", "64x128r3_store", "64x128r3_accum"),
    ((64, 7, 7, 32, 2048, 2), "128x128r3_store", None, None),
    ((33, 28, 28, 320, 32, 2), None, "128x128r3_store", None),
    ((40, 41, 40, 64, 32, 2), None, "128x64r3_store", "128x64r3_accum"),
    ((40, 41, 40, 32, 512, 2), "256x128r2_store", None, None),
    ((40, 41, 40, 512, 32, 2), None, "256x128r2_store", None),
]


def _layer(n, h, w, ci, co, k, twice):
    t, b = W.Block(), W.Block()
    t.cba(0, co, k, act=W.ACT_NONE)
    v = b.cba(0, ci, 1, act=W.ACT_NONE)
    u = b.cba(v, co, k, act=W.ACT_NONE)
    if twice:
        b.add(u, b.cba(v, co, k, act=W.ACT_NONE))
    return W.Workload("ring_tiles", n, (32, h, w), [t], [b], "bf16", lr=0.05)


def _classes(wl, op):
    d = parity.make_distiller(wl, wl.batch, "bf16")
    d.teacher_relay(torch.from_numpy(W.make_input(wl)).cuda())
    d.set_profile(True)
    d.student_step(1, wl.lr)
    return [p["name"] for p in d.get_profile() if p["op"] == op]


@pytest.mark.parametrize("shape,fwd,dgrad,accum", RINGS)
def test_every_tile_and_depth_of_the_ring(shape, fwd, dgrad, accum):
    wl = _layer(*shape, accum is not None)
    # (op 1 and, of two readers, op 2, whose backward pass comes first)
    first, last = _classes(wl, 2 if accum else 1), _classes(wl, 1)
    for kind, want, names in (("igemm_fwd_", fwd, last), ("igemm_dgrad_", dgrad, first), ("igemm_dgrad_", accum, last)):
        assert want is None or kind + want in names, (kind + want, names)
    worst = local_parity.run_and_check(wl, wl.batch)
    print(", ".join(f"{key} {e:.1e}" for key, e in sorted(worst.items())), flush=True)


# (batch, h, w, k, stride): reductions in one piece and columns of up to 2048 rows, whose batch norms add in one order at every channel count
SAME = [(1, 9, 7, 1, 1), (5, 9, 7, 3, 1), (10, 14, 14, 3, 1), (6, 13, 13, 3, 2), (7, 9, 9, 2, 1), (9, 2, 2, 3, 1), (41, 7, 7, 1, 1), (16, 11, 11, 3, 1)]


@pytest.mark.parametrize("wide", [64, 96])
@pytest.mark.parametrize("n,h,w,k,s", SAME)
def test_same_bits_as_staging_through_registers(n, h, w, k, s, wide):
    """48 channels between the layers, no multiple of the K step, against the same network with zeros for the channels from 48 on: 16 channels
    of a tap are one matrix instruction on either side, in the same order, and one of zeros adds nothing."""
    def run(mid):
        t, b = W.Block(), W.Block()
        t.cba(0, 64, k, s)
        b.cba(b.cba(b.cba(0, mid, 1), mid, k, s), 64, 1)
        wl = W.Workload("ring_bits", n, (32, h, w), [t], [b], "bf16", lr=0.05)
        d = pbd.Distiller(wl)
        d.bind("cuda:0")
        for net, blk, j, slot, arr in W.iter_params(W.Workload("ring_bits", n, (32, h, w), [t], [_block(48, k, s)], "bf16", lr=0.05)):
            if net == W.NET_STUDENT:
                full = np.full(W.param_shapes(wl, net, blk)[(j, slot)], 1.0 if slot in (W.P_GAMMA, W.P_RVAR) else 0.0, dtype=np.float32)
                full[tuple(slice(0, e) for e in arr.shape)] = arr
                arr = full
            d.load_param(net, blk, j, slot, arr)
        d.teacher_relay(torch.from_numpy(W.make_input(wl)).cuda())
        d.set_profile(True)
        d.student_step(1, wl.lr)
        d.sync()
        names = [p["name"] for p in d.get_profile() if p["op"] == 1 and p["name"].startswith("igemm_")]
        assert len(names) == 2 and all(("r3_" in x or "r2_" in x) == (mid != 48) for x in names), names
        got = {"loss": d.losses.cpu().numpy()}
        for j in range(3):
            got[f"conv{j}"], got[f"value{j}"], got[f"grad{j}"] = d.read_conv_out(0, j), d.read_value(0, j + 1), d.read_grad_value(0, j + 1)
            if j < 2:
                for what in ("conv", "value", "grad"):
                    assert not got[f"{what}{j}"][:, 48:].any()
                    got[f"{what}{j}"] = got[f"{what}{j}"][:, :48]
        return got
    ref, got = run(48), run(wide)
    for name in ref:
        np.testing.assert_array_equal(got[name], ref[name], err_msg=name)


def _block(mid, k, s):
    b = W.Block()
    b.cba(b.cba(b.cba(0, mid, 1), mid, k, s), 64, 1)
    return b
