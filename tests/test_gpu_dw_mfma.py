"""Depthwise convolutions on the matrix cores (dw_mfma_kernel, dw_wgrad_mfma_kernel, dw_wgrad_s2_mfma_kernel) at the edges
of their tiles of 16 x 16 or 8 x 16 pixels x 32 channels: every operation of a one-block step, and the teacher's folded form, against the plain fp64 oracle
primitives on the tensors that the library read (local_parity.py).  Its bounds: one bfloat16 rounding of a result (2^-9 of
it, 2e-2 of the largest allowed) forward and backward-data; the weight gradient is a float32 sum of products of bfloat16 numbers
(exact), held to TOL_DW - a wrong tap, shift or mask is off by the size of the result."""
import numpy as np
import pytest
import torch

import local_parity
import parity
from paper_2301_12443_amd import workloads as W

pytestmark = pytest.mark.gpu

# A weight gradient sums n products in chains of at most d = 400 additions (176 of a tile, the tiles of a workgroup, a lane's share
# of the workgroups), so it is off by at most d 2^-24 of the sum of the products' magnitudes.  With random signs that sum is
# at most 0.4 sqrt(n) times the largest of a layer's components (mean magnitude of a product 0.64, the largest of some hundred
# sums 2 sqrt(n) and more): 400 x 6e-8 x 0.4 x sqrt(n), 3e-3 at the 3e5 pixels of the largest layer here.  A lost or doubled
# part of 1 % of the pixels shows as sqrt(0.01) = 10 %, of 0.01 % as 1 %.
TOL_DW = 3e-3


def _tiles_per_workgroup(n, h, w, c, blocks, tile_h=16):
    """How many tiles one workgroup of a launch of at most `blocks` takes (2048 forward and backward-data, 768 weight gradient, 512
    weight gradient at stride 2)."""
    tiles, chunks = n * -(-h // tile_h) * -(-w // 16), max(1, blocks // -(-c // 32))
    return -(-tiles // chunks)


# (batch, h, w, channels, k, stride)
SHAPES = [
    (1, 8, 12, 8, 3, 1),         # the smallest image, one vector of channels
    (3, 16, 16, 40, 5, 1),       # exactly one tile, a channel group and a quarter
    (2, 17, 33, 72, 7, 1),       # one row and one column into the next tiles
    (1, 15, 31, 32, 3, 1),       # one short of a tile both ways
    (2, 14, 14, 144, 5, 1),      # the late layers: one ragged tile
    (1, 49, 13, 24, 7, 1),       # three tiles and a row
    (40, 32, 20, 96, 7, 1),      # three groups, an empty right half
    (260, 33, 37, 8, 3, 1),      # several tiles per workgroup, forward and backward, ragged both ways
    (260, 33, 37, 8, 5, 1),
    (260, 33, 37, 8, 7, 1),
    (3, 9, 8, 64, 3, 1),         # 8 wide: only the weight gradient takes the matrix cores
    (2, 31, 47, 16, 5, 1),       # half a channel group
    (5, 4, 5, 40, 5, 1),      # a corner of a tile
    (3, 16, 32, 40, 3, 2),    # stride 2 (8 x 16 tiles of the output): exactly one tile of an even image
    (2, 17, 33, 72, 5, 2),    # one output row and column into the next tiles, odd image
    (2, 31, 30, 24, 7, 2),
    (60, 33, 63, 96, 7, 2),   # several tiles per workgroup
    (4, 7, 7, 32, 5, 2),
    (2, 2, 3, 16, 3, 2),
]


@pytest.mark.parametrize("n,h,w,c,k,stride", SHAPES)
def test_every_operation_of_a_small_block(n, h, w, c, k, stride):
    t, b = W.Block(), W.Block()
    v = t.cba(0, c, 1, act=W.ACT_RELU6)
    v = t.cba(v, c, k, stride, groups=c, act=W.ACT_RELU6)
    t.cba(v, 16, 1, act=W.ACT_NONE)
    v = b.cba(0, c, 1, act=W.ACT_RELU6)
    # two readers of v: the second backward-data launch adds onto the first one's result
    d1 = b.cba(v, c, k, stride, groups=c, act=W.ACT_RELU6)
    d2 = b.cba(v, c, 3, stride, groups=c, act=W.ACT_NONE)
    b.cba(b.add(d1, d2), 16, 1, act=W.ACT_NONE)
    if n == 260:
        assert _tiles_per_workgroup(n, h, w, c, 2048) == 2 and _tiles_per_workgroup(n, h, w, c, 768) == 4
    if n == 60:
        assert _tiles_per_workgroup(n, (h + 1) // 2, (w + 1) // 2, c, 512, 8) == 3
    wl = W.Workload("dw_mfma", n, (8, h, w), [t], [b], "bf16", lr=0.05)
    worst = local_parity.run_and_check(wl, n, tol_dw=TOL_DW)
    print(", ".join(f"{key} {e:.1e}" for key, e in sorted(worst.items())), flush=True)


# (batch, h, w, channels, k, activation): more than 4096 pixels, so the layer in front leaves its normalisation to the
# depthwise layer, its only reader
FOLDED = [
    (5, 33, 31, 40, 3, W.ACT_RELU6),
    (6, 29, 27, 72, 5, W.ACT_RELU),
    (17, 17, 16, 24, 7, W.ACT_RELU6),
    (100, 7, 7, 48, 5, W.ACT_RELU6),
    (250, 35, 40, 24, 3, W.ACT_RELU),      # several tiles per workgroup, ragged, the last ones' right half empty
    (250, 35, 40, 24, 5, W.ACT_RELU6),
    (250, 35, 40, 24, 7, W.ACT_RELU6),
]


@pytest.mark.parametrize("n,h,w,c,k,act", FOLDED)
def test_normalisation_in_the_staging(n, h, w, c, k, act):
    t, b = W.Block(), W.Block()
    t.cba(0, 16, 1, act=W.ACT_NONE)
    v = b.cba(0, c, 1, act=act)
    v = b.cba(v, c, k, groups=c, act=W.ACT_RELU6)
    b.cba(v, 16, 1, act=W.ACT_NONE)
    if n == 250:
        assert _tiles_per_workgroup(n, h, w, c, 2048) == 2 and _tiles_per_workgroup(n, h, w, c, 768) == 3
    wl = W.Workload("dw_folded", n, (8, h, w), [t], [b], "bf16", lr=0.05)
    worst = local_parity.run_and_check(wl, n, tol_dw=TOL_DW)     # (reads the value between the two layers: formed on request, after the update)
    print(", ".join(f"{key} {e:.1e}" for key, e in sorted(worst.items())), flush=True)


# (batch, h, w, channels, k, activation in front, activation behind): the backward pass of such a layer in one kernel
BACKWARD = [
    (17, 16, 16, 8, 5, W.ACT_RELU, W.ACT_NONE),        # exactly one tile, one vector of channels
    (30, 14, 14, 40, 7, W.ACT_RELU6, W.ACT_RELU6),     # one ragged tile, a channel group and a quarter
    (5, 33, 31, 72, 3, W.ACT_RELU6, W.ACT_RELU),       # one row into the next tiles, one column short of them
    (3, 49, 37, 24, 7, W.ACT_RELU, W.ACT_NONE),
    (70, 8, 12, 136, 3, W.ACT_RELU, W.ACT_RELU6),
    (90, 50, 20, 8, 5, W.ACT_RELU6, W.ACT_RELU6),      # several tiles a workgroup in neither round
    (290, 35, 40, 16, 7, W.ACT_RELU6, W.ACT_RELU),     # several in both, the last ones' right half empty
]


@pytest.mark.parametrize("n,h,w,c,k,front,behind", BACKWARD)
def test_backward_in_one_kernel(n, h, w, c, k, front, behind):
    """Every operation against the oracle; and the architecture round, where the kernel leaves the filter alone, against the weight
    round: the same gradients up to the last bit of a stored bfloat16 number (the sums over the batch are grouped differently)."""
    t, b = W.Block(), W.Block()
    t.cba(0, 16, 1, act=W.ACT_NONE)
    v = b.mix([b.cba(0, 16, 1, act=W.ACT_NONE), b.cba(0, 16, 1, act=W.ACT_NONE)], [0.5, 0.5])
    v = b.cba(v, c, 1, act=front)
    v = b.cba(v, c, k, groups=c, act=behind)
    b.cba(v, 16, 1, act=W.ACT_NONE)
    wl = W.Workload("dw_backward", n, (8, h, w), [t], [b], "bf16", lr=0.05)
    worst = local_parity.run_and_check(wl, n, tol_dw=TOL_DW)
    print(", ".join(f"{key} {e:.1e}" for key, e in sorted(worst.items())), flush=True)
    grads = []
    for arch in (False, True):
        d = parity.make_distiller(wl, n, "bf16")
        d.teacher_relay(torch.from_numpy(W.make_input(wl, batch=n)).cuda())
        d.set_profile(True)
        (d.arch_step if arch else d.student_step)(1, wl.lr)
        names = {p["name"] for p in d.get_profile()}
        assert f"dw_{'dgrad' if arch else 'wgrad'}_mfma_bn_k{k}" in names, names
        d.set_profile(False)
        grads.append([d.read_grad_value(0, i) for i in (3, 4, 5)])       # of the mix, the layer in front and the depthwise one
    for x, y in zip(*grads):
        assert np.max(np.abs(x - y)) < 2.0 ** -7 * np.max(np.abs(x))


@pytest.mark.parametrize("folded", [False, True])
@pytest.mark.parametrize("k", [3, 5, 7])
def test_statistics_of_channels_far_from_zero(k, folded):
    """Batch statistics from the forward kernel where a workgroup begins with a tile whose right half is empty (40 columns:
    tiles of 16, 16 and 8; 17 tiles a workgroup).  Every channel is a checkerboard of two numbers up to 500 deviations from
    zero and the filter is its middle tap, so about any pixel of the image all sums are small whole numbers, exact in float32.
    About zero instead, a lane's 352 squares need more than its 24 bits, and the lost ones are a quarter of the variance and more."""
    n, h, w = 11000, 16, 40
    top = np.array([251, 241, 231, 221, 201, 191, 181, 171], dtype=np.float32)
    c = top.size
    assert _tiles_per_workgroup(n, h, w, c, 2048) == 17
    t, b = W.Block(), W.Block()
    t.cba(0, 16, 1, act=W.ACT_NONE)
    v = b.cba(0, c, 1, act=W.ACT_RELU) if folded else 0        # (a rectified value is normalised in the staging: top - 1 +- 1)
    v = b.cba(v, c, k, groups=c, act=W.ACT_NONE)
    b.cba(v, 16, 1, act=W.ACT_NONE)
    op = 1 if folded else 0
    wl = W.Workload("dw_far", n, (c, h, w), [t], [b], "bf16", lr=0.05)
    d = parity.make_distiller(wl, n, "bf16")
    middle = np.zeros((c, 1, k, k), dtype=np.float32)
    middle[:, :, k // 2, k // 2] = 1.0
    d.load_param(W.NET_STUDENT, 0, op, W.P_WEIGHT, middle)
    if folded:
        d.load_param(W.NET_STUDENT, 0, 0, W.P_WEIGHT, np.eye(c, dtype=np.float32).reshape(c, c, 1, 1))
        d.load_param(W.NET_STUDENT, 0, 0, W.P_BETA, top - 1)
    board = np.indices((h, w)).sum(axis=0) % 2
    x = torch.from_numpy(top[:, None, None] - board.astype(np.float32)).cuda().expand(n, c, h, w).contiguous()
    torch.cuda.synchronize()                                   # (the library works on a stream of its own)
    d.teacher_relay(x)
    d.student_step(1, wl.lr)
    d.sync()
    mean, invstd = d.read_batch_stats(0, op)
    print("variance + 1e-5:", invstd.astype(np.float64) ** -2, flush=True)
    np.testing.assert_array_equal(mean, top - 1 if folded else top - 0.5)
    np.testing.assert_allclose(invstd, ((1.0 if folded else 0.25) + 1e-5) ** -0.5, rtol=2.0 ** -23)


def test_a_second_reader_keeps_the_matrix_cores():
    """Backward-data that adds to a gradient already there runs on the same kernel as the first one."""
    t, b = W.Block(), W.Block()
    t.cba(0, 16, 1, act=W.ACT_NONE)
    v = b.cba(0, 40, 1, act=W.ACT_NONE)
    outs = [b.cba(v, 40, k, groups=40, act=W.ACT_NONE) for k in (3, 5, 7, 3)]
    b.cba(b.add(b.add(outs[0], outs[1]), b.add(outs[2], outs[3])), 16, 1, act=W.ACT_NONE)
    wl = W.Workload("dw_readers", 3, (8, 17, 21), [t], [b], "bf16", lr=0.05)
    d = parity.make_distiller(wl, 3, "bf16")
    d.teacher_relay(torch.from_numpy(W.make_input(wl, batch=3)).cuda())
    d.sync()
    d.set_profile(True)
    d.student_step(1, wl.lr)
    names = sorted(p["name"] for p in d.get_profile() if p["name"].startswith("dw_dgrad"))
    assert names == ["dw_dgrad_mfma_acc_k3", "dw_dgrad_mfma_acc_k5", "dw_dgrad_mfma_acc_k7", "dw_dgrad_mfma_k3"], names
    local_parity.run_and_check(wl, 3, tol_dw=TOL_DW)


@pytest.mark.parametrize("n,h,w,c", [(57, 97, 101, 64),        # ragged tiles of 8 x 16, one group of 64 channels
                                     (68, 56, 72, 128)])       # whole ones, two groups
def test_three_by_three_on_tensors_beyond_the_caches(n, h, w, c):
    """From 64 MiB on, whole 64-channel groups: forward without statistics (teacher) and backward-data, storing and adding,
    run on the tile kernel."""
    assert n * h * w * c * 2 >= 64 << 20
    t, b = W.Block(), W.Block()
    v = t.cba(0, c, 1, act=W.ACT_RELU6)
    v = t.cba(v, c, 3, groups=c, act=W.ACT_RELU6)
    t.cba(v, 8, 1, act=W.ACT_NONE)
    v = b.cba(0, c, 1, act=W.ACT_RELU6)
    d1 = b.cba(v, c, 3, groups=c, act=W.ACT_RELU6)
    d2 = b.cba(v, c, 3, groups=c, act=W.ACT_NONE)
    b.cba(b.add(d1, d2), 8, 1, act=W.ACT_NONE)
    wl = W.Workload("dw_large", n, (8, h, w), [t], [b], "bf16", lr=0.05)
    d = parity.make_distiller(wl, n, "bf16")
    d.set_profile(True)
    d.teacher_relay(torch.from_numpy(W.make_input(wl, batch=n)).cuda())
    d.student_step(1, wl.lr)
    d.sync()
    names = [p["name"] for p in d.get_profile() if p["name"].startswith(("dw_fwd", "dw_dgrad"))]
    assert names == ["dw_fwd_tile_k3", "dw_fwd_mfma_k3", "dw_fwd_mfma_k3", "dw_dgrad_tile_k3", "dw_dgrad_tile_k3"], names
    err = local_parity.teacher_block_error(d, wl, 0, (0, n // 2 + 1, n - 1))
    assert err < local_parity.TOL_BF16, err
    local_parity.run_and_check(wl, n, {0: ({1}, {1})})         # one depthwise forward, and the value that both read


@pytest.mark.parametrize("k,stride", [(3, 1), (5, 1), (7, 1), (5, 2)])
def test_many_channel_groups_divide_the_workgroups(k, stride):
    """Thirty groups of channels, ragged tiles, several tiles a workgroup: one layer, forward and backward."""
    n, h, w, c = 60, 17, 19, 960
    t, b = W.Block(), W.Block()
    t.cba(0, 16, 1, act=W.ACT_NONE)
    v = b.cba(0, c, 1, act=W.ACT_RELU6)
    v = b.cba(v, c, k, stride, groups=c, act=W.ACT_RELU6)
    b.cba(v, 16, 1, act=W.ACT_NONE)
    if stride == 2:
        t.cba(1, 16, 3, 2, act=W.ACT_NONE)
    wl = W.Workload("dw_groups", n, (8, h, w), [t], [b], "bf16", lr=0.05)
    local_parity.run_and_check(wl, n, {0: ({1}, {1, 2})}, tol_dw=TOL_DW)


# (batch, h, w, channels, k) where the forward, the folded and the backward-weight kernel part ways: small images, few or many tiles
@pytest.mark.parametrize("n,h,w,c,k,fwd,wgrad", [
    (128, 4, 4, 960, 5, "slide", "wgrad"),             # 3840 tiles x groups, 1/16 of them in the image
    (128, 4, 4, 384, 5, "mfma", "mfma"),               # 1536
    (128, 5, 5, 960, 7, "slide", "wgrad"),
    (128, 5, 6, 960, 7, "slide", "mfma"),
    (100, 7, 8, 384, 7, "slide", "mfma"),              # more than 4096 pixels, and yet the layer in front is not folded
    (33, 7, 8, 384, 7, "mfma", "mfma"),
    (9, 2, 2, 40, 5, "mfma", "wgrad"),
    (1100, 2, 2, 32, 5, "mfma", "wgrad"),              # more than 4096 pixels on the matrix cores, weight gradient not: not folded
    (128, 6, 6, 960, 5, "mfma_bn", "mfma_bn"),
    (128, 8, 8, 640, 3, "slide", "wgrad"),
    (33, 8, 8, 384, 3, "slide", "mfma"),
])
def test_small_images(n, h, w, c, k, fwd, wgrad):
    t, b = W.Block(), W.Block()
    t.cba(0, 16, 1, act=W.ACT_NONE)
    v = b.cba(0, c, 1, act=W.ACT_RELU6)
    v = b.cba(v, c, k, groups=c, act=W.ACT_RELU6)
    b.cba(v, 16, 1, act=W.ACT_NONE)
    wl = W.Workload("dw_small", n, (8, h, w), [t], [b], "bf16", lr=0.05)
    d = parity.make_distiller(wl, n, "bf16")
    d.teacher_relay(torch.from_numpy(W.make_input(wl, batch=n)).cuda())
    d.sync()
    d.set_profile(True)
    d.student_step(1, wl.lr)
    names = {p["name"] for p in d.get_profile()}
    assert f"dw_fwd_{fwd}_k{k}" in names, names
    assert (f"dw_wgrad_{wgrad}_k{k}" if wgrad != "wgrad" else f"dw_wgrad_k{3 if k == 3 else 7}") in names, names
    local_parity.run_and_check(wl, n, tol_dw=TOL_DW)


# (batch, h, w, channels, k, kernel class of the stride-2 weight gradient): both sides of its rule
@pytest.mark.parametrize("n,h,w,c,k,wgrad", [
    (5, 25, 25, 192, 3, "dw_wgrad_s2_mfma_k3"),
    (33, 49, 33, 40, 3, "dw_wgrad_k3"),
    (33, 49, 33, 40, 5, "dw_wgrad_s2_mfma_k5"),
    (128, 4, 4, 640, 5, "dw_wgrad_k7"),
    (128, 9, 11, 640, 7, "dw_wgrad_s2_mfma_k7"),
])
def test_stride_two_weight_gradient(n, h, w, c, k, wgrad):
    t, b = W.Block(), W.Block()
    t.cba(0, 16, 1, 2, act=W.ACT_NONE)
    v = b.cba(0, c, 1, act=W.ACT_RELU6)
    v = b.cba(v, c, k, 2, groups=c, act=W.ACT_RELU6)
    b.cba(v, 16, 1, act=W.ACT_NONE)
    wl = W.Workload("dw_s2", n, (8, h, w), [t], [b], "bf16", lr=0.05)
    d = parity.make_distiller(wl, n, "bf16")
    d.teacher_relay(torch.from_numpy(W.make_input(wl, batch=n)).cuda())
    d.sync()
    d.set_profile(True)
    d.student_step(1, wl.lr)
    names = {p["name"] for p in d.get_profile()}
    assert wgrad in names, names
    local_parity.run_and_check(wl, n, tol_dw=TOL_DW)


@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
@pytest.mark.parametrize("k", [3, 5, 7])
def test_a_non_finite_input_stays_within_the_filter(k, bad):
    """One infinity or NaN per image in what a frozen teacher's depthwise layer reads reaches the k x k outputs around it and
    no other, as in the plain kernels (force_direct): at tile edges, at the image's edge, inside."""
    n, h, w, c = 6, 18, 35, 40
    t, s = W.Block(), W.Block()
    t.cba(0, c, k, groups=c, act=W.ACT_NONE)
    s.cba(0, c, 1, act=W.ACT_NONE)
    wl = W.Workload("dw_inf", n, (c, h, w), [t], [s], "bf16", lr=0.05)
    x = W.make_input(wl, batch=n).copy()
    near = np.zeros((n, c, h, w), dtype=bool)
    for i, (p, q) in enumerate([(0, 0), (7, 7), (15, 16), (17, 34), (16, 31), (9, 20)]):
        x[i, 3 + i, p, q] = bad
        near[i, 3 + i, max(0, p - k // 2):p + k // 2 + 1, max(0, q - k // 2):q + k // 2 + 1] = True
    out = []
    for direct in (True, False):
        d = parity.make_distiller(wl, n, "bf16", force_direct=direct)
        d.teacher_relay(torch.from_numpy(x).cuda())
        d.sync()
        out.append(d.read_act(1))
    ref, got = out
    np.testing.assert_array_equal(~np.isfinite(ref), near)
    np.testing.assert_array_equal(got[near], ref[near])
    assert np.isfinite(got[~near]).all()
    assert local_parity._max_rel(got[~near], ref[~near]) < 2.0 ** -7       # (two roundings to bfloat16 of float32 sums)
