"""Batch norms whose elementwise passes add the partial sums themselves (bn_apply_sums_kernel, bn_bwd_apply_sums_kernel): column lengths on either
side of the rule's lines (2048 rows, 3500 and 4096 for narrow ones, 4096 for the adds that ride in the passes, 8 MB), one to many slabs of unequal width, sums from the convolution's
store and from a pass of their own, a residual add in both passes, a block's loss.  Every operation against the plain fp64 oracle primitives on the
tensors that the library read, at the bounds of local_parity.py; the profile classes say which kernels ran."""
import numpy as np
import pytest
import torch

import local_parity
import parity
from paper_2301_12443_amd import workloads as W

pytestmark = pytest.mark.gpu

# (batch, h, w, channels)
CASES = [
    (1, 32, 64, 24),             # 2048 rows: the whole-column kernels
    (3, 1, 683, 8),              # 2049 narrow rows: again
    (1, 1, 3500, 24),            # the last of 48 and 96 bytes
    (1, 1, 3501, 32),            # the first of 64; 128
    (3, 1, 683, 64),             # 2049 rows
    (3, 1, 1367, 8),             # 4101 rows, one vector of channels
    (5, 19, 23, 72),             # nine vectors: slabs of five and four
    (64, 8, 8, 136),             # 4096 rows
    (17, 13, 19, 520),           # 4199 rows, nine slabs
    (16, 31, 31, 40),            # 76 chunks; 241 row tiles of the store
    (7, 33, 35, 48),             # 8085 rows: 127 row tiles
    (16, 33, 33, 64),            # 137: the separate passes again
    (9, 31, 33, 456),            # 8.4 MB: again
]


@pytest.mark.parametrize("precision", ["bf16", "f32"])
@pytest.mark.parametrize("n,h,w,c", CASES)
def test_elementwise_passes_that_add_the_sums(n, h, w, c, precision):
    t, b = W.Block(), W.Block()
    t.cba(0, c, 1, act=W.ACT_NONE)
    v = b.cba(0, c, 1, act=W.ACT_RELU)
    u = b.cba(v, c, 3, groups=c, act=W.ACT_RELU6)
    u = b.cba(u, c, 1, act=W.ACT_NONE)
    b.add(v, u, act=W.ACT_RELU)
    wl = W.Workload("bn_sums", n, (16, h, w), [t], [b], precision, lr=0.05)
    worst = local_parity.run_and_check(wl, n, precision=precision, overrides={W.P_BETA: 3.0} if precision == "f32" else None)
    print(", ".join(f"{key} {e:.1e}" for key, e in sorted(worst.items())), flush=True)
    d = parity.make_distiller(wl, n, precision)
    d.teacher_relay(torch.from_numpy(W.make_input(wl, batch=n)).cuda())
    d.set_profile(True)
    d.student_step(1, wl.lr)
    names = {p["name"] for p in d.get_profile()}
    m = n * h * w
    slabs = (c // 8 + 7) // 8
    rows = 256 // -(-(c // 8) // slabs) * 4                        # a chunk: four rows a thread, a slab's vectors side by side
    small = m * c * (2 if precision == "bf16" else 4) <= 8 << 20 and -(-m // rows) <= 128
    row = c * (2 if precision == "bf16" else 4)
    columns = m > (2048 if row >= 128 else 3500 if row >= 64 else 4096)
    assert ("bn_bwd_apply_sums" in names) == (small and columns), names
    few = precision == "f32" or -(-m // 64) <= 128                # (bfloat16: as many partial sums as the convolution's store has row tiles)
    assert (not names.isdisjoint({"bn_apply_sums", "bn_apply_sums_add"})) == (small and few and m > 4096), names


@pytest.mark.parametrize("n,h,w,c", [(7, 33, 35, 48), (16, 31, 31, 40), (64, 16, 16, 64)])
def test_float32_means_round_once_a_chunk(n, h, w, c):
    """The mean's distance from its 64-bit value over the float32 differences from the pivot that the library adds, in standard deviations, 2-norm
    over channels and seeds, against what the roundings on its way give: three additions in a thread, one at the end of a chunk, one of the
    result, each up to half a unit in the last place (2^-24 of the value, over sqrt 3 as a 2-norm; less above a power of two).  Row lanes added in float, in
    order, are beyond it (48 channels: 1.5e-8)."""
    unit = 2.0 ** -24 / np.sqrt(3.0)
    errors, bounds = [], []
    for seed in range(6):
        t, b = W.Block(), W.Block()
        t.cba(0, c, 1, act=W.ACT_NONE)
        b.cba(0, c, 1, act=W.ACT_NONE)
        wl = W.Workload("bn_sums", n, (16, h, w), [t], [b], "f32", lr=0.05)
        wl.seed = seed
        d = parity.make_distiller(wl, n, "f32")
        d.teacher_relay(torch.from_numpy(W.make_input(wl, batch=n)).cuda())
        d.student_step(1, wl.lr)
        y = d.read_conv_out(0, 0).transpose(0, 2, 3, 1).reshape(-1, c)
        term = (y - y[0]).astype(np.float64)               # (float32 differences)
        m, std = len(y), y.astype(np.float64).std(0)
        mean = y[0].astype(np.float64) + term.mean(0)
        errors.append((d.read_batch_stats(0, 0)[0] - mean) / std)
        vectors = c // 8
        lanes = 256 // -(-vectors // ((vectors + 7) // 8))
        term = np.concatenate([term, np.zeros((-m % (4 * lanes), c))]).reshape(-1, 4, lanes, c)
        roundings = [np.cumsum(term, axis=1)[:, 1:].reshape(-1, c), term.sum((1, 2))]
        bounds.append((sum(((unit * r) ** 2).sum(0) for r in roundings) / m ** 2 + (unit * mean) ** 2) / std ** 2)
    error, bound = np.sqrt(np.mean(np.square(errors))), np.sqrt(np.mean(bounds))
    print(f"{error:.2e} of {bound:.2e}", flush=True)
    assert error < bound


@pytest.mark.parametrize("n,h,w,c", [(7, 33, 35, 48), (16, 31, 31, 40), (64, 16, 16, 64)])
def test_bfloat16_losses_round_once_a_chunk(n, h, w, c):
    """The loss that rides in the reduction, relative to 64 bits on the tensors that the library read, 2-norm over 24 seeds: the result's rounding (its last
    place, over sqrt 12) and one of each chunk's sum; a fifth more for what 24 draws of a rounding may be above their mean (two standard
    deviations).  Rows and threads added in float are beyond it (40 channels: 4.5e-8)."""
    errors, bounds = [], []
    for seed in range(24):
        t, b = W.Block(), W.Block()
        t.cba(0, c, 1, act=W.ACT_NONE)
        v = b.cba(0, c, 1, act=W.ACT_RELU)
        b.add(v, b.cba(v, c, 1, act=W.ACT_NONE), act=W.ACT_RELU)
        wl = W.Workload("bn_sums", n, (16, h, w), [t], [b], "bf16", lr=0.05)
        wl.seed = seed
        d = parity.make_distiller(wl, n, "bf16")
        d.teacher_relay(torch.from_numpy(W.make_input(wl, batch=n)).cuda())
        d.student_step(1, wl.lr)
        d.sync()
        s, a = d.read_value(0, 3).astype(np.float64), d.read_act(1).astype(np.float64)
        loss = np.mean((s - a) ** 2)
        chunks = -(-n * h * w // (256 // (c // 8) * 4))
        errors.append(d.losses[0].item() / loss - 1.0)
        bounds.append((np.spacing(np.float32(loss)) / loss) ** 2 / 12 + 2.0 ** -48 / 3 / chunks)
    error, bound = np.sqrt(np.mean(np.square(errors))), 1.2 * np.sqrt(np.mean(bounds))
    print(f"{error:.2e} of {bound:.2e}", flush=True)
    assert error < bound
