"""Batch norms whose elementwise passes add the partial sums themselves (bn_apply_sums_kernel, bn_bwd_apply_sums_kernel): column lengths on either
side of the rule's lines (2048 rows, 4096 for the adds that ride in the passes, 8 MB), one to many slabs of unequal width, sums from the convolution's
store and from a pass of their own, a residual add in both passes, a block's loss.  Every operation against the plain fp64 oracle primitives on the
tensors that the library read, at the bounds of local_parity.py; the profile classes say which kernels ran."""
import pytest
import torch

import local_parity
import parity
from paper_2301_12443_amd import workloads as W

pytestmark = pytest.mark.gpu

# (batch, h, w, channels)
CASES = [
    (1, 32, 64, 24),             # 2048 rows: the whole-column kernels
    (3, 1, 683, 8),              # 2049 rows, one vector of channels
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
    assert ("bn_bwd_apply_sums" in names) == (small and m > 2048), names
    few = precision == "f32" or -(-m // 64) <= 128                # (bfloat16: as many partial sums as the convolution's store has row tiles)
    assert (not names.isdisjoint({"bn_apply_sums", "bn_apply_sums_add"})) == (small and few and m > 4096), names
