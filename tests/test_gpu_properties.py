"""Properties that hold at any size, checked at the full BASELINE configurations in the launch
configuration the benchmark times (bf16, MFMA), plus the ABI's state and error handling on a GPU."""
import ctypes as C

import numpy as np
import pytest

import parity
from paper_2301_12443_amd import pbd, workloads as W

pytestmark = pytest.mark.gpu

FULL = ["vgg16_dsconv", "mbv2_mbconv_k5e4", "mbv2_supernet", "resnet50_x1.5"]


def _state(d, wl):
    out = []
    for b in range(wl.B):
        for (j, slot), shape in W.param_shapes(wl, W.NET_STUDENT, b).items():
            out.append(d.read_tensor(pbd.PBD_PARAM, 1, b, j, slot, shape).copy())
    return out


@pytest.mark.parametrize("name", FULL)
def test_full_size_step_is_deterministic_and_split_calls_agree(name):
    """pbd_distill_step == pbd_teacher_relay + pbd_student_step in any block order, bit for bit
    (Sec. IV-B: blocks are independent), and two runs give identical bits (ordered reductions)."""
    import torch
    wl = W.CONFIGS[name]()
    x = torch.from_numpy(W.make_input(wl)).cuda()
    a = parity.make_distiller(wl)
    a.distill_step(x, wl.lr); a.distill_step(x, wl.lr); a.sync()
    la = a.losses.cpu().numpy().copy()
    assert np.all(np.isfinite(la)) and np.all(la > 0)
    sa = _state(a, wl)
    del a
    torch.cuda.empty_cache()
    b = parity.make_distiller(wl)
    lb = np.zeros_like(la)
    for step in range(2):
        b.teacher_relay(x)
        for i in reversed(range(1, wl.B + 1)):
            b.student_step(i, wl.lr)
        b.sync()
        lb = b.losses.cpu().numpy().copy()
    np.testing.assert_array_equal(la, lb)
    for ta, tb in zip(sa, _state(b, wl)):
        np.testing.assert_array_equal(ta, tb)


def test_no_graph_option_gives_the_same_bits():
    """The captured graph replays exactly the launches that no_graph issues one by one."""
    import torch
    wl = W.CONFIGS["vgg16_dsconv"]()
    x = torch.from_numpy(W.make_input(wl)).cuda()
    out = []
    for no_graph in (False, True):
        d = pbd.Distiller(wl, no_graph=no_graph)
        d.bind("cuda:0"); d.load_params()
        for _ in range(3):
            d.distill_step(x, wl.lr)
        d.sync()
        assert d.uses_graph() == (not no_graph)
        out.append((d.losses.cpu().numpy().copy(), _state(d, wl)))
        del d
    np.testing.assert_array_equal(out[0][0], out[1][0])
    for ta, tb in zip(out[0][1], out[1][1]):
        np.testing.assert_array_equal(ta, tb)


def test_teacher_without_relaying_gives_the_same_step():
    """Sec. III vs Sec. IV-A: re-running T_1..T_i from the input before every block (the baseline's
    redundant teacher work) and relaying the activations are the same computation, bit for bit."""
    import torch
    wl = W.CONFIGS["vgg16_dsconv"]()
    x = torch.from_numpy(W.make_input(wl)).cuda()
    a = parity.make_distiller(wl)
    a.teacher_relay(x)
    for i in range(1, wl.B + 1):
        a.student_step(i, wl.lr)
    a.sync()
    b = parity.make_distiller(wl)
    for i in range(1, wl.B + 1):
        views = b.teacher_prefix(x, i)
        assert views[i].ptr and (i == wl.B or not views[i + 1].ptr)
        b.student_step(i, wl.lr)
    b.sync()
    np.testing.assert_array_equal(a.losses.cpu().numpy(), b.losses.cpu().numpy())
    for ta, tb in zip(_state(a, wl), _state(b, wl)):
        np.testing.assert_array_equal(ta, tb)
    # a block beyond the prefix has no valid target
    b.teacher_prefix(x, 1)
    with pytest.raises(RuntimeError):
        b.student_step(2, wl.lr)


@pytest.mark.parametrize("name", ["mbv2_mbconv_k5e4", "resnet50_x1.5"])
def test_full_size_teacher_relay_on_sampled_images(name):
    """The relayed activations at the full batch and image size of configs 3-5 (config 4 shares config 3's
    teacher), checked on sampled images: the frozen teacher uses its running statistics (Sec. II-A), so
    image n of every A_i depends on image n of A_{i-1} alone and the oracle can compute it at batch 1.
    Each block is compared with the PLAIN fp64 oracle's T_i applied to the library's own A_{i-1} at 2e-2
    (one block deep, the half-ulp rounding of the stored tensors in between stays far below the bound; over
    the whole 52-layer chain of MobileNetV2 it adds up to 1.8e-2 and more)."""
    import torch
    import local_parity
    wl = W.CONFIGS[name]()
    x = W.make_input(wl)
    d = parity.make_distiller(wl)
    d.distill_step(torch.from_numpy(x).cuda(), wl.lr)      # the launch configuration the benchmark times
    d.sync()
    assert d.uses_graph()
    images = (0, wl.batch // 2 + 1, wl.batch - 1)
    for b in range(wl.B):
        err = local_parity.teacher_block_error(d, wl, b, images)
        print(f"[{name}] T_{b + 1} on images {images}: {err:.2e}", flush=True)
        assert err < 2e-2, (b, err)


def test_relay_views_and_shared_input():
    """S_i reads the very buffer T_i read: the view of A_{i-1} handed out by the relay."""
    import torch
    wl = W.tiny_cnn()
    d = parity.make_distiller(wl)
    views = d.teacher_relay(torch.from_numpy(W.make_input(wl)).cuda())
    shapes = W.activation_shapes(wl)
    for i, v in enumerate(views):
        assert (v.n, v.c, v.h, v.w) == (wl.batch, *shapes[i]) and v.c_phys % 8 == 0 and v.ptr
    d.student_step(2, wl.lr)
    np.testing.assert_array_equal(d.read_value(1, 0), d.read_act(1))


def test_state_and_argument_errors_on_device():
    import torch
    wl = W.tiny_cnn()
    d = pbd.Distiller(wl)
    L = pbd.lib()
    assert L.pbd_sync(d.h) == -4                                   # not bound
    ws = torch.empty(d.workspace_bytes() + 512, dtype=torch.uint8, device="cuda")
    base = (ws.data_ptr() + 255) // 256 * 256
    assert L.pbd_bind(d.h, base, d.workspace_bytes() - 1, None) == -3
    assert L.pbd_bind(d.h, base + 8, d.workspace_bytes(), None) == -3
    assert L.pbd_bind(d.h, None, d.workspace_bytes(), None) == -3
    d.bind()
    loss = torch.zeros(1, device="cuda")
    v = pbd.pbd_tensor()
    assert L.pbd_student_step(d.h, 1, C.byref(v), C.byref(v), 0.1, loss.data_ptr()) == -4   # no relay yet
    views = d.teacher_relay(torch.from_numpy(W.make_input(wl)).cuda())
    assert L.pbd_student_step(d.h, 0, C.byref(views[0]), C.byref(views[1]), 0.1, loss.data_ptr()) == -1
    assert L.pbd_student_step(d.h, 5, C.byref(views[0]), C.byref(views[1]), 0.1, loss.data_ptr()) == -1
    assert L.pbd_student_step(d.h, 1, C.byref(views[1]), C.byref(views[1]), 0.1, loss.data_ptr()) == -2
    assert L.pbd_student_step(d.h, 1, C.byref(views[0]), C.byref(views[1]), float("nan"), loss.data_ptr()) == -1
    assert L.pbd_student_step(d.h, 1, C.byref(views[0]), C.byref(views[1]), 0.1, None) == -1
    assert L.pbd_teacher_relay(d.h, None, None) == -1
    buf = np.zeros(4, dtype=np.float32)
    fp = buf.ctypes.data_as(C.POINTER(C.c_float))
    assert L.pbd_load_param(d.h, 1, 0, 0, 0, fp, 4) == -2           # wrong element count
    assert L.pbd_load_param(d.h, 1, 9, 0, 0, fp, 4) == -1
    assert L.pbd_read_tensor(d.h, 1, 0, 0, 0, 0, fp, 4) == -1       # teacher has no gradients
    assert L.pbd_read_act(d.h, 9, fp, 4) == -1
    assert b"block" in L.pbd_last_error(d.h) or L.pbd_last_error(d.h)
    assert L.pbd_student_step(d.h, 1, C.byref(views[0]), C.byref(views[1]), 0.1, loss.data_ptr()) == 0
    d.sync()
    assert np.isfinite(loss.item())


@pytest.mark.parametrize("batch,bn", [(8, {"bn_small_fwd", "bn_small_bwd"}),
                                      (96, {"bn_stats", "bn_apply", "bn_bwd_reduce", "bn_bwd_apply",
                                            "bn_small_fwd", "bn_small_bwd"})])
def test_profile_records_every_launch(batch, bn):
    import torch
    wl = W.tiny_cnn()
    d = parity.make_distiller(wl, batch=batch, precision="bf16")
    x = torch.from_numpy(W.make_input(wl, batch=batch)).cuda()
    d.distill_step(x, wl.lr)
    d.set_profile(True); d.reset_profile()
    d.distill_step(x, wl.lr)
    prof = d.get_profile()
    names = {p["name"] for p in prof}
    assert {"cast_input", "mse_loss_grad", "sgd_momentum"} | bn <= names
    for prefix in ("igemm_fwd_", "igemm_dgrad_", "wgrad_"):
        assert any(n.startswith(prefix) for n in names), (prefix, names)
    assert any(n.startswith("igemm_fwd_") and n.endswith("_affine") for n in names)      # teacher: fused BN + ReLU
    assert all(p["ms"] > 0 for p in prof) and all(p["bytes"] > 0 for p in prof)


@pytest.mark.parametrize("call", ["student_step", "student_step_static", "distill_step"])
@pytest.mark.parametrize("precision", ["bf16", "f32"])
def test_a_value_that_nobody_reads_trains_nothing(precision, call):
    """Layers whose values lead nowhere get no gradient: their weights and momenta stay as they were, whatever the
    memory behind the parameters held when the workspace was bound."""
    import torch
    t, s = W.Block(), W.Block()
    t.cba(0, 24, 3)
    v = s.cba(0, 32, 1)
    dangling = [s.cba(v, 40, 3), s.cba(v, 32, 3, groups=32), s.cba(v, 32, 5, 2, groups=32)]
    dangling.append(s.cba(dangling[0], 48, 1))
    s.cba(v, 24, 3)
    wl = W.Workload("dangling", 8, (8, 20, 20), [t], [s], precision, lr=0.05)
    d = pbd.Distiller(wl)
    d.bind("cuda:0")
    d._ws.fill_(255)                                   # NaN in every type
    torch.cuda.synchronize()
    base = (d._ws.data_ptr() + 255) // 256 * 256
    assert pbd.lib().pbd_bind(d.h, base, d.workspace_bytes(), d._stream.cuda_stream) == 0
    d.load_params()
    x = torch.from_numpy(W.make_input(wl)).cuda()
    for _ in range(2):
        if call == "distill_step":
            d.distill_step(x, wl.lr)
        else:
            d.teacher_relay(x)
            getattr(d, call)(1, wl.lr)
    d.sync()
    assert np.isfinite(d.losses.cpu().numpy()).all()
    for (j, slot), shape in W.param_shapes(wl, W.NET_STUDENT, 0).items():
        if slot > W.P_BETA:
            continue
        got = d.read_tensor(pbd.PBD_PARAM, 1, 0, j, slot, shape)
        start = W.make_param(wl, W.NET_STUDENT, 0, j, slot, shape)
        moved = not np.array_equal(got, start)
        assert np.isfinite(got).all() and moved == (j + 1 not in dangling), (j, slot)
        if j + 1 in dangling:
            for kind in (pbd.PBD_GRAD, pbd.PBD_MOMENTUM):
                assert not d.read_tensor(kind, 1, 0, j, slot, shape).any(), (j, slot, kind)


@pytest.mark.parametrize("n,hw,classes", [
    # 51200 rows, 400 tiles of 128 columns or 200: the short reduction (576) keeps two narrow workgroups a unit, 1152 takes the wide one
    (200, 16, ["igemm_fwd_256x64x32_affine", "igemm_fwd_256x128x64_affine"]),
    # 37632 rows: 147 wide tiles would be too few for the 256-row kernel, 294 narrow ones are not
    (48, 28, ["igemm_fwd_256x64x32_affine", "igemm_fwd_256x64x32_affine"]),
])
def test_tiles_of_a_launch_that_does_not_fill_the_chip_twice(n, hw, classes):
    import torch

    import local_parity
    t, s = W.Block(), W.Block()
    v = t.cba(0, 128, 3); t.cba(v, 128, 3)
    s.cba(0, 128, 1)
    wl = W.Workload("one_round", n, (64, hw, hw), [t], [s], "bf16", lr=0.05)
    d = parity.make_distiller(wl, n, "bf16")
    d.set_profile(True)
    d.teacher_relay(torch.from_numpy(W.make_input(wl, batch=n)).cuda())
    d.sync()
    assert [p["name"] for p in d.get_profile() if p["name"].startswith("igemm_")] == classes
    err = local_parity.teacher_block_error(d, wl, 0, (0, n // 2 + 1, n - 1))
    assert err < 2e-2, err
