"""The work that users of this framework have it do, as timed cases.

A case names a workload of `paper_2301_12443_amd.workloads`, its batch, image size and precision, and what a program
calls on it:

  step      `distill_step`: one whole step on one batch (relay, every student block, its update)
  pipeline  `pipeline_step` for `batches` batches and a `pipeline_flush`: a short run of the training loop, the
            teacher one batch ahead of the students
  nas       `distill_arch_step`, then `distill_step` on the same batch: one step of the architecture search
  relay     `teacher_relay` alone: the device that only evaluates the teacher, and the frozen network's inference
  block     `student_step` of one block against activations already relayed: a device that owns one block

A training program leaves the trained state in the workspace and copies it out at a checkpoint, not after every step;
`run` therefore hands it out as a mapping that reads a block's state through `read_tensor` when it is looked at.
"""
import numpy as np
import torch

from paper_2301_12443_amd import pbd, workloads as W

DEVICE = "cuda:0"
LR = 0.005                    # small enough that thousands of passes over the same few batches stay finite
LR_ALPHA = 0.005              # ... of the architecture parameters


def _case(name, net, batch, hw, precision, call, **more):
    case = {"net": net, "batch": batch, "hw": hw, "precision": precision, "call": call, **more}
    return {"name": name, **case} if name else case


def listed():
    return [
        # the smallest job there is: eight 32 x 32 images, float32; launches and their order are all of it
        _case("tiny_f32_step", "tiny_cnn", 8, 32, "f32", "step"),
        # CIFAR-sized distillation at its usual batch, as a training loop runs it
        _case("vgg_pipeline", "vgg16_dsconv", 256, 32, "bf16", "pipeline", batches=4),
        # a third of that batch, the share of one of three devices that split it
        _case("vgg_third_step", "vgg16_dsconv", 85, 32, "bf16", "step"),
        # the same networks in float32, for those who want no bfloat16 rounding
        _case("vgg_f32_step", "vgg16_dsconv", 64, 32, "f32", "step"),
        # ImageNet-sized inverted residuals (5 x 5 depthwise student), as a training loop runs it
        _case("mbv2_pipeline", "mbv2_mbconv_k5e4", 128, 224, "bf16", "pipeline", batches=4),
        # the same with an odd image and batch size: ragged tiles everywhere
        _case("mbv2_odd_step", "mbv2_mbconv_k5e4", 33, 193, "bf16", "step"),
        # architecture search: the weight round at the full batch
        _case("supernet_step", "mbv2_supernet", 64, 224, "bf16", "step"),
        # ... and a whole search step (both rounds) on a quarter of it
        _case("supernet_nas", "mbv2_supernet", 16, 224, "bf16", "nas"),
        # the largest job: ResNet-50 into a x1.5 wide student at batch 256, as a training loop runs it
        _case("resnet_pipeline", "resnet50_x1.5", 256, 224, "bf16", "pipeline", batches=3),
        # a quarter of that batch, one whole step
        _case("resnet_quarter_step", "resnet50_x1.5", 64, 224, "bf16", "step"),
        # the teacher alone
        _case("resnet_relay", "resnet50_x1.5", 256, 224, "bf16", "relay"),
        # one device of a split: the third block on a third of the batch
        _case("resnet_block3", "resnet50_x1.5", 85, 224, "bf16", "block", block=3),
    ]


# per workload: batch range, image sizes, and the calls with their share
_RANGES = {
    "tiny_cnn": ((1, 64), (32, 32), ("step", "step", "pipeline")),
    "vgg16_dsconv": ((16, 256), (32, 40), ("pipeline", "step", "relay", "block")),
    "mbv2_mbconv_k5e4": ((8, 128), (128, 224), ("pipeline", "step", "relay", "block")),
    "mbv2_supernet": ((4, 64), (128, 224), ("step", "nas", "block")),
    "resnet50_x1.5": ((16, 256), (160, 224), ("pipeline", "step", "relay", "block")),
}


def draw(rng):
    net = rng.choice(list(_RANGES))
    (lo, hi), (hw_lo, hw_hi), calls = _RANGES[net]
    precision = "f32" if net == "tiny_cnn" or (net == "vgg16_dsconv" and rng.random() < 0.3) else "bf16"
    if precision == "f32":
        hi = min(hi, 64)
    batch = min(hi, max(lo, round(lo * (hi / lo) ** rng.random())))
    case = _case(None, net, batch, rng.randint(hw_lo, hw_hi), precision, rng.choice(calls))
    if case["call"] == "pipeline":
        case["batches"] = rng.randint(2, 3)
    if case["call"] == "block":
        case["block"] = rng.randint(1, W.CONFIGS[net]().B)
    return case


def _workload(case, seed=0):
    make = W.CONFIGS[case["net"]]
    if case["net"] == "tiny_cnn":
        wl = make(case["batch"])
    else:
        wl = make(case["batch"], case["hw"], case["precision"])
    wl.seed = seed
    return wl


def _trained_blocks(case, wl):
    """The student blocks (from 0) that a pass trains."""
    if case["call"] == "relay":
        return []
    return [case["block"] - 1] if case["call"] == "block" else list(range(wl.B))


class _Trained(dict):
    """What a pass has trained, one flat float32 array per block and kind: "weights" (weights, gamma, beta),
    "statistics" (running mean and variance), "momentum" and, of a search, "alpha"."""

    _SLOTS = {"weights": (pbd.PBD_PARAM, W.P_WEIGHT, W.P_BETA), "statistics": (pbd.PBD_PARAM, W.P_RMEAN, W.P_RVAR),
              "momentum": (pbd.PBD_MOMENTUM, W.P_WEIGHT, W.P_BETA)}

    def __init__(self, d, params, kinds, alphas):
        super().__init__((f"block{b + 1}.{kind}", (b, kind)) for b in params for kind in kinds)
        self._d, self._params, self._alphas = d, params, alphas

    def __getitem__(self, key):
        b, kind = super().__getitem__(key)
        if kind == "alpha":
            return np.concatenate([self._d.read_alpha(b, j, n) for j, n in self._alphas[b]])
        code, first, last = self._SLOTS[kind]
        return np.concatenate([self._d.read_tensor(code, pbd.PBD_STUDENT, b, j, slot, shape).ravel()
                               for (j, slot), shape in self._params[b].items() if first <= slot <= last])


class _Borrowed:
    """A pbd_tensor view as torch takes foreign device memory (bfloat16 has no code of its own there); torch keeps
    it, and with it the owner of the memory, as long as the tensor lives."""

    def __init__(self, view, owner):
        self.owner = owner
        self.__cuda_array_interface__ = {"shape": (view.n, view.h, view.w, view.c_phys), "data": (view.ptr, False), "version": 2,
                                         "typestr": "<i2" if view.dtype == pbd.PBD_BF16 else "<f4"}


def _as_tensor(view, owner):
    t = torch.as_tensor(_Borrowed(view, owner), device=DEVICE)
    return t.view(torch.bfloat16) if view.dtype == pbd.PBD_BF16 else t


def prepare(case, seed):
    wl = _workload(case, seed)
    d = pbd.Distiller(wl)
    d.bind(DEVICE)
    trained = _trained_blocks(case, wl)
    for net, blocks in ((pbd.PBD_TEACHER, range(wl.B)), (pbd.PBD_STUDENT, trained)):
        for b in blocks:
            for (j, slot), shape in W.param_shapes(wl, net, b).items():
                d.load_param(net, b, j, slot, W.make_param(wl, net, b, j, slot, shape))
    g = torch.Generator(device=DEVICE).manual_seed(seed)
    xs = [torch.randn((wl.batch, *wl.in_shape), generator=g, device=DEVICE) for _ in range(case.get("batches", 1))]
    torch.cuda.synchronize()          # the library works on a stream of its own
    if case["call"] == "block":
        d.teacher_relay(xs[0])
        d.sync()
    out = {}
    if trained:
        # (behind many layers the momentum is no measure of a step: a value on the other side of a rectifier's kink
        # reroutes a gradient, and two correct orders of summation are 40 % apart in bfloat16 behind twelve of them)
        kinds = ["weights", "statistics"] + ["momentum"] * (case["net"] == "tiny_cnn") + ["alpha"] * (case["call"] == "nas")
        params = {b: W.param_shapes(wl, pbd.PBD_STUDENT, b) for b in trained}
        alphas = {b: [(j, len(op.inputs)) for j, op in enumerate(wl.student[b].ops) if op.type == W.OP_MIX] for b in trained}
        out = {"losses": d.losses[trained[0]:trained[-1] + 1], "trained": _Trained(d, params, kinds, alphas)}
    return {"case": case, "d": d, "xs": xs, "out": out}


def run(state):
    case, d, xs = state["case"], state["d"], state["xs"]
    call = case["call"]
    if call == "relay":
        return {f"A_{i}": _as_tensor(v, d) for i, v in enumerate(d.teacher_relay(xs[0]))}
    if call == "step":
        d.distill_step(xs[0], LR)
    elif call == "pipeline":
        for x in xs:
            d.pipeline_step(x, LR)
        d.pipeline_flush()
    elif call == "nas":
        d.distill_arch_step(xs[0], LR_ALPHA)
        d.distill_step(xs[0], LR)
    else:
        d.student_step(case["block"], LR)
    return state["out"]


def _block_work(block, in_shape, batch, rounds):
    """(forward flops, backward flops, elements of all op outputs) of a block; `rounds`: the backward passes taken,
    of "weights" and "alpha"."""
    shapes = W.block_shapes(block, in_shape)
    fwd = bwd = elems = 0
    above = [False] * len(shapes)     # a mix lies at or above the value: an architecture round needs its gradient
    for j, op in enumerate(block.ops):
        n = batch * int(np.prod(shapes[j + 1]))
        elems += n
        above[j + 1] = op.type == W.OP_MIX or any(above[v] for v in op.inputs)
        if op.type == W.OP_CBA:
            f = 2 * n * op.k * op.k * (shapes[op.inputs[0]][0] // op.groups)
            fwd += f
            if "weights" in rounds:   # the weights' gradient, and the input's unless that is the teacher's activation
                bwd += f * (2 if op.inputs[0] else 1)
            if "alpha" in rounds:
                bwd += f * above[op.inputs[0]]
    return fwd, bwd, elems


def work(case):
    """Each input read and each result written once: x, the parameters and the optimiser's state, the relayed A_i;
    and of every student layer's output, which has to wait for the backward pass, one write and one read of the
    value and of its gradient.  What lies between two layers of the teacher need not reach memory."""
    wl = _workload(case)
    acts = W.activation_shapes(wl)
    batch, es = wl.batch, 2 if case["precision"] == "bf16" else 4
    rounds = {"nas": ["weights", "alpha"], "relay": []}.get(case["call"], ["weights"])
    passes = case.get("batches", 1)
    n_bytes = flops = 0
    if case["call"] != "block":
        n_bytes += 4 * batch * int(np.prod(wl.in_shape))
        for b in range(wl.B):
            f, _, _ = _block_work(wl.teacher[b], acts[b], batch, [])
            flops += f * (2 if case["call"] == "nas" else 1)
            n_bytes += es * batch * int(np.prod(acts[b + 1]))
            n_bytes += sum(es * int(np.prod(s)) for s in W.param_shapes(wl, pbd.PBD_TEACHER, b).values())
    for b in _trained_blocks(case, wl):
        f, g, elems = _block_work(wl.student[b], acts[b], batch, rounds)
        flops += f * len(rounds) + g
        n_bytes += 4 * es * elems * len(rounds) + es * batch * int(np.prod(acts[b]) + np.prod(acts[b + 1]))
        n_bytes += sum(16 * int(np.prod(s)) for s in W.param_shapes(wl, pbd.PBD_STUDENT, b).values())
    return {"bytes": n_bytes * passes, "flops": flops * passes}


def tolerance(case):
    """About four times what the path was seen to differ by: the bfloat16 calls from the library's plain direct
    kernels (other orders of summation at the same precision), the float32 ones from the same steps in 64 bits."""
    if case["call"] == "relay":
        return {"rel": 0.03, "max": 0.36}
    if case["net"] == "tiny_cnn":
        return {"rel": 1e-4, "max": 5e-3}     # (a rectifier's kink within rounding moves the momentum)
    if case["precision"] == "f32":
        return {"rel": 1.2e-5, "max": 5.2e-4}
    return {"rel": 8e-3, "max": 0.11}
