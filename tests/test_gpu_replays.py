"""Steps replayed from a graph: whole steps and pipelined steps in turn, nothing waited for between the calls but eager work of the caller
on its own stream, twice on one workspace binding and once more on another, leave the bits that the launches leave when they are
sent one by one.  Contexts that come and go, several at a time, leave nothing behind that the next ones trip over."""
import dataclasses

import numpy as np
import pytest

from paper_2301_12443_amd import pbd, workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [8, 40, 128])
def test_replays_leave_the_bits_of_single_launches(batch):
    import torch
    wl = dataclasses.replace(W.vgg16_dsconv(), batch=batch)
    xs = [torch.from_numpy(W.make_input(wl, step=s)).cuda() for s in range(3)]
    runs = []
    for no_graph in (True, False):
        d = pbd.Distiller(wl, no_graph=no_graph)
        got = []
        for _ in range(2):
            d.bind("cuda:0")
            d.load_params()
            torch.cuda.synchronize()
            for again in range(2):
                for x in xs:
                    d.distill_step(x, wl.lr)
                    xs[0].mul(1.0001).sum()
                for x in xs:
                    d.pipeline_step(x, wl.lr)
                d.pipeline_flush()
                d.distill_step(xs[1], wl.lr)
                d.sync()
                got.append(d.losses.cpu().numpy().copy())
                if not again:
                    d.set_pipeline_order(list(range(wl.B, -1, -1)))
        assert d.uses_graph() == (not no_graph)
        for b in range(wl.B):
            for (j, slot), shape in W.param_shapes(wl, W.NET_STUDENT, b).items():
                got.append(d.read_tensor(pbd.PBD_PARAM, 1, b, j, slot, shape))
        runs.append(got)
    assert len(runs[0]) == len(runs[1])
    for a, b in zip(*runs):
        assert np.array_equal(a, b)


def test_contexts_that_come_and_go():
    """Three contexts at a time take turns and are dropped, again and again, at the batches of short launches."""
    import torch
    losses = {}
    for again in range(2):
        for batch in (8, 16, 32, 48, 64):
            wl = W.vgg16_dsconv(batch)
            x = torch.from_numpy(W.make_input(wl)).cuda()
            contexts = []
            for _ in range(3):
                d = pbd.Distiller(wl)
                d.bind("cuda:0")
                d.load_params()
                contexts.append(d)
            torch.cuda.synchronize()
            for _ in range(4):
                for d in contexts:
                    d.distill_step(x, wl.lr)
            torch.cuda.synchronize()
            for d in contexts:
                assert d.uses_graph()
                got = d.losses.cpu().numpy()
                assert np.array_equal(got, losses.setdefault(batch, got.copy()))
            del contexts, d
