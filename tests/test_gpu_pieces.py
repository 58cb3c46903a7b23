"""A step goes out as one graph with its branches inside or, where its launches are short (in_pieces), as a graph of each block on
several streams.  VGG-16 on both sides of that rule: whole steps and pipelined steps in turn, nothing waited for between the calls but eager
work of the caller on its own stream, twice on one workspace binding and once more on another, leave the bits that the launches
leave when they are sent one by one."""
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
        for _ in range(2):                                # (a new binding chooses its streams anew)
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
