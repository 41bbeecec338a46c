"""What the calls of a context see of one another: parameters and later calls,
marches cut into several calls, beams set at different steps."""
import dataclasses

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def _prop(insts, precision, **kw):
    from paper_2306_15678_amd.march import Propagator, desc_of
    return Propagator([desc_of(i) for i in insts], precision=precision, **kw)


def test_captured_read_out_sees_later_parameters():
    """A caller's own graph of a read-out, taken right after a parameter
    change: its replays read the parameters that are set by then, and leave
    them as they are."""
    import torch
    inst = dataclasses.replace(W.config4_sparse(), n=128, sigma=0.02)
    u0 = W.initial_field(inst)
    first, second = (np.array(W.THETA0) + W.random_theta(k, 0.3) for k in (1, 2))
    stream = torch.cuda.Stream()
    p = _prop([inst], 32, stream=stream)
    p.set_field(0, u0)
    p.propagate(3)
    p.set_theta(0, first)           # the screen still pending takes it
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        out = p.intensity(0, device=True)
    want = {}
    for name, theta in (("first", first), ("second", second)):
        p.set_theta(0, theta)
        want[name] = p.intensity(0)
    assert not np.array_equal(want["first"], want["second"])
    for name, theta in (("second", second), ("first", first), ("second", second)):
        p.set_theta(0, theta)
        with torch.cuda.stream(stream):
            graph.replay()
        p.synchronize()
        assert np.array_equal(out.cpu().numpy(), want[name]), name
        assert np.array_equal(p.intensity(0), want[name]), name
    p.close()
