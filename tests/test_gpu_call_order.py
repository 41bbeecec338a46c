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


@pytest.mark.parametrize("terms", [W.KPM, W.TERM_KERR | W.TERM_ANSATZ, W.KPM | W.TERM_ANSATZ])
@pytest.mark.parametrize("precision", [32, 64])
@pytest.mark.parametrize("n", [128, 768])
def test_power_trace_does_not_depend_on_the_cuts(n, precision, terms):
    """Ten steps in one call and in calls of 4, 1 and 5: the same field and
    the same power and peak of every step, bit for bit."""
    theta = np.array(W.THETA0) + W.random_theta(n, 0.2)
    inst = W.Instance(n=n, length=4e-3, dz=0.01, n_steps=10, medium=W.Medium(terms=terms),
                      w0=0.5e-3, power=400 * W.P_CR, sigma=0.2, seed=100 + n)
    u0 = W.initial_field(inst)
    out = []
    for cuts in ((10,), (4, 1, 5)):
        p = _prop([inst], precision)
        p.set_field(0, u0)
        p.set_theta(0, theta)
        power, peak = [], []
        for k in cuts:
            p.propagate(k)
            pw, pk = p.diag(0, k)
            power += list(pw)
            peak += list(pk)
        out.append((np.array(power), np.array(peak), p.field(0)))
        p.close()
    for a, b in zip(*out):
        assert np.array_equal(a, b), np.argwhere(a != b)[:8]


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
