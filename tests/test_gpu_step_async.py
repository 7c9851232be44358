"""hlb_step with the default options launches its steps and returns, however
often a call is repeated: it does not wait for the stream, takes no device
memory and leaves a capture alone that the caller has open on another stream."""
import numpy as np
import pytest

from paper_2202_11770_amd import geometry as G
from paper_2202_11770_amd import hlb

pytestmark = pytest.mark.gpu

CALLS = 8  # equal calls


def _sim(g):
    tables = [np.array([0.01 if io.kind == G.VELOCITY else 1.0]) for io in g.iolets]
    return hlb.Simulation.create(g, 0.8, tables=tables)


def test_repeated_calls_do_not_wait():
    import torch
    sim = _sim(G.tree(seed=2, generations=5, scale=0.5))  # 1.1e6 sites, some 60 us a step against 4 of a launch
    sim.step(1)
    hlb.hlb_sync(sim.ctx)
    held = hlb.hlb_info(sim.ctx)["device_bytes"]
    sim.step(2000)  # work ahead, longer than all calls together take to launch
    ahead = torch.cuda.Event()
    ahead.record()  # the null stream: behind the steps
    for k in range(CALLS):
        sim.step(60)
        assert not ahead.query(), f"call {k} waited for the steps ahead of it"
    assert hlb.hlb_info(sim.ctx)["device_bytes"] == held
    hlb.hlb_sync(sim.ctx)
    assert sim.t == 2001 + 60 * CALLS
    sim.close()


def test_a_capture_elsewhere_stays_valid():
    import torch
    g = G.cylinder()
    sim, ref = _sim(g), _sim(g)
    for _ in range(CALLS):
        ref.step(200)
    x = torch.ones(1 << 10, device="cuda")
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s, capture_error_mode="global"):
        x.mul_(2.0)
        for _ in range(CALLS):
            sim.step(200)
        x.add_(1.0)
    assert float(x[0]) == 1.0  # captured, not run
    for k in range(3):
        graph.replay()
        torch.cuda.synchronize()
        assert float(x[0]) == 2.0 ** (k + 2) - 1.0
    assert np.array_equal(hlb.hlb_get_state(sim.ctx), hlb.hlb_get_state(ref.ctx))
    sim.close()
    ref.close()
