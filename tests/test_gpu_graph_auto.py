"""Repeated hlb_step calls that the library replays as graphs by itself: the
same sequence of calls on the context's own stream and on a stream of the
caller (plain launches), with eager work, table and option changes and state
resets between, every intermediate state bit for bit."""
import numpy as np
import pytest

from paper_2202_11770_amd import geometry as G
from paper_2202_11770_amd import hlb

pytestmark = pytest.mark.gpu


def _run(n, storage, scheme, stream):
    import torch
    g = G.cylinder()
    tables = [0.01 * (1 + 0.5 * np.sin(2 * np.pi * np.arange(37) / 37)) if io.kind == G.VELOCITY else
              1.0 + 0.001 * np.cos(2 * np.pi * np.arange(53) / 53) for io in g.iolets]
    sim = hlb.Simulation.create(g, 0.8, storage=storage, scheme=scheme, tables=tables)
    if stream is not None:
        hlb.hlb_set_stream(sim.ctx, stream.cuda_stream)
    k_in = [k for k, io in enumerate(g.iolets) if io.kind == G.VELOCITY][0]
    hlb.hlb_snapshot_alloc(sim.ctx, 1)
    x = torch.zeros(1 << 20, device="cuda")
    out = []
    for call in range(24):
        if call == 9:  # other values in the same table
            hlb.hlb_set_iolet_table(sim.ctx, k_in, 0.015 * np.ones(37))
        if call == 11:  # another table length: another device array
            hlb.hlb_set_iolet_table(sim.ctx, k_in, 0.012 * np.ones(5))
        if call == 12:
            hlb.hlb_snapshot_save(sim.ctx, 0)
        if call == 17:  # an odd count in between, then back to the snapshot
            sim.step(3)
            hlb.hlb_snapshot_restore(sim.ctx, 0)
        if call == 20:
            phi = np.zeros(g.n)
            phi[g.wall_sites()] = 0.1
            hlb.hlb_set_porosity(sim.ctx, phi)
        x.mul_(1.0)  # work of the null stream around the calls
        sim.step(n)
        x.add_(1.0)
        out.append(hlb.hlb_get_state(sim.ctx))
    assert sim.t == (24 - 5) * n
    m, r = hlb.hlb_mass_balance(sim.ctx)
    sim.close()
    return out, m


@pytest.mark.parametrize("n", [67, 80])
@pytest.mark.parametrize("storage,scheme", [("f64", "pull"), ("f32", "pull"), ("f16", "pull"), ("f64", "push")])
def test_repeated_calls_match_plain_launches(n, storage, scheme):
    import torch
    print(f"case: {n} steps a call, {storage} {scheme}", flush=True)
    a, ma = _run(n, storage, scheme, None)
    b, mb = _run(n, storage, scheme, torch.cuda.Stream())
    for k, (x, y) in enumerate(zip(a, b)):
        assert np.array_equal(x, y), f"call {k} differs"
    assert ma == mb
