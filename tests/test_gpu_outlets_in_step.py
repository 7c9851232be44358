"""Windkessel outlets advanced at the end of the step kernel: more outlets
than a workgroup has threads, none with a site at all, replayed graphs; and the
adjoint sweep, which steps in buffers of its own, leaves every part of the
caller's state as it was."""
import numpy as np
import pytest

import oracle
from paper_2202_11770_amd import geometry as G
from paper_2202_11770_amd import hlb
from _parity import errors, fmt, random_field

pytestmark = pytest.mark.gpu

MODEL = (1.0, 0.002, 500.0, 0.004, 0.0005)


@pytest.mark.parametrize("scheme,graph_steps", [("pull", 0), ("pull", 4), ("push", 0)])
def test_more_outlets_than_threads(scheme, graph_steps):
    g = G.tree(seed=2, generations=9, scale=0.35)
    outs = [k for k, io in enumerate(g.iolets) if io.kind == G.PRESSURE]
    assert len(outs) == 512
    s = np.arange(50)
    tables = [0.01 + 0.002 * np.sin(s / 8.0) if io.kind == G.VELOCITY else None for io in g.iolets]
    models = {k: (1.0, 0.001 * (1 + j % 7), 400.0 + j, 0.004, 0.0) for j, k in enumerate(outs)}
    prob = oracle.Problem(g, 0.7, tables=tables)
    f = prob.init()
    want = prob.run_windkessel(f, 0, 13, models)
    sim = hlb.Simulation.create(g, 0.7, tables=tables, scheme=scheme, graph_steps=graph_steps)
    for k, m in models.items():
        hlb.hlb_set_windkessel(sim.ctx, k, m)
    sim.step(13)
    e = errors(*sim.macros(), *prob.macros(f))
    worst = max(abs(a - b) / max(abs(b), 1e-6) for k in outs for a, b in zip(hlb.hlb_windkessel_state(sim.ctx, k), want[k]))
    sim.close()
    print(f"case: {g.n} sites, {len(outs)} outlets, {scheme}, graph {graph_steps}: {fmt(e)}; outlets {worst:.1e}", flush=True)
    assert e["e_rho"] <= 1e-12 and e["e_u"] <= 1e-12 and worst <= 1e-9


@pytest.mark.parametrize("scheme", ["pull", "push"])
def test_outlet_without_sites(scheme):
    """No iolet site in the domain: the outflow is zero and X leaks at 1/(R2 C) a step."""
    g = G.sealed_box(8)
    g.iolets.append(G.Iolet(G.PRESSURE, G.OUTLET, (1e4, 0.0, 0.0), (1.0, 0.0, 0.0), 2.0, table=np.array([1.0])))
    sim = hlb.Simulation.create(g, 0.8, scheme=scheme)
    hlb.hlb_set_windkessel(sim.ctx, 0, MODEL)
    sim.step(20)
    rho, X, q = hlb.hlb_windkessel_state(sim.ctx, 0)
    sim.close()
    want = MODEL[4] * (1.0 - 1.0 / (MODEL[3] * MODEL[2])) ** 20
    assert q == 0.0 and abs(X - want) <= 1e-15 and abs(rho - 1.0 - want) <= 1e-15


@pytest.mark.parametrize("slots", [1, 2, 5])
def test_sweep_leaves_the_callers_state(slots):
    g = G.tree(seed=3, generations=3, target_sites=30000)
    outs = [k for k, io in enumerate(g.iolets) if io.kind == G.PRESSURE]
    tables = [np.array([0.01]) if io.kind == G.VELOCITY else None for io in g.iolets]
    sim = hlb.Simulation.create(g, 0.7, tables=tables, adjoint=True)
    ref = hlb.Simulation.create(g, 0.7, tables=tables, adjoint=True)
    rho, u = random_field(g.n, 4)
    for x in (sim, ref):
        for k in outs[:3]:
            hlb.hlb_set_windkessel(x.ctx, k, MODEL)
        hlb.hlb_init_equilibrium(x.ctx, rho, u)
        x.step(3)  # an odd number: the current buffer is the second one
    before = (bytes(hlb.hlb_state_save(sim.ctx)), [hlb.hlb_windkessel_state(sim.ctx, k) for k in outs[:3]],
              hlb.hlb_mass_balance(sim.ctx), sim.macros())
    first = hlb.hlb_adjoint_run(sim.ctx, 9, 5, 12, slots)
    after = (bytes(hlb.hlb_state_save(sim.ctx)), [hlb.hlb_windkessel_state(sim.ctx, k) for k in outs[:3]],
             hlb.hlb_mass_balance(sim.ctx), sim.macros())
    assert before[:3] == after[:3] and all(np.array_equal(a, b) for a, b in zip(before[3], after[3]))
    again = hlb.hlb_adjoint_run(sim.ctx, 9, 5, 12, slots)
    # J and the table rows are summed by atomics: rounding
    assert abs(again[0] - first[0]) <= 1e-12 * abs(first[0]) and np.allclose(again[1], first[1], rtol=1e-10, atol=1e-300)
    # a sweep between two runs of steps changes nothing in them
    sim.step(4)
    ref.step(4)
    for a, b in zip(sim.macros(), ref.macros()):
        assert np.abs(a - b).max() <= 1e-13
    sim.close()
    ref.close()
