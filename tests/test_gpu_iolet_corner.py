"""Sites that touch two and three iolets at once (edges and a corner of a box
with iolets on three faces), porous walls beside them, and table times beyond
2^32: the iolet groups' gather against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2202_11770_amd import geometry as G
from paper_2202_11770_amd import hlb
from _parity import errors, fmt, random_field

pytestmark = pytest.mark.gpu


def _corner_box(kinds, n=9):
    """n x n x n box with an inlet-role iolet on each of the faces x, y, z = 0."""
    normals = [(1.0, 0.0, 0.0), (0.0, 1.0, 0.0), (0.0, 0.0, 1.0)]
    mid = (n - 1) / 2.0
    iolets = [G.Iolet(kind, G.INLET, tuple(-0.5 if a == k else mid for a in range(3)), normals[k], 2.0 * n)
              for k, kind in enumerate(kinds)]
    g = G.build_sites(G._pack(np.ones(n ** 3, dtype=bool)), (n, n, n), iolets)
    links = [set(row[row < -1].tolist()) for row in g.nbr]
    assert max(len(s) for s in links) == 3 and sum(len(s) == 2 for s in links) >= 3 * (n - 1)
    return g


V, P = G.VELOCITY, G.PRESSURE
TABLES = {V: 0.01 + 0.002 * np.sin(np.arange(7)), P: 1.0 + 1e-3 * np.cos(np.arange(5))}


def _bars(storage, steps):
    """FP64 as every parity case; FP32 and FP16 three times the random walk of the storage rounding of 19 values per
    step (deviations up to w (rho - 1) = 0.06 here), the velocity relative to 0.01."""
    if storage == "f64":
        return 1e-12, 1e-12
    e = 3.0 * np.sqrt(19.0 * steps) * 0.06 * (2.0 ** -24 if storage == "f32" else 2.0 ** -11)
    return e, e / 0.01


@pytest.mark.parametrize("storage,scheme", [("f64", "pull"), ("f32", "pull"), ("f16", "pull"), ("f64", "push")])
@pytest.mark.parametrize("kinds", [(V, P, V), (P, P, V), (V, V, V)])
@pytest.mark.parametrize("porous", [False, True])
def test_sites_touching_several_iolets(kinds, porous, storage, scheme):
    g = _corner_box(kinds)
    tau, steps, tables = 0.8, 40, [TABLES[k] for k in kinds]
    phi = np.random.default_rng(3).uniform(0.0, 0.3, g.n) if porous else None
    rho0, u0 = random_field(g.n, 5)
    prob = oracle.Problem(g, tau, tables=tables, phi=phi)
    f = prob.init(rho0, u0)
    prob.run(f, 0, steps)
    sim = hlb.Simulation.create(g, tau, storage=storage, scheme=scheme, tables=tables)
    if porous:
        hlb.hlb_set_porosity(sim.ctx, phi)
    hlb.hlb_init_equilibrium(sim.ctx, rho0, u0)
    sim.step(steps)
    e = errors(*sim.macros(), *prob.macros(f))
    sim.close()
    print(f"case: {kinds} porous={porous} {storage} {scheme}: {fmt(e)}", flush=True)
    bar = _bars(storage, steps)
    assert e["e_rho"] <= bar[0] and e["e_u"] <= bar[1]


def test_two_windkessel_outlets_at_one_site():
    g = _corner_box((P, P, V))
    tables = [None, None, TABLES[V]]
    models = {0: (1.0, 0.002, 500.0, 0.004, 0.0), 1: (1.0, 0.001, 0.0, 0.003, 0.0)}
    prob = oracle.Problem(g, 0.8, tables=tables)
    f = prob.init()
    want = prob.run_windkessel(f, 0, 30, models)
    sim = hlb.Simulation.create(g, 0.8, tables=tables)
    for k, m in models.items():
        hlb.hlb_set_windkessel(sim.ctx, k, m)
    sim.step(30)
    e = errors(*sim.macros(), *prob.macros(f))
    got = {k: hlb.hlb_windkessel_state(sim.ctx, k) for k in models}
    sim.close()
    print(f"case: two Windkessel outlets at one site: {fmt(e)}", flush=True)
    assert e["e_rho"] <= 1e-12 and e["e_u"] <= 1e-12
    for k in models:
        assert all(abs(a - b) <= 1e-11 * max(abs(b), 1e-1) for a, b in zip(got[k], want[k]))


def test_table_times_beyond_32_bits():
    """The same table values at t0 and at t0 + a multiple of both table lengths: bit for bit the same steps."""
    g = _corner_box((V, P, V))
    out = []
    for t0 in (4, 4 + 35 * (2 ** 32 // 35 + 1), 4 + 35 * (2 ** 32 // 35)):  # 2^32 is crossed in the last one's steps
        sim = hlb.Simulation.create(g, 0.8, tables=[TABLES[V], TABLES[P], TABLES[V]])
        hlb.hlb_init_equilibrium(sim.ctx, None, None, t0)
        sim.step(40)
        out.append(sim.macros())
        sim.close()
    for other in out[1:]:
        assert all(np.array_equal(a, b) for a, b in zip(out[0], other))
