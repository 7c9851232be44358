"""Steps of a state that stays in the Infinity Cache (both buffers between 20
and 208 MB: cached stores and, in FP64 and FP32, the short chain of row loads),
fields against the oracle, with a bulk group that ends inside a block."""
import numpy as np
import pytest

import oracle
from paper_2202_11770_amd import geometry as G
from paper_2202_11770_amd import hlb
from _parity import random_field

pytestmark = pytest.mark.gpu

STEPS = 6


def _bar(storage):
    """The stored values of a site sum to at most drho + 3 u + 6 u^2 = 0.073 in magnitude (drho 0.01, u 0.02), and
    every step rounds each of them to half a unit of the storage's last place: STEPS 0.073 eps in density and in
    momentum at most, twice that for the sums' propagation through collisions that do not shrink them; FP32 computes
    in its storage's precision, with two further roundings of that size per step.  FP64: as every parity case."""
    if storage == "f64":
        return 1e-12
    return STEPS * 0.073 * (2 * 2.0 ** -11 if storage == "f16" else 6 * 2.0 ** -24)


@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
@pytest.mark.parametrize("porous", [False, True])
def test_fields_while_the_state_is_cached(storage, porous):
    g = G.tree(seed=3, generations=4, scale=0.35)
    tables = [np.array([0.01 if io.kind == G.VELOCITY else 1.001]) for io in g.iolets]
    phi = np.random.default_rng(7).uniform(0.0, 0.3, g.n) if porous else None
    rho0, u0 = random_field(g.n, 5)
    prob = oracle.Problem(g, 0.7, tables=tables, phi=phi)
    f = prob.init(rho0, u0)
    prob.run(f, 0, STEPS)
    rho_r, u_r, wss_r = prob.macros(f)
    sim = hlb.Simulation.create(g, 0.7, storage=storage, tables=tables)
    info = sim.info()
    mb = 2 * 19 * info["n_padded"] * {"f64": 8, "f32": 4, "f16": 2}[storage] / 1e6
    assert 20.0 <= mb <= 208.0 and info["group_sites"][0] % 256 != 0
    if porous:
        hlb.hlb_set_porosity(sim.ctx, phi)
    hlb.hlb_init_equilibrium(sim.ctx, rho0, u0)
    sim.step(STEPS)
    rho, u, wss = sim.macros()
    sim.close()
    bar = _bar(storage)
    e = (np.abs(rho - rho_r).max(), np.abs(u - u_r).max(), np.abs(wss - wss_r).max())
    print(f"case: {storage} porous {porous}, {mb:.0f} MB: {e[0]:.2e} {e[1]:.2e} {e[2]:.2e}, bar {bar:.2e}", flush=True)
    assert e[0] <= bar and e[1] <= bar
    assert e[2] <= 4 * bar  # two projections of the second moments, |c c| <= 2 in sum
