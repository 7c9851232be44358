"""The boundary mass flux kept as partial sums: the balance residual over
porous walls on a state with more wavefronts than partial sums, and the same
residual, bit for bit, after every call that folds, keeps or restores them."""
import numpy as np
import pytest

from paper_2202_11770_amd import geometry as G
from paper_2202_11770_amd import hlb
from _parity import random_field

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage,scheme", [("f64", "pull"), ("f32", "pull"), ("f64", "push")])
def test_porous_flux_closes_the_balance(storage, scheme):
    g = G.tree(seed=3, generations=4, scale=0.35)
    assert g.n > 64 * 4096
    steps = 12
    sim = hlb.Simulation.create(g, 0.7, storage=storage, scheme=scheme, tables=[np.array([0.01 if io.kind == G.VELOCITY else 1.0])
                                                                               for io in g.iolets])
    rng = np.random.default_rng(7)
    phi = rng.uniform(0.0, 0.5, g.n)
    hlb.hlb_set_porosity(sim.ctx, phi)
    rho, u = random_field(g.n, 11)
    rho += 0.02  # above the reservoir's density: the walls leak
    hlb.hlb_init_equilibrium(sim.ctx, rho, u)
    m0, r0 = hlb.hlb_mass_balance(sim.ctx)
    sim.step(steps)
    m1, r1 = hlb.hlb_mass_balance(sim.ctx)
    # rounding per site and step: 19 stored values (FP64: weights up to 1/3; shifted: deviations below 0.05 of
    # them), the same again for the flux terms of the wall links
    eps, size = (2.0 ** -53, 1.0) if storage == "f64" else (2.0 ** -24, 0.05)
    bound = steps * 38 * eps * size * g.n
    print(f"case: {storage} {scheme}: mass change {m1 - m0:.6e}, residual {r1:.3e}, bound {bound:.3e}", flush=True)
    assert abs(m1 - m0) > 100 * bound  # what the boundaries moved is far above the rounding
    assert abs(r1) <= bound
    assert hlb.hlb_mass_balance(sim.ctx) == (m1, r1)
    hlb.hlb_snapshot_alloc(sim.ctx, 1)
    sim.step(3)
    hlb.hlb_snapshot_save(sim.ctx, 0)  # folds the sums of three steps
    m2, r2 = hlb.hlb_mass_balance(sim.ctx)
    assert abs(r2) <= bound * (steps + 3) / steps
    buf = hlb.hlb_state_save(sim.ctx)
    sim.step(4)
    hlb.hlb_snapshot_restore(sim.ctx, 0)
    assert hlb.hlb_mass_balance(sim.ctx) == (m2, r2)
    sim.step(5)
    hlb.hlb_state_load(sim.ctx, buf)
    assert hlb.hlb_mass_balance(sim.ctx) == (m2, r2)
    sim.close()
