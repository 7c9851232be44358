"""A field asked for alone is the field asked for with the others, bit for
bit, from the values as they are (after a set-up, and the push scheme) and
from the gathered ones, solid and porous."""
import itertools

import numpy as np
import pytest

from paper_2202_11770_amd import geometry as G
from paper_2202_11770_amd import hlb
from _parity import random_field

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
@pytest.mark.parametrize("scheme", ["pull", "push"])
@pytest.mark.parametrize("porous", [False, True])
def test_each_field_alone(storage, scheme, porous):
    g = G.tree(seed=2, generations=3, scale=0.15)
    assert g.n % 256 != 0
    tables = [np.array([0.01 if io.kind == G.VELOCITY else 1.001]) for io in g.iolets]
    sim = hlb.Simulation.create(g, 0.7, storage=storage, scheme=scheme, tables=tables)
    if porous:
        hlb.hlb_set_porosity(sim.ctx, np.random.default_rng(1).uniform(0.0, 0.2, g.n))
    hlb.hlb_init_equilibrium(sim.ctx, *random_field(g.n, 3))
    names = ("rho", "u", "wss")
    for steps in (0, 1, 3):  # 0: the set-up's own values
        sim.step(steps)
        whole = hlb.hlb_macros(sim.ctx)
        state = hlb.hlb_get_state(sim.ctx)
        np.testing.assert_allclose(state.sum(1), whole[0], rtol=1e-14)
        assert np.any(whole[2] > 0.0)
        for k in (1, 2):
            for want in itertools.combinations(names, k):
                part = hlb.hlb_macros(sim.ctx, want)
                for name, a, b in zip(names, part, whole):
                    assert (a is None) == (name not in want)
                    assert a is None or np.array_equal(a, b), f"{name} of {want} after {steps} more steps"
    sim.close()
