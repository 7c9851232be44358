"""A state buffer restores the state, the time and the mass bookkeeping, and
nothing that a running step counts with: whatever stands in the unused words
of its header, Windkessel outlets go on after hlb_state_load."""
import numpy as np
import pytest

from paper_2202_11770_amd import geometry as G
from paper_2202_11770_amd import hlb

pytestmark = pytest.mark.gpu

ACC = 8 + 4 * 8 + 4 * 4 + 8  # magic, four 64-bit and four 32-bit numbers, m0: the bookkeeping follows


@pytest.mark.parametrize("word", [1, 2, 3])
@pytest.mark.parametrize("scheme", ["pull", "push"])
def test_unused_words_of_the_header_do_not_matter(scheme, word):
    g = G.cylinder()
    tables = [np.array([0.01 if io.kind == G.VELOCITY else 1.0]) for io in g.iolets]
    k = [k for k, io in enumerate(g.iolets) if io.kind == G.PRESSURE][0]
    out = []
    for damaged in (False, True):
        sim = hlb.Simulation.create(g, 0.8, scheme=scheme, tables=tables)
        hlb.hlb_set_windkessel(sim.ctx, k, (1.0, 0.01, 2000.0, 0.02, 0.0))
        hlb.hlb_init_equilibrium(sim.ctx, None, np.tile(0.02 * -np.array(g.iolets[k].normal), (g.n, 1)))
        sim.step(5)
        q5 = hlb.hlb_windkessel_state(sim.ctx, k)[2]
        blob = hlb.hlb_state_save(sim.ctx)
        assert blob[ACC + 8:ACC + 32] == bytes(24)
        if damaged:
            blob[ACC + 8 * word:ACC + 8 * word + 4] = (7).to_bytes(4, "little")
        hlb.hlb_state_load(sim.ctx, blob)
        sim.step(20)
        rho, x, q = hlb.hlb_windkessel_state(sim.ctx, k)
        assert abs(q - q5) > 1e-3 * abs(q5) > 0.0  # the outlet goes on
        out.append((rho, x, q, sim.macros()[0], hlb.hlb_mass_balance(sim.ctx)[0]))
        sim.close()
    # the outflow is summed by atomics: equal to rounding
    for a, b in zip(*out):
        np.testing.assert_allclose(b, a, rtol=1e-11, atol=1e-14)
