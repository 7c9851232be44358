"""FP16 step with its segment rows in LDS where every position of a block is a
segment of its own (a random caller order kept by the library) and where the
group ends inside a block: the same fields, bit for bit, as in the default
order."""
import numpy as np
import pytest

from paper_2202_11770_amd import geometry as G
from paper_2202_11770_amd import hlb
from _parity import random_field

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("radius,length", [(3.0, 9), (8.0, 64), (11.0, 73)])
def test_random_order_has_one_segment_per_position(radius, length):
    g = G.cylinder(radius=radius, length=length, box=int(2 * radius) + 4)
    perm = np.random.default_rng(2).permutation(g.n)
    q = G.permute(g, perm)
    rho, u = random_field(g.n, 9)
    out = []
    for geom, order, r0, u0 in ((g, None, rho, u), (q, "input", rho[perm], u[perm])):
        sim = hlb.Simulation.create(geom, 0.8, storage="f16", order=order)
        info = sim.info()
        hlb.hlb_init_equilibrium(sim.ctx, r0, u0)
        sim.step(20)
        out.append(sim.macros())
        sim.close()
    assert info["n_segments"] == info["group_sites"][0]
    print(f"case: {g.n} sites, {info['n_segments']} segments", flush=True)
    for a, b in zip(*out):
        assert np.array_equal(a[perm], b)
