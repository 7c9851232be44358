"""The ghost density's fill, bit for bit: with the collision switched off
(tau so large that omega times any difference vanishes) a step only streams,
and the populations that a pressure iolet fills are compared with the same
multiply-adds done in exact arithmetic, rounded where the fill rounds."""
from fractions import Fraction

import numpy as np
import pytest

from paper_2202_11770_amd import geometry as G
from paper_2202_11770_amd import hlb
from _parity import random_field

pytestmark = pytest.mark.gpu

C = np.array([[0, 0, 0], [1, 0, 0], [-1, 0, 0], [0, 1, 0], [0, -1, 0], [0, 0, 1], [0, 0, -1], [1, 1, 0], [-1, -1, 0],
              [1, -1, 0], [-1, 1, 0], [1, 0, 1], [-1, 0, -1], [1, 0, -1], [-1, 0, 1], [0, 1, 1], [0, -1, -1],
              [0, 1, -1], [0, -1, 1]])
OPP = [0] + [i + 1 if i % 2 else i - 1 for i in range(1, 19)]
STORE = {"f64": np.float64, "f32": np.float32, "f16": np.float16}
RHO = 1.003  # the outlets' density


def _fma(a, b, c):
    """a b + c with one rounding to the operands' type."""
    x = Fraction(float(a)) * Fraction(float(b)) + Fraction(float(c))
    if x == 0:
        return type(a)(0)
    m, d = abs(x.numerator), x.denominator
    e = m.bit_length() - d.bit_length()
    e -= Fraction(m, d) < (Fraction(2) ** e)  # 2^e <= |x| < 2^(e+1)
    ulp = Fraction(2) ** (e - (23 if type(a) is np.float32 else 52))
    return type(a)(float(round(x / ulp) * ulp))  # round: half to even


def _fill(T, i, s, n, shifted):
    """Population i at density RHO and the velocity of the stored values s along n."""
    s = s.astype(T)
    dr, j = T(0), [T(0)] * 3
    for q in range(19):
        dr = dr + s[q]
        for a in range(3):
            if C[q, a]:
                j[a] = j[a] + (s[q] if C[q, a] > 0 else -s[q])
    rho = T(1) + dr if shifted else dr
    u = [x / rho for x in j]
    n = [T(x) for x in n]
    un = _fma(u[2], n[2], _fma(u[0], n[0], u[1] * n[1]))
    g = [un * x for x in n]
    sq = _fma(g[2], g[2], _fma(g[0], g[0], g[1] * g[1]))
    x, y, z = (T(v) for v in C[i])
    if C[i, 0] and C[i, 1]:
        cu = _fma(n[1], un, -g[0]) if (x, y) == (-1, 1) else _fma(x * n[0], un, y * g[1])
    else:
        cu = x * g[0] + y * g[1]
    if C[i, 2]:
        cu = _fma(z * n[2], un, cu)
    q = _fma(T(-1.5), sq, _fma(T(3), cu, (T(4.5) * cu) * cu))
    w = T(1) / T(18 if i <= 6 else 36)
    if shifted:
        return w * _fma(q, T(RHO), T(RHO - 1.0))
    return (w * T(RHO)) * (T(1) + q)


@pytest.mark.parametrize("scheme", ["pull", "push"])
@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
def test_fill_rounds_as_written(storage, scheme):
    g = G.tree(seed=2, generations=3, scale=0.15)
    tables = [np.array([0.01 if io.kind == G.VELOCITY else RHO]) for io in g.iolets]
    sim = hlb.Simulation.create(g, 1e300, storage=storage, scheme=scheme, tables=tables)
    rho, u = random_field(g.n, 3, umax=0.08)
    hlb.hlb_init_equilibrium(sim.ctx, rho, u)
    shifted = storage != "f64"
    w = np.array([1 / 3] + [1 / 18] * 6 + [1 / 36] * 12) if shifted else np.zeros(19)
    S = STORE[storage]
    own = (hlb.hlb_get_state(sim.ctx) - w).astype(S)  # the stored values
    states = []
    for _ in range(2):
        sim.step(1)
        states.append(hlb.hlb_get_state(sim.ctx))
    sim.close()
    T = np.float64 if storage == "f64" else np.float32
    checked = 0
    for i in range(1, 19):
        for x in np.nonzero(g.nbr[:, OPP[i]] < -1)[0]:
            io = g.iolets[-g.nbr[x, OPP[i]] - 2]
            if io.kind != G.PRESSURE or np.unique(g.nbr[x][g.nbr[x] < -1]).size > 1:
                continue
            stepped = S(_fill(T, i, own[x], io.normal, shifted)) + w[i]
            if scheme == "push":  # the step's own fill, in the buffer
                assert states[0][x, i] == stepped, f"site {x} direction {i}"
                checked += 1
                continue
            # the fields' fill, in FP64 from the stored values
            assert states[0][x, i] == _fill(np.float64, i, own[x], io.normal, shifted) + w[i], f"site {x} direction {i}"
            y = g.nbr[x, i]
            if y >= 0:  # the step's fill, moved on by the second step
                assert states[1][y, i] == stepped, f"site {x} direction {i}, moved to {y}"
                checked += 1
    assert checked > 300
