"""The fused reverse step: sites that touch several iolets (against the
oracle's reference adjoint), odd step counts with every checkpoint count
(which of the two buffers holds the next adjoint), and the 64-bit address
path of buffers beyond 4 GiB (against central differences)."""
import numpy as np
import pytest

import oracle
from paper_2202_11770_amd import geometry as G
from paper_2202_11770_amd import hlb
from _parity import random_field
from test_gpu_iolet_corner import P, TABLES, V, _corner_box

pytestmark = pytest.mark.gpu


def rel(a, b):
    return float(np.linalg.norm(np.asarray(a) - np.asarray(b)) / max(np.linalg.norm(np.asarray(b)), 1e-300))


@pytest.mark.parametrize("objective", ["wss", "flux"])
@pytest.mark.parametrize("porous", [False, True])
@pytest.mark.parametrize("kinds", [(V, P, V), (P, P, V), (P, P, P)])
def test_adjoint_at_sites_touching_several_iolets(kinds, porous, objective):
    g = _corner_box(kinds)
    tau, n, w0 = 0.8, 23, 9
    tables = [np.resize(TABLES[k], n) for k in kinds]
    phi = np.random.default_rng(3).uniform(0.0, 0.3, g.n) if porous else None
    rho0, u0 = random_field(g.n, 5)
    prob = oracle.Problem(g, tau, tables=tables, phi=phi)
    w = np.array([1.0, -0.5, 0.7]) if objective == "flux" else None
    Jr, dAr, dphir = prob.adjoint(prob.init(rho0, u0), 0, n, w0, n, weights=w)
    sim = hlb.Simulation.create(g, tau, tables=tables, adjoint=True)
    if porous:
        hlb.hlb_set_porosity(sim.ctx, phi)
    if w is not None:
        hlb.hlb_set_objective(sim.ctx, hlb.HLB_OBJ_IOLET_FLUX, w)
    hlb.hlb_init_equilibrium(sim.ctx, rho0, u0)
    for slots in (1, 2, 5, n + 1):
        J, dA, dphi, _ = hlb.hlb_adjoint_run(sim.ctx, n, w0, n, slots)
        print(f"case: {kinds} porous={porous} {objective} {slots} slots: J {abs(J - Jr) / abs(Jr):.1e} "
              f"tables {rel(dA, dAr):.1e} phi {rel(dphi, dphir):.1e}", flush=True)
        assert abs(J - Jr) <= 1e-12 * abs(Jr) and rel(dA, dAr) <= 1e-10 and rel(dphi, dphir) <= 1e-10
    sim.close()


def test_wide_addressing_adjoint_vs_finite_differences():
    """304 x 304 x 310 duct: 4.3 GB per buffer.  The outflow objective is smooth in the densities and the porosity:
    central differences with h = 1e-4 are off by about h^2 (1e-8) and rounding far below."""
    import torch
    g = G.duct(304, 304, 310)
    tau, n = 0.8, 4
    sim = hlb.Simulation.create(g, tau, adjoint=True)
    assert 19 * 8 * hlb.hlb_info(sim.ctx)["n_padded"] > 2 ** 32
    rng = np.random.default_rng(8)
    R = [1.006 + 1e-3 * rng.uniform(-1, 1, n), 1.0 + 1e-3 * rng.uniform(-1, 1, n)]
    phi = torch.full((g.n,), 0.05, dtype=torch.float64, device="cuda")
    vR = [rng.uniform(-1, 1, n) for _ in R]
    vphi = torch.rand(g.n, dtype=torch.float64, device="cuda", generator=torch.Generator(device="cuda").manual_seed(1))
    hlb.hlb_set_objective(sim.ctx, hlb.HLB_OBJ_IOLET_FLUX, np.array([-0.5, 1.0]))

    def J(eR, ephi, grads=False):
        for k in range(2):
            hlb.hlb_set_iolet_table(sim.ctx, k, R[k] + eR * vR[k])
        p = phi + ephi * vphi
        hlb.hlb_set_porosity_device(sim.ctx, p)
        out = torch.empty(1, dtype=torch.float64, device="cuda")
        dA = torch.empty(2, n, dtype=torch.float64, device="cuda") if grads else None
        dphi = torch.empty(g.n, dtype=torch.float64, device="cuda") if grads else None
        hlb.hlb_adjoint_run_device(sim.ctx, n, 0, n, 2, out, dA, dphi)
        torch.cuda.synchronize()
        return (out.item(), dA.cpu().numpy(), float((dphi * vphi).sum())) if grads else out.item()

    J0, dA, dphi = J(0.0, 0.0, True)
    h = 1e-4
    fd_R = (J(h, 0.0) - J(-h, 0.0)) / (2 * h)
    fd_p = (J(0.0, h) - J(0.0, -h)) / (2 * h)
    ad_R = sum(float(dA[k] @ vR[k]) for k in range(2))
    print(f"case: wide adjoint {g.n} sites: J {J0:.6e}; densities {ad_R:.9e} vs {fd_R:.9e}; "
          f"porosity {dphi:.9e} vs {fd_p:.9e}", flush=True)
    assert abs(ad_R - fd_R) <= 1e-6 * abs(fd_R)
    assert abs(dphi - fd_p) <= 1e-6 * abs(fd_p)
    # the WSS objective's value against the fields of the forward run
    J(0.0, 0.0)
    hlb.hlb_set_objective(sim.ctx, hlb.HLB_OBJ_WSS)
    out = torch.empty(1, dtype=torch.float64, device="cuda")
    hlb.hlb_adjoint_run_device(sim.ctx, n, 1, n, 2, out)
    wss = torch.empty(g.n, dtype=torch.float64, device="cuda")
    want = 0.0
    for t in range(n):
        sim.step(1)
        if t >= 1:
            hlb.hlb_macros_device(sim.ctx, wss=wss)
            torch.cuda.synchronize()
            want += float(wss.sum())
    assert abs(out.item() - want) <= 1e-12 * want
    sim.close()
