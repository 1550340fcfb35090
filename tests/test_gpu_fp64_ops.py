"""FP64 HLLC and HLLE near their switches (supersonic and transonic sides, equal
states, contacts at rest, far units) against the oracle, through one step of a
group of random states."""
import numpy as np
import pytest

import oracle as O
from paper_1103_3373_amd import workloads as W
from tests._util import scaled_max_err

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["mach10", "transonic", "contact", "scaled_up", "scaled_down"])
@pytest.mark.parametrize("scheme,recon", [(0, 1), (1, 0), (2, 1)])
@pytest.mark.parametrize("rs", [1, 2])
def test_fp64_solvers(kind, scheme, recon, rs):
    from paper_1103_3373_amd import hydro as H
    gamma, n = 1.4, 32
    rng = np.random.default_rng(rs)
    shape = (n, n, n)
    rho, p = rng.lognormal(0, 0.3, shape), rng.lognormal(0, 0.3, shape)
    v = [0.3 * rng.standard_normal(shape) for _ in range(3)]
    if kind == "mach10":
        v[0] += 12.0
        v[2] -= 9.0
    elif kind == "transonic":
        v[1] += 1.18
    elif kind == "contact":
        v, p = [np.zeros(shape)] * 3, np.ones(shape)
    U = W.primitive_to_conserved(rho, *v, p, gamma)
    if kind.startswith("scaled"):  # density and energy in units far from 1
        U *= 1e60 if kind == "scaled_up" else 1e-60
        if kind == "scaled_down":  # the floors (1e-10) are not scaled
            U *= 1e52
    g = H.ghost_width(scheme, recon)
    G = O.fill_ghosts_periodic(U, g)
    dt = 0.5 * O.cfl_dt(U, 1 / n, gamma, 0.3)
    ref, rflux = O.solve_groups(G, g, dt, 1 / n, gamma, scheme, recon, rs, 1, O.F_CHAR, want_flux=True)
    out = torch.empty((8, 5, 16, 16, 16), dtype=torch.float64, device="cuda")
    flux = torch.empty((8, 3, 2, 5, 16, 16), dtype=torch.float64, device="cuda")
    H.solve_groups(torch.from_numpy(G).cuda(), out, flux, dt=dt, dh=1 / n, gamma=gamma, scheme=scheme, recon=recon,
                   riemann=rs, char=True)
    # the FP64 bar of one step
    assert scaled_max_err(out.cpu().numpy(), ref) <= 1e-12
    assert scaled_max_err(flux.cpu().numpy(), rflux) <= 1e-12
