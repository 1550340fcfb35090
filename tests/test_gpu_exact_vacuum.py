"""The exact Riemann solver at the edge of vacuum, where the star pressure
underflows."""
import numpy as np
import pytest

import oracle as O
from paper_1103_3373_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("plain", [False, True])
@pytest.mark.parametrize("bulk", [0.0, 8.0, -8.0])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_edge_of_vacuum(plain, bulk, dtype):
    """Pairs that recede at (1 - e) of the speed that generates vacuum, e from
    1e-2 to 1e-9 over the rows of a box (gamma 1.4, whose fan powers 5 and 7
    are real for any base).  With a bulk velocity above 5 sqrt(gamma) + sqrt(gamma)
    every wave leaves in its direction, so that the x fluxes are the physical
    fluxes of the cells upwind (the step is too short to change them): to the
    parity bars, which are 100 roundings of the largest flux and more."""
    from paper_1103_3373_amd import hydro as H
    gamma, n = 1.4, 32
    e = 10.0 ** np.random.default_rng(1).uniform(-9, -2, (n, n, 1))
    speed = 2 / (gamma - 1) * np.sqrt(gamma) * (1 - e)  # a pair recedes at twice that, vacuum at 2 (cL + cR) / (gamma - 1)
    u = bulk + np.where(np.arange(n)[None, None, :] < n // 2, -speed, speed)
    one = np.ones_like(u)
    U = W.primitive_to_conserved(one, u, 0 * u, 0 * u, one, gamma)
    g = H.ghost_width(H.MHM, H.PLM)
    D = torch.from_numpy(O.fill_ghosts_periodic(U, g)).to(device="cuda", dtype=dtype)
    out = torch.empty((8, 5, 16, 16, 16), dtype=dtype, device="cuda")
    flux = torch.empty((8, 3, 2, 5, 16, 16), dtype=dtype, device="cuda")
    H.solve_groups(D, out, flux, dt=1e-20, dh=1 / n, gamma=gamma, scheme=H.MHM, recon=H.PLM, riemann=H.EXACT, plain=plain)
    assert torch.isfinite(out).all() and torch.isfinite(flux).all()
    if bulk:
        E = 1 / (gamma - 1) + 0.5 * u * u
        F = np.stack([u, u * u + 1, 0 * u, 0 * u, u * (E + 1)])  # of the cells
        F = F if bulk < 0 else np.roll(F, 1, 3)                   # at each cell's lower x face
        got, bar = flux[:, 0].double().cpu().numpy(), 1e-12 if dtype == torch.float64 else 1e-5
        for G in range(8):
            gx, y, z = G % 2, slice(16 * (G // 2 % 2), 16 * (G // 2 % 2) + 16), slice(16 * (G // 4), 16 * (G // 4) + 16)
            for f in range(2):
                want = F[:, z, y, (16 * (gx + f)) % n]
                assert np.abs(got[G, f] - want).max() <= bar * np.abs(F[4]).max(), (G, f)
