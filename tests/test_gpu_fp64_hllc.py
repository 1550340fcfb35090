"""FP64 HLLC on supersonic sides: the physical flux of that side, as rounded
there, also where the sound speed is lost beside the velocity."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
GAMMA = 1.4


def _solve(H, W, scheme):
    """One step of groups that are uniform each: states W [n, 5] (primitive)."""
    g = H.ghost_width(scheme, H.PLM)
    N = 16 + 2 * g
    U = np.empty_like(W)
    U[:, 0] = W[:, 0]
    U[:, 1:4] = W[:, :1] * W[:, 1:4]
    U[:, 4] = W[:, 4] / (GAMMA - 1.0) + 0.5 * W[:, 0] * (W[:, 1:4] ** 2).sum(1)
    n = len(W)
    G = torch.from_numpy(np.ascontiguousarray(np.broadcast_to(U[:, :, None, None, None], (n, 5, N, N, N)))).cuda()
    out = torch.empty((n, 5, 16, 16, 16), dtype=torch.float64, device="cuda")
    flux = torch.empty((n, 3, 2, 5, 16, 16), dtype=torch.float64, device="cuda")
    H.solve_groups(G, out, flux, dt=1e-3, dh=1 / 16, gamma=GAMMA, scheme=scheme, recon=H.PLM, riemann=H.HLLC)
    return U, out.cpu().numpy(), flux.cpu().numpy()


@pytest.mark.parametrize("scheme", [0, 1])
def test_cold_flow_stays_finite(scheme):
    """Speeds of 2^40 at the pressure floor: the fastest wave speed rounds to
    the velocity itself.  A uniform flow stays as it is."""
    from paper_1103_3373_amd import hydro as H
    v = 2.0 ** 40
    W = np.array([[1, v, 0, 0, 0], [1, -v, 0, 0, 0], [1, 0, v, 0, 0], [1, 0, 0, -v, 0], [4, v, -v, v, 0]], dtype=np.float64)
    U, out, flux = _solve(H, W, scheme)
    assert np.isfinite(out).all() and np.isfinite(flux).all()
    assert np.array_equal(out, np.broadcast_to(U[:, :, None, None, None], out.shape))


def test_mass_flux_of_a_supersonic_side():
    """Uniform groups that move faster than sound along every axis (VL, whose
    face states are then the cells' own): the mass flux is rho v rounded once."""
    from paper_1103_3373_amd import hydro as H
    rng = np.random.default_rng(3)
    n = 64
    W = np.empty((n, 5))
    W[:, 0], W[:, 4] = rng.lognormal(0, 1, n), rng.lognormal(0, 1, n)
    c = np.sqrt(GAMMA * W[:, 4] / W[:, 0])
    W[:, 1:4] = rng.choice([-1.0, 1.0], (n, 3)) * c[:, None] * rng.uniform(1.5, 20, (n, 3))
    U, _, flux = _solve(H, W, H.VL)
    v = U[:, 1:4] * (1.0 / U[:, :1])  # the kernels' primitive velocity: a rounded reciprocal, one product
    for d in range(3):
        want = (U[:, 0] * v[:, d])[:, None, None, None]
        assert np.array_equal(flux[:, d, :, 0], np.broadcast_to(want, flux[:, d, :, 0].shape)), d
