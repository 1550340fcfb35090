"""The exact Riemann solver in the fused kernels against the paper-style kernel
(HYDRO_PLAIN): whole groups and groups split along z, vacuum and strong shocks."""
import numpy as np
import pytest

from paper_1103_3373_amd import workloads as W
from tests._util import scaled_max_err

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def H():
    from paper_1103_3373_amd import hydro
    hydro.lib()
    return hydro


def _both(H, G, dt, dtype, **kw):
    got = []
    for plain in (False, True):
        out = torch.empty((G.shape[0], 5, 16, 16, 16), dtype=dtype, device="cuda")
        flux = torch.empty((G.shape[0], 3, 3, 5, 16, 16), dtype=dtype, device="cuda")
        H.get_diag(reset=True)
        H.solve_groups(G, out, flux, dt=dt, dh=1 / 64, gamma=1.4, riemann=H.EXACT, plain=plain, flux_mid=True, **kw)
        got.append((out.double().cpu().numpy(), flux.double().cpu().numpy(), H.get_diag(reset=True)))
    return got


@pytest.mark.parametrize("n", [1, 5, 48, 520])
@pytest.mark.parametrize("scheme,recon,limiter,char", [(0, 0, 1, False), (0, 1, 3, True), (1, 0, 2, True), (1, 1, 1, False),
                                                       (2, 0, 0, True), (2, 1, 1, True)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_exact_fused_equals_plain(H, n, scheme, recon, limiter, char, dtype):
    g = H.ghost_width(scheme, recon)
    # 128 x 128 x 144: 576 groups of a blast field, the first n of them
    U = W.lognormal_blast_box(64, gamma=1.4, seed=5, radius_cells=5)
    box = torch.from_numpy(np.tile(U, (1, 2, 2, 2))).to(device="cuda", dtype=dtype)
    box = torch.cat([box, box[:, :16]], 1).contiguous()
    G = H.fill_ghosts_periodic(box, g)[-n:].contiguous()
    (a, fa, _), (b, fb, _) = _both(H, G, 4e-4, dtype, scheme=scheme, recon=recon, limiter=limiter, char=char)
    # One step: 1e-12 in FP64; FP32 solves to a relative change of 1e-6
    bar = 1e-12 if dtype == torch.float64 else 1e-5
    assert scaled_max_err(a, b) <= bar and scaled_max_err(fa, fb) <= bar


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_exact_vacuum_and_shock(H, dtype):
    """A receding pair that generates vacuum is counted on both paths (where its fan has no real
    state at the face, NaN in the same cells); a colliding pair is not."""
    for speed, vacuum in ((6.0, True), (-3.0, False)):
        x = (np.arange(64) + 0.5) / 64
        u = np.where((x > 0.25) & (x < 0.75), speed, -speed)[None, None, :] * np.ones((32, 32, 1))
        U = W.primitive_to_conserved(np.ones_like(u), u, 0 * u, 0 * u, 0.4 * np.ones_like(u), 1.4)
        G = H.fill_ghosts_periodic(torch.from_numpy(U).to(device="cuda", dtype=dtype), 2)
        (a, fa, da), (b, fb, db) = _both(H, G, 1e-4, dtype, scheme=0, recon=0, limiter=1, char=False)
        assert (da["roe_fallbacks"] > 0) == (db["roe_fallbacks"] > 0) == vacuum
        bar = 1e-12 if dtype == torch.float64 else 1e-5
        for p, q in ((a, b), (fa, fb)):
            assert np.array_equal(np.isnan(p), np.isnan(q)) and (vacuum or not np.isnan(p).any())
            assert scaled_max_err(p[~np.isnan(p)], q[~np.isnan(q)]) <= bar
