"""Small launches split each group's planes over several workgroups: the same
bits, face fluxes and diagnostic counts as whole groups, and the oracle."""
import numpy as np
import pytest

import oracle as O
from paper_1103_3373_amd import workloads as W
from tests._util import scaled_max_err

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def H():
    from paper_1103_3373_amd import hydro
    hydro.lib()
    return hydro


def test_split_rule(H):
    """Workgroups of a box step without a pinned shape (256 compute units, or
    the device's): one group per workgroup once the chip is full, 16 workgroups
    per group on the smallest boxes."""
    spec = H.make_spec(H.CTU, H.PPM, H.HLLC, gamma=1.4, char=True)
    f64 = H.make_spec(H.CTU, H.PPM, H.HLLC, gamma=1.4, char=True, f64=True)
    try:
        H.set_launch_shape(spec, 0, 4)
        H.set_launch_shape(f64, 0, 2)
        assert H.get_launch_shape(spec, (32, 32, 32)) == (8 * 16, 4, 1)
        assert H.get_launch_shape(f64, (32, 32, 32)) == (8 * 16, 2, 1)
        assert H.get_launch_shape(spec, (128, 128, 128)) == (512, 4, 1)
        grids = [H.get_launch_shape(spec, (16 * k, 64, 64))[0] for k in range(1, 17)]
        assert all(g % (16 * k) == 0 and 1 <= g // (16 * k) <= 16 for k, g in enumerate(grids, 1))
        # a pinned variant without split kernels, or a pinned smaller grid, keeps whole groups
        H.set_launch_shape(spec, 0, 2)
        assert H.get_launch_shape(spec, (32, 32, 32)) == (8, 2, 1)
        H.set_launch_shape(spec, 7, 4)
        assert H.get_launch_shape(spec, (32, 32, 32)) == (7, 4, 1)
    finally:
        H.set_launch_shape(spec, 0, 4)
        H.set_launch_shape(f64, 0, 2)


@pytest.mark.gpu
@pytest.mark.parametrize("scheme", [0, 1, 2])
@pytest.mark.parametrize("recon,rs,char,limiter", [(1, 1, True, 1), (1, 0, True, 1), (0, 2, False, 2), (0, 0, True, 0)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_split_keeps_the_bits(H, scheme, recon, rs, char, limiter, dtype):
    """Boxes of 4 to 96 groups (16, 11 or 8, 5 and 2 workgroups per group):
    box step with and without fluxes and the ghosted-groups solve against the
    same launch with whole groups (one workgroup fewer than groups pinned)."""
    gamma, f64 = 1.4, dtype == torch.float64
    spec = H.make_spec(scheme, recon, rs, limiter, gamma=gamma, char=char, f64=f64)
    g = H.ghost_width(scheme, recon)
    kw = dict(dh=1 / 64, gamma=gamma, scheme=scheme, recon=recon, riemann=rs, limiter=limiter, char=char)
    try:
        for nx, ny, nz in ((32, 32, 16), (48, 48, 32), (48, 64, 64), (96, 64, 64)):
            # a blast and a near-vacuum corner: floors are hit and counted
            U = W.lognormal_blast_box(96, gamma=gamma, seed=nx + nz, radius_cells=4)[:, :nz, :ny, :nx].copy()
            U[:, :3, :3, :3] *= 1e-9
            B = torch.from_numpy(W.box_to_groups(U)).to(device="cuda", dtype=dtype)
            n = B.shape[0]
            dt = 0.3 * O.cfl_dt(U, 1 / 64, gamma, 0.3)
            dtd = torch.tensor([dt], dtype=torch.float64, device="cuda")
            G = H.fill_ghosts_periodic(B, g, grouped=True, shape=(nx, ny, nz))
            got = []
            for grid in (0, n - 1):
                H.set_launch_shape(spec, grid, 2 if f64 else 4)
                H.get_diag(reset=True)
                a, b, c = torch.empty_like(B), torch.empty_like(B), torch.empty_like(B)
                fb = torch.empty((n, 3, 3, 5, 16, 16), dtype=dtype, device="cuda")
                fg = torch.empty_like(fb)
                H.step_box(B, a, (nx, ny, nz), dtd, **kw)
                H.step_box(B, b, (nx, ny, nz), dtd, flux=fb, flux_mid=True, **kw)
                H.solve_groups(G, c, fg, dt=dt, flux_mid=True, **kw)
                got.append((a, b, c, fb, fg, H.get_diag(reset=True)))
            for x, y in zip(*got):
                assert torch.equal(x, y) if torch.is_tensor(x) else x == y, (nx, ny, nz)
            assert torch.equal(got[0][0], got[0][1])
            if f64:  # and the oracle: the FP64 bar of one step
                ref, _ = O.solve_groups(G.cpu().numpy(), g, dt, 1 / 64, gamma, scheme, recon, rs, limiter,
                                        O.F_CHAR if char else 0)
                assert scaled_max_err(got[0][2].cpu().numpy(), np.asarray(ref)) <= 1e-12
    finally:
        H.set_launch_shape(spec, 0, 2 if f64 else 4)
