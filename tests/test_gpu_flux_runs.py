"""Box steps that store face fluxes march through runs of z-consecutive groups
like those that do not: the fluxes of every group of a run against one group
per run and the oracle."""
import numpy as np
import pytest

import oracle as O
from paper_1103_3373_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _max_rel(a, b, axis):
    """max |a - b| over max |b|, per variable along `axis`."""
    a = a.double().movedim(axis, 0).reshape(5, -1)
    b = b.double().movedim(axis, 0).reshape(5, -1)
    return ((a - b).abs().max(1).values / b.abs().max(1).values).max().item()


@pytest.mark.parametrize("scheme,recon,rs", [(2, 1, 1), (2, 1, 0), (2, 0, 1), (0, 1, 1), (0, 1, 0), (1, 1, 1)])
@pytest.mark.parametrize("mid", [False, True])
def test_flux_of_runs(scheme, recon, rs, mid):
    """Runs of 2 and 4 groups, several items per workgroup and one: updated
    cells and fluxes agree with one group per run to the FP32 parity bar (1e-5
    of each variable's maximum, per face direction), the updated cells are
    those of the same run without fluxes to the same bar, an inner face of a
    run is the same number in both groups that share it, and the grid changes
    nothing."""
    from paper_1103_3373_amd import hydro as H
    gamma, nx, ny, nz = 1.4, 32, 16, 128
    box = W.lognormal_blast_box(128, gamma=gamma, seed=41, radius_cells=4)[:, :nz, :ny, :nx].copy()
    B = torch.from_numpy(W.box_to_groups(box)).to(device="cuda", dtype=torch.float32)
    dt = O.cfl_dt(box, 1 / 128, gamma, 0.3)
    dtd = torch.tensor([dt], dtype=torch.float64, device="cuda")
    spec = H.make_spec(scheme, recon, rs, H.VANLEER, gamma=gamma, char=True)
    kw = dict(dh=1 / 128, gamma=gamma, scheme=scheme, recon=recon, riemann=rs, char=True)
    nf, per = (3 if mid else 2), (nx // 16) * (ny // 16)

    def step(zrun, grid, flux):
        H.set_launch_shape(spec, grid, 4, zrun)
        assert H.get_launch_shape(spec, (nx, ny, nz))[2] == zrun
        out = torch.full_like(B, float("nan"))
        F = torch.full((B.shape[0], 3, nf, 5, 16, 16), float("nan"), device="cuda") if flux else None
        H.step_box(B, out, (nx, ny, nz), dtd, flux=F, flux_mid=mid, **kw)
        return out, F

    try:
        ref, fref = step(1, 0, True)
        for zrun in (2, 4):
            out, F = step(zrun, 0, True)
            assert torch.isfinite(out).all() and torch.isfinite(F).all()
            assert _max_rel(out, ref, 1) <= 1e-5
            for d in range(3):
                assert _max_rel(F[:, d], fref[:, d], 2) <= 1e-5, (zrun, d)
            assert _max_rel(step(zrun, 0, False)[0], out, 1) <= 1e-5
            z = np.arange(B.shape[0]) // per
            inner = np.nonzero((z + 1) % zrun != 0)[0]
            assert torch.equal(F[inner, 2, 1], F[inner + per, 2, 0])
            o2, f2 = step(zrun, 3, True)
            assert torch.equal(o2, out) and torch.equal(f2, F)
    finally:
        H.set_launch_shape(spec, 0, 4)
