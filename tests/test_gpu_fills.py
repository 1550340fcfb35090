"""Ghost fills at the edges of their launch rules: few and many groups, outputs
off the 16-byte grid, and coarse fields that are staged in LDS as a whole, a
layer at a time, or read directly."""
import numpy as np
import pytest

import oracle as O
from paper_1103_3373_amd import workloads as W
from tests._util import scaled_max_err

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def H():
    from paper_1103_3373_amd import hydro
    hydro.lib()
    return hydro


def _out(n, N, dtype, shift):
    size = n * 5 * N ** 3
    buf = torch.full((size + 4,), float("nan"), dtype=dtype, device="cuda")
    return buf, buf[shift:shift + size].view(n, 5, N, N, N)


@pytest.mark.parametrize("shape", [(16, 16, 16), (48, 48, 112), (64, 64, 64), (80, 64, 208)])  # 1, 63, 64, 260 groups
@pytest.mark.parametrize("g", [0, 1, 2, 3, 4, 7])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_periodic_fill(H, shape, g, dtype):
    nx, ny, nz = shape
    rng = np.random.default_rng(nx + g)
    box = rng.standard_normal((5, nz, ny, nx)).astype(np.float32 if dtype == torch.float32 else np.float64)
    want = O.fill_ghosts_periodic(box.astype(np.float64), g)
    for shift in (0, 1, 3):
        buf, out = _out(want.shape[0], 16 + 2 * g, dtype, shift)
        H.fill_ghosts_periodic(torch.from_numpy(box).cuda(), g, out=out)
        np.testing.assert_array_equal(out.double().cpu().numpy(), want)
        grouped = torch.from_numpy(W.box_to_groups(box)).cuda()
        out.fill_(float("nan"))
        H.fill_ghosts_periodic(grouped, g, out=out, grouped=True, shape=shape)
        np.testing.assert_array_equal(out.double().cpu().numpy(), want)
        edge = torch.cat([buf[:shift], buf[shift + out.numel():]])
        assert torch.isnan(edge).all()  # nothing beside it was written


# (ng0, level counts, coarse size): the coarse field coarser than every level (staged as a whole), as fine as level 0
# and half as fine as level 1 (layers), and finer than level 0 (read directly); 5 to 1,001 groups.
CASES = [(2, (1, 1, 3), 6), (2, (8, 20, 100), 32), (4, (20, 40, 69), 16), (2, (6, 40, 200), 96), (4, (60, 440, 501), 64)]


@pytest.mark.parametrize("ng0,counts,cn", CASES)
@pytest.mark.parametrize("g", [0, 2, 3, 4])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_amr_fill(H, ng0, counts, cn, g, dtype):
    rng = np.random.default_rng(cn + g)
    lay = W.amr_layout(counts, base_n=16 * ng0, seed=cn)
    lay = lay[rng.permutation(len(lay))]
    real = np.float32 if dtype == torch.float32 else np.float64
    fine = rng.standard_normal((len(lay), 5, 16, 16, 16)).astype(real)
    c0, c1 = (rng.standard_normal((5, cn, cn, cn)).astype(real) for _ in range(2))
    alpha = [0.25, 1.0, 0.625]
    want = O.fill_groups_amr(fine.astype(np.float64), lay, ng0, alpha, c0.astype(np.float64), c1.astype(np.float64), g)
    lay_d = torch.from_numpy(np.ascontiguousarray(lay)).cuda()
    gmap = H.build_group_map(lay_d, ng0, 3)
    got = []
    for shift in (0, 1):
        buf, out = _out(len(lay), 16 + 2 * g, dtype, shift)
        H.fill_groups_amr(torch.from_numpy(fine).cuda(), lay_d, gmap, ng0, alpha, torch.from_numpy(c0).cuda(),
                          torch.from_numpy(c1).cuda(), g, out=out)
        got.append(out.clone())
        assert torch.isnan(torch.cat([buf[:shift], buf[shift + out.numel():]])).all()
    assert torch.equal(got[0], got[1])
    # the oracle sums eight weighted corners, the kernel interpolates axis by axis: a few roundings; FP32 rounds once
    bar = 2e-7 if dtype == torch.float32 else 2e-15
    assert scaled_max_err(got[0].double().cpu().numpy(), want) <= bar
    N = 16 + 2 * g
    inner = (slice(None), slice(None)) + (slice(g, N - g),) * 3
    np.testing.assert_array_equal(got[0].double().cpu().numpy()[inner], fine.astype(np.float64))
