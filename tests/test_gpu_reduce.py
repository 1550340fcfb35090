"""Time step and conserved sums: ragged numbers of groups, arrays off the
16-byte grid, special values and graph replays, against IEEE evaluations in
numpy (the time step bit for bit)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
GAMMA, CFL, DH = 1.4, 0.5, 1 / 48


@pytest.fixture(scope="module")
def H():
    from paper_1103_3373_amd import hydro
    hydro.lib()
    return hydro


def _state(n, dtype, seed):
    rng = np.random.default_rng(seed)
    U = np.empty((n, 5, 16, 16, 16))
    U[:, 0] = rng.lognormal(0.0, 1.0, U[:, 0].shape)
    U[:, 1:4] = rng.standard_normal(U[:, 1:4].shape) * U[:, :1]
    U[:, 4] = rng.lognormal(0.0, 1.0, U[:, 0].shape) + 0.5 * (U[:, 1:4] ** 2).sum(1) / U[:, 0]
    return U.astype(np.float32 if dtype == torch.float32 else np.float64)


def _want_dt(U):
    """The same expressions in numpy: correctly rounded, no contraction; NaN speeds never win."""
    with np.errstate(all="ignore"):
        r, x, y, z, e = (U[:, k].astype(np.float64) for k in range(5))
        vx, vy, vz = x / r, y / r, z / r
        p = (GAMMA - 1.0) * (e - 0.5 * (x * vx + y * vy + z * vz))
        c = np.sqrt(GAMMA * p / r)
        av = np.abs(vx)
        for v in (np.abs(vy), np.abs(vz)):
            av = np.where(v > av, v, av)
        s = av + c
        m = np.max(np.where(s > 0, s, 0.0))
        return CFL * DH / m


@pytest.mark.parametrize("n", [1, 3, 31, 128, 129, 511, 513, 2047, 2048, 2101])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("shift", [0, 1])
def test_dt_and_sums(H, n, dtype, shift):
    U = _state(n, dtype, n)
    buf = torch.empty(U.size + 4, dtype=dtype, device="cuda")
    D = buf[shift:shift + U.size].view(U.shape)
    D.copy_(torch.from_numpy(U))
    dt, sums = H.cfl_dt_sums(D, DH, GAMMA, CFL)
    dt1, s1 = H.cfl_dt(D, DH, GAMMA, CFL), H.conserved_sums(D, DH)
    dtb = torch.empty(1, dtype=torch.float64, device="cuda")
    table = H.seg_table([(D, D, None, dtb, 1.0, DH, 0, n)], "cuda")
    H.cfl_dt_batch(table, 1, n, gamma=GAMMA, cfl=CFL, f64=dtype == torch.float64)
    want = _want_dt(U)
    assert dt.item() == dt1.item() == dtb.item() == want
    assert torch.equal(sums, s1)
    exact, scale = U.astype(np.float64).sum((0, 2, 3, 4)), np.abs(U.astype(np.float64)).sum((0, 2, 3, 4))
    # partial sums in a tree: a few hundred roundings of at most 2^-53 of the sum of magnitudes
    assert np.all(np.abs(sums.cpu().numpy() / DH ** 3 - exact) <= 1e-13 * scale)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_dt_special_values(H, dtype):
    """Zero and tiny densities, negative pressures, zero momenta, infinities and NaN: as IEEE arithmetic has them."""
    tiny = np.finfo(np.float32 if dtype == torch.float32 else np.float64).tiny
    cells = [(1.0, 0.0, -0.0, 0.0, 2.5), (1.0, 3.0, 0.0, 0.0, 1.0), (0.0, 0.0, 0.0, 0.0, 1.0), (np.nan, 1, 1, 1, 9),
             (1.0, 1.0, 1.0, 1.0, np.nan), (tiny, 0.0, 0.0, 0.0, tiny), (-1.0, 1.0, 0.0, 0.0, 2.0),
             (np.inf, 1.0, 1.0, 1.0, 1.0), (1.0, 0.0, 0.0, 0.0, 0.0)]
    for k, cell in enumerate(cells + [(0.0, 1.0, 0.0, 0.0, 1.0), (1.0, 0.0, 0.0, 0.0, np.inf)]):
        U = np.broadcast_to(np.array([1.0, 0.1, 0.0, 0.0, 1.5])[None, :, None, None, None], (2, 5, 16, 16, 16)).copy()
        U[1, :, 3, 4, 5] = cell
        D = torch.from_numpy(U).to(device="cuda", dtype=dtype)
        assert H.cfl_dt(D, DH, GAMMA, CFL).item() == _want_dt(D.cpu().numpy()), (k, cell)


def test_counters_wrap_over_calls_and_replays(H):
    """Alternating sizes, more calls than counter sets, and a graph of two reductions replayed between eager calls."""
    states = [torch.from_numpy(_state(n, torch.float32, 9 + n)).cuda() for n in (1, 5, 200, 600)]
    want = [(H.cfl_dt(D, DH, GAMMA, CFL).item(), H.conserved_sums(D, DH)) for D in states]
    for q in range(80):
        D, (dt, sums) = states[q % 4], want[q % 4]
        a, b = H.cfl_dt_sums(D, DH, GAMMA, CFL)
        assert a.item() == dt and torch.equal(b, sums), q
    a, b = torch.empty(1, dtype=torch.float64, device="cuda"), torch.empty(5, dtype=torch.float64, device="cuda")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        H.cfl_dt(states[2], DH, GAMMA, CFL, dt_out=a)
        H.cfl_dt_sums(states[3], DH, GAMMA, CFL, dt_out=a, sums_out=b)
    for q in range(5):
        a.zero_(), b.zero_()
        graph.replay()
        assert a.item() == want[3][0] and torch.equal(b, want[3][1])
        assert H.cfl_dt(states[q % 4], DH, GAMMA, CFL).item() == want[q % 4][0]
