"""Refluxing and restriction in one launch against the oracle where patches
meet: every cell beside one, two or three refined patches, across the periodic
boundary, and boxes of two patches a side (a patch's both neighbours are one)."""
import numpy as np
import pytest

import oracle as O

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("n,count", [(16, 1), (16, 3), (16, 8), (32, 20), (48, 1), (48, 90), (64, 511)])
def test_correct_dense_patches(n, count, dtype):
    """FP64 bit for bit (same expressions in the same order); FP32 to the
    rounding of one FP32 store of the FP64 result (half an ulp of the scale)."""
    from paper_1103_3373_amd import hydro as H
    rng = np.random.default_rng(100 * n + count)
    ngf, gc = n // 8, (n // 16) ** 3
    at = rng.permutation(ngf ** 3)[:count]
    lay = np.stack([0 * at, 16 * (at % ngf), 16 * (at // ngf % ngf), 16 * (at // ngf ** 2)], 1).astype(np.int32)
    real = np.float64 if dtype == torch.float64 else np.float32
    def draw(*shape):
        return rng.standard_normal(shape).astype(real).astype(np.float64) + 3.0
    coarse, cflux = draw(gc, 5, 16, 16, 16), draw(gc, 3, 3, 5, 16, 16)
    fine, fflux = draw(count, 5, 16, 16, 16), draw(count, 3, 2, 5, 16, 16)
    if real is np.float32:
        coarse, cflux, fine, fflux = (a.astype(real).astype(np.float64) for a in (coarse, cflux, fine, fflux))
    dt, dh = 2e-3, 1.0 / n
    want = O.amr_correct(coarse, (n, n, n), cflux, fine, lay, fflux, dt, dh)
    dev = lambda a: torch.from_numpy(a).to(device="cuda", dtype=dtype)
    lay_d = torch.from_numpy(lay).cuda()
    got = dev(coarse)
    H.amr_correct(got, n, dev(cflux), dev(fine), lay_d, H.build_group_map(lay_d, ngf, 1), dev(fflux), dt, dh)
    got = got.cpu().numpy().astype(np.float64)
    if dtype == torch.float64:
        np.testing.assert_array_equal(got, want)
    else:
        assert np.abs(got - want).max() <= 2.0 ** -24 * np.abs(want).max()
