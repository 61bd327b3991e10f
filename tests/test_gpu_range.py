"""Lengths whose squares come near the largest binary32 number."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def native():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1911_08275_amd import native
    native.lib()
    return native


@pytest.mark.parametrize("unit", [1.0, 1e10, 1e16, 1e18])
@pytest.mark.parametrize("ravg", [False, True])
@pytest.mark.parametrize("stat", ["xi", "wp"])
def test_long_lengths(native, stat, ravg, unit):
    """Binary32 calls in growing units (squares up to 4.2e37).  Two cells of
    6.55 along x; pairs across most of one, so that the frame's origin lies
    between them, and units of one record, which a group of four fills up."""
    from paper_1911_08275_amd import synth

    def cat(x, z):
        x, z = np.asarray(x) * unit, np.asarray(z) * unit
        return synth.Catalog(x, np.zeros_like(x), z, np.ones_like(x))

    x1, z1 = np.append(np.linspace(6.413, 6.547, 15), 13.2), np.linspace(0.0, 0.09, 16)
    x2, z2 = np.array([0.1]), np.array([0.045])
    edges = np.array([1.0, 6.32, 6.5])
    dx, dz = x1[:, None] - x2, z1[:, None] - z2
    s = np.sqrt(dx * dx + (dz * dz if stat == "xi" else 0.0)).ravel()
    want = np.histogram(s, edges)[0]
    assert np.abs(s[:, None] - edges).min() > 1e-4 and want.min() >= 1
    d1, d2 = native.to_device(cat(x1, z1)), native.to_device(cat(x2, z2))
    print("lengths", stat, ravg, unit, flush=True)
    opt = dict(precision="fp32", refine=(1, 1, 1), need_ravg=ravg)
    for a, b in ((d1, d2), (d2, d1)):
        g = (native.countpairs_cross(a, b, edges * unit, **opt) if stat == "xi" else
             native.countpairs_cross_wp(a, b, edges * unit, 2.0 * unit, 1, **opt))
        assert (g.npairs.ravel() == want).all()
        if ravg:
            mean = [s[(s >= lo) & (s < hi)].mean() for lo, hi in zip(edges, edges[1:])]
            np.testing.assert_allclose(g.ravg.ravel() / unit, mean, rtol=1e-12)
            assert (g.wsum.ravel() == want).all()
