"""w_p histograms that overflow or are drained while a launch runs: cells of
many millions of points, whose counts are known without an oracle.  Counts are
whole numbers, so the tolerance is equality."""
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


def _say(*a):
    print(*a, flush=True)


def _points(native, x, parts, dtype=None, w=None):
    """Points at x with z uniform over each part (n, z0, z1) in turn."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(7)
    z = torch.cat([z0 + (z1 - z0) * torch.rand(n, generator=g, device="cuda",
                                               dtype=dtype or torch.float64)
                   for n, z0, z1 in parts])
    ww = None if w is None else torch.full(z.shape, w, device="cuda", dtype=torch.float64)
    return native.DevicePoints(torch.full_like(z, x), torch.zeros_like(z), z, ww)


# One column of z-cells of 0.5 (pi_max 0.5, refine 1), r_p = 1 for every pair;
# the points at 0 and 2.5 are out of reach and fix the grid.
FAR = [(1, 0.0, 0.0), (1, 2.5, 2.5)]
BIG, NEXT = (0.9, 1.2), (1.3, 1.35)      # two neighbouring cells, all within pi_max of SET1
SET1 = [(256, 1.0, 1.1)]                 # four tiles: the four waves of one workgroup
EDGES = np.array([0.5, 1.5])


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_one_bin_beyond_32_bits(native, prec):
    """Four waves put 256 x 2e7 pairs into one counter's copies before the
    first of them takes the totals (at its second cell)."""
    big, nxt = 20_000_000, 100
    d1 = _points(native, 0.0, SET1)
    d2 = _points(native, 1.0, [(big,) + BIG, (nxt,) + NEXT] + FAR)
    _say("one bin", prec)
    g = native.countpairs_cross_wp(d1, d2, EDGES, 0.5, 1, precision=prec, refine=(1, 1, 1))
    assert int(g.npairs.sum()) == 256 * (big + nxt)


def test_one_copy_beyond_32_bits(native):
    """256 pi bins and four copies of the histogram: 64 lanes add the records
    of one cell of more than 2^26 points to the same copy of one counter."""
    import torch
    big, nxt = (1 << 26) + (1 << 20), 100
    d1 = _points(native, 0.0, [(256, 1.0, 1.0)], torch.float32)
    d2 = _points(native, 1.0, [(big, 0.951, 0.951), (nxt,) + NEXT] + FAR, torch.float32)
    edges = np.array([0.2, 0.3, 0.4, 0.5, 1.5])
    _say("one copy", big)
    g = native.countpairs_cross_wp(d1, d2, edges, 0.5, 256, precision="fp32", refine=(1, 1, 1))
    dz = 1.0 - float(np.float32(0.951))
    assert int(g.npairs[3, int(dz / (0.5 / 256))]) == 256 * big
    assert int(g.npairs.sum()) == 256 * (big + nxt)
    assert g.stats["cell_pairs"] == 8   # a cut unit counts once
