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


# edges and pi bins, and with them the copies of the histogram: many, and one
# (whose 256 lanes meet in every counter)
BINS = {"few": (EDGES, 4), "many": (np.linspace(0.5, 1.5, 21) + 1 / 64, 256)}


@pytest.mark.parametrize("bins", sorted(BINS))
@pytest.mark.parametrize("prec,ravg", [("fp32", False), ("fp64", False), ("fp32", True),
                                       ("fp64", True)])
def test_flush_while_others_add(native, bins, prec, ravg):
    """Every wave takes the totals of its workgroup's histogram several times
    (after each 2^22 records) while the other three add to it: counts, and sums
    of weights, that are exact in binary64.  Every term of the mean is 1/2 to
    5e-15 (the square root), and what a sum of such terms keeps of each is too:
    the means are 1 within 1e-12 many times over."""
    edges, npi = BINS[bins]
    n1 = 300
    parts = [((1 << 22) + 5, 1.06, 1.06), ((1 << 22) - 77, 0.69, 0.69), (4099, 1.31, 1.31),
             (1001, 0.9, 0.9)]
    d1 = _points(native, 0.0, [(n1, 1.0, 1.0)], w=2.0)
    d2 = _points(native, 1.0, parts + FAR, w=0.25)
    _say("flush", bins, prec, ravg)
    g = native.countpairs_cross_wp(d1, d2, edges, 0.5, npi, precision=prec, refine=(1, 1, 1),
                                   need_ravg=ravg)
    want = np.zeros((len(edges) - 1, npi), dtype=np.uint64)
    k = int(np.searchsorted(edges, 1.0, side="right")) - 1
    for n, z, _ in parts:
        want[k, int(abs(z - 1.0) / (0.5 / npi))] += np.uint64(n1 * n)
    assert (g.npairs == want).all()
    if ravg:
        assert (g.wsum == 0.5 * want.astype(np.float64)).all()
        np.testing.assert_allclose(g.ravg, (want > 0).astype(np.float64), rtol=1e-12)


@pytest.mark.parametrize("npi", [128, 256])
def test_plan_of_few_waves(native, npi):
    """A plan's w_p histogram per wave, 32 or 64 KB of it: workgroups of four
    and two waves."""
    import oracle
    from paper_1911_08275_amd import synth
    rng = np.random.Generator(np.random.PCG64(npi))
    edges = np.linspace(0.2, 6.0, 61)
    cats = [synth.Catalog(*(rng.uniform(0.0, 31.0, n) for _ in range(3))) for n in (700, 3001)]
    _say("plan waves", npi)
    plan = native.Plan([native.to_device(c) for c in cats], wp_edges=edges, pimax=6.0,
                       npibins=npi, precision="fp32", periodic=True, boxsize=31.0,
                       refine=(1, 1, 1))
    plan.execute()
    _, wp = plan.results()
    waves = plan.stats()[1]["waves"]
    plan.close()
    assert waves == 512 // npi
    for m, c in enumerate(cats):
        ref = oracle.wp(c, edges, 6.0, npi, periodic=True, box=31.0).npairs
        assert (wp[m].reshape(ref.shape) == ref).all(), m
