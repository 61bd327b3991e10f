"""Pair-kernel loops at the sizes where each can go wrong, against the CPU
FP64 oracle.  All results are whole numbers, so the tolerance is equality."""
import numpy as np
import pytest

import oracle
from paper_1911_08275_amd import synth

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


def _cloud(n, box, seed):
    """Half uniform points, half on a lattice of spacing 1/4 (separations on
    the edges and on integer line-of-sight bins), some of them doubled."""
    rng = np.random.Generator(np.random.PCG64(seed))
    u = rng.uniform(0, box, (n - n // 2, 3))
    k = rng.integers(0, int(4 * box), (n // 2, 3)) * 0.25
    k[: len(k) // 8] = k[-(len(k) // 8):] if len(k) >= 8 else k[:0]
    p = np.concatenate([u, k], 0)
    return synth.Catalog(*(np.ascontiguousarray(p[:, a]) for a in range(3)))


# edge sets: one slot and two-edge units only; few; more than any unit's few;
# two edges closer than the binary32 error; a first bin that starts at zero
EDGES = {
    "one_bin": np.array([0.5, 6.0]),
    "from_zero": np.array([0.0, 1.0, 2.5, 6.0]),
    "ten": np.linspace(0.25, 6.0, 11),
    "sixty": np.linspace(0.1, 6.0, 61),
    "close": np.array([0.5, 2.0, 2.0 + 1e-7, 3.0, 5.75, 5.75 * (1 + 1e-9), 6.0]),
}


@pytest.mark.parametrize("name", sorted(EDGES))
@pytest.mark.parametrize("n,refine", [(37, (1, 1, 1)), (3001, (1, 1, 1)), (6007, (3, 3, 2))])
def test_wp_loops(native, name, n, refine):
    """Units of every slot count (table and one to three edges), 1 to many
    records, own cells, r_p and pi ties, pruned and not."""
    edges, box = EDGES[name], 31.0
    cat = _cloud(n, box, 5)
    ref = oracle.wp(cat, edges, 6.0, 6, periodic=True, box=box)
    d = native.to_device(cat)
    for noprune in (False, True):
        _say("wp loops", name, n, refine, noprune)
        g = native.countpairs_wp(d, edges, 6.0, 6, precision="fp32", periodic=True, boxsize=box,
                                 refine=refine, no_prune=noprune)
        assert (g.npairs.reshape(ref.npairs.shape) == ref.npairs).all()
        assert g.stats["precision"] == "fp32"
    if n > 3000:
        assert g.stats["rechecks"] > 0


@pytest.mark.parametrize("name", sorted(EDGES))
@pytest.mark.parametrize("n,refine", [(37, (1, 1, 1)), (3001, (1, 1, 1)), (6007, (3, 3, 2))])
def test_xi_loops(native, name, n, refine):
    """Units counted at once, by one to three edges and by the table; 1 to
    many records, own cells, ties, pruned and not; both precisions (their
    counters have one column per pair of lanes)."""
    edges, box = EDGES[name], 31.0
    cat = _cloud(n, box, 6)
    ref = oracle.xi(cat, edges, periodic=True, box=box)
    d = native.to_device(cat)
    for prec in ("fp64", "fp32"):
        for noprune in (False, True):
            _say("xi loops", name, n, refine, prec, noprune)
            g = native.countpairs_xi(d, edges, precision=prec, periodic=True, boxsize=box,
                                     refine=refine, no_prune=noprune)
            assert (g.npairs == ref.npairs).all()
            assert g.stats["precision"] == prec
    if n > 3000:
        assert g.stats["rechecks"] > 0


@pytest.mark.parametrize("name", sorted(EDGES))
@pytest.mark.parametrize("refine", [(1, 1, 1), (3, 3, 2)])
def test_fused_loops(native, name, refine):
    """w_p and xi in one launch, the xi edges reaching less far than, as far
    as and with other slot counts than the r_p edges."""
    edges, box = EDGES[name], 31.0
    cats = [_cloud(n, box, 9 + n) for n in (63, 3001, 4500)]
    devs = [native.to_device(c) for c in cats]
    for xe in (edges, np.array([0.25, 0.5, 2.5]), np.linspace(0.5, 6.0, 23)):
        _say("fused loops", name, refine, len(xe))
        plan = native.Plan(devs, xi_edges=xe, wp_edges=edges, pimax=6.0, npibins=6,
                           precision="fp32", periodic=True, boxsize=box, refine=refine)
        plan.execute()
        xi, wp = plan.results()
        plan.close()
        for m, c in enumerate(cats):
            rw = oracle.wp(c, edges, 6.0, 6, periodic=True, box=box).npairs
            assert (wp[m].reshape(rw.shape) == rw).all(), m
            assert (xi[m] == oracle.xi(c, xe, periodic=True, box=box).npairs).all(), m


@pytest.mark.parametrize("mode", ["xi", "wp"])
@pytest.mark.parametrize("n", [1, 2, 64, 65, 129, 4097, 40_000])
def test_launch_sizes(native, mode, n):
    """From one tile to more tiles than waves: workgroups without items, part
    of their waves with items, items by position and from the queues, the end
    totals of a workgroup; weighted (sums within 1e-12, the accumulation error
    of under 2^20 binary64 additions) and not."""
    rng = np.random.Generator(np.random.PCG64(n))
    cat = _cloud(n, 60.0, 3)
    cat = synth.Catalog(cat.x, cat.y, cat.z, rng.uniform(0.5, 1.5, n))
    edges = np.linspace(0.5, 6.0, 8)
    d = native.to_device(cat)
    ref = (oracle.xi(cat, edges, periodic=True, box=60.0) if mode == "xi"
           else oracle.wp(cat, edges, 6.0, 5, periodic=True, box=60.0))
    for prec in ("fp64", "fp32"):
        for ravg in (False, True):
            _say("launch sizes", mode, n, prec, ravg)
            opt = dict(precision=prec, periodic=True, boxsize=60.0, refine=(3, 3, 3), need_ravg=ravg)
            g = (native.countpairs_xi(d, edges, **opt) if mode == "xi"
                 else native.countpairs_wp(d, edges, 6.0, 5, **opt))
            assert (g.npairs.reshape(ref.npairs.shape) == ref.npairs).all()
            if ravg:
                np.testing.assert_allclose(g.wsum.reshape(ref.wsum.shape), ref.wsum, rtol=1e-12)
                np.testing.assert_allclose(g.ravg.reshape(ref.ravg.shape), ref.ravg, rtol=1e-12)


@pytest.mark.parametrize("n", [1, 63, 1025, 262_145, 1_048_579])
def test_bounding_box(native, n):
    """The joint bounding box of a non-periodic call around its loads (a
    point per thread, four per thread, one more): the last point of either set
    alone holds an extreme, and its partner sits beside it."""
    rng = np.random.Generator(np.random.PCG64(n))
    p = rng.uniform(0.0, 60.0, (n, 3))
    q = rng.uniform(0.0, 60.0, (9, 3))
    p[-1] = (200.0, -90.0, 300.0)
    q[0] = (200.5, -90.25, 300.0)
    q[-1] = (-150.0, 170.0, -80.0)
    p[0] = (-150.0, 170.0, -79.5) if n > 1 else p[0]
    A, B = (synth.Catalog(*(np.ascontiguousarray(v[:, a]) for a in range(3))) for v in (q, p))
    edges = np.array([0.25, 1.0, 2.0, 4.0])
    ref = oracle.xi(A, edges, periodic=False, other=B)
    assert ref.npairs[0] >= (2 if n > 1 else 1)
    for prec in ("fp64", "fp32"):
        _say("bounding box", n, prec)
        for a, b in ((A, B), (B, A)):
            g = native.countpairs_cross(native.to_device(a), native.to_device(b), edges,
                                        precision=prec, periodic=False)
            assert (g.npairs == ref.npairs).all()
