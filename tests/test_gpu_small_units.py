"""w_p units of a few records (counted one by one) and just more (in groups of
four), alone and with xi in one launch, against the CPU oracle.  Counts are
whole numbers: equality."""
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


def _cells(per, seed):
    """per points in each cell of side 3 of a box of 30, half of the
    coordinates on a lattice of 1/4 (separations on edges and on pi bins)."""
    rng = np.random.Generator(np.random.PCG64(seed))
    g = np.stack(np.meshgrid(*[np.arange(10.0) * 3.0] * 3, indexing="ij"), -1).reshape(-1, 1, 3)
    u = rng.uniform(0.0, 3.0, (len(g), per, 3))
    q = np.floor(u * 4) / 4
    p = (g + np.where(rng.random(u.shape) < 0.5, q, u)).reshape(-1, 3)
    return synth.Catalog(*(np.ascontiguousarray(p[:, a]) for a in range(3)))


@pytest.mark.parametrize("per", [1, 3, 4, 7, 8, 9])
@pytest.mark.parametrize("name,edges", [("two", np.array([0.5, 3.0])),
                                        ("eight", np.linspace(0.0, 3.0, 9))])
def test_units_around_the_limit(native, per, name, edges):
    cat = _cells(per, per)
    d, opt = native.to_device(cat), dict(precision="fp32", periodic=True, boxsize=30.0)
    wp = oracle.wp(cat, edges, 3.0, 3, periodic=True, box=30.0).npairs
    xi = oracle.xi(cat, edges, periodic=True, box=30.0).npairs
    for noprune in (False, True):
        print("small units", name, per, noprune, flush=True)
        g = native.countpairs_wp(d, edges, 3.0, 3, refine=(1, 1, 1), no_prune=noprune, **opt)
        assert (g.npairs.reshape(wp.shape) == wp).all()
        plan = native.Plan([d, d], xi_edges=edges, wp_edges=edges, pimax=3.0, npibins=3,
                           refine=(1, 1, 1), no_prune=noprune, **opt)
        plan.execute()
        px, pw = plan.results()
        plan.close()
        for m in range(2):
            assert (pw[m].reshape(wp.shape) == wp).all() and (px[m] == xi).all()


@pytest.mark.parametrize("edges", [np.array([0.5, 6.0]), np.linspace(0.25, 6.0, 11),
                                   np.array([0.5, 2.0, 2.0 + 1e-7, 3.0, 5.75, 6.0])])
@pytest.mark.parametrize("refine", [(1, 1, 1), (3, 3, 2), (2, 2, 8)])
@pytest.mark.parametrize("n", [4500, 7000])
def test_fused_by_density(native, n, refine, edges):
    """w_p and xi in one launch on either side of the density that picks its
    kernel (6 100 points here): xi edges as the r_p edges, fewer and more."""
    box, rng = 18.5, np.random.Generator(np.random.PCG64(n))
    cats = []
    for m in (n, 700, 5):
        p = rng.uniform(0.0, box, (m, 3))
        p[::2] = rng.integers(0, int(4 * box), p[::2].shape) * 0.25
        cats.append(synth.Catalog(*(np.ascontiguousarray(p[:, a]) for a in range(3))))
    devs = [native.to_device(c) for c in cats]
    for xe in (edges, np.array([0.25, 0.5, 2.5]), np.linspace(0.5, 6.0, 23)):
        print("fused", n, refine, len(edges), len(xe), flush=True)
        plan = native.Plan(devs, xi_edges=xe, wp_edges=edges, pimax=6.0, npibins=6,
                           precision="fp32", periodic=True, boxsize=box, refine=refine)
        for _ in range(2):
            plan.execute()
            xi, wp = plan.results()
            for m, c in enumerate(cats):
                rw = oracle.wp(c, edges, 6.0, 6, periodic=True, box=box).npairs
                assert (wp[m].reshape(rw.shape) == rw).all(), m
                assert (xi[m] == oracle.xi(c, xe, periodic=True, box=box).npairs).all(), m
        plan.close()
