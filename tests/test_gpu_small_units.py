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
