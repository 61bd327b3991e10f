"""Bins narrower than a thirty-second of an octave of the squared separation:
equal counts, and few pairs evaluated again in binary64."""
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


EDGES = {
    "far": np.linspace(5.0, 6.0, 41),
    "first": np.concatenate([[4.00, 4.02], np.linspace(4.5, 6.0, 4)]),
    "from_zero": np.concatenate([[0.0], np.linspace(5.2, 6.0, 30)]),
}


@pytest.mark.parametrize("name", sorted(EDGES))
@pytest.mark.parametrize("stat", ["xi", "wp", "fused"])
def test_narrow_bins(native, stat, name):
    """Uniform points: at most 1 pair in 100 lies within the binary32 error of
    an edge or pi bin (bounds of some 1e-5 of R_max^2 per edge, 41 edges)."""
    edges, box = EDGES[name], 31.0
    rng = np.random.Generator(np.random.PCG64(11))
    cat = synth.Catalog(*(rng.uniform(0.0, box, 6007) for _ in range(3)))
    d, opt = native.to_device(cat), dict(precision="fp32", periodic=True, boxsize=box,
                                         refine=(2, 2, 2))
    wp = oracle.wp(cat, edges, 6.0, 6, periodic=True, box=box).npairs
    xi = oracle.xi(cat, edges, periodic=True, box=box).npairs
    print("narrow", stat, name, flush=True)
    if stat == "fused":
        plan = native.Plan([d], xi_edges=edges, wp_edges=edges, pimax=6.0, npibins=6, **opt)
        plan.execute()
        px, pw = plan.results()
        st = plan.stats()[1]
        plan.close()
        assert (px[0] == xi).all() and (pw[0].reshape(wp.shape) == wp).all()
    else:
        g = (native.countpairs_xi(d, edges, **opt) if stat == "xi" else
             native.countpairs_wp(d, edges, 6.0, 6, **opt))
        ref = xi if stat == "xi" else wp
        assert (g.npairs.reshape(ref.shape) == ref).all()
        st = g.stats
    assert st["rechecks"] < 0.01 * st["candidates"]
