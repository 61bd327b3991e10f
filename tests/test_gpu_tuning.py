"""What the launch settings of plans and calls are tuned on."""
import json

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


def test_wp_plan_tuned_as_it_runs(native, tmp_path, monkeypatch):
    """The trial calls of a w_p plan run its histogram per wave, so their last
    candidate has two waves per workgroup; a single w_p call always has four,
    and its settings say so."""
    from paper_1911_08275_amd import synth
    cache = tmp_path / "tune.json"
    monkeypatch.setenv("CP_AUTOTUNE", "1")
    monkeypatch.setenv("CP_AUTOTUNE_CACHE", str(cache))
    rng = np.random.Generator(np.random.PCG64(3))
    cat = synth.Catalog(*(rng.uniform(0.0, 60.0, 4000) for _ in range(3)))
    d, edges = native.to_device(cat), np.linspace(0.5, 6.0, 8)
    print("w_p plan tuning", flush=True)
    plan = native.Plan([d, d], wp_edges=edges, pimax=6.0, npibins=6, precision="fp32",
                       periodic=True, boxsize=60.0)
    assert native.last_stats()["waves"] == 2
    plan.execute()
    _, wp = plan.results()
    plan.close()
    g = native.countpairs_wp(d, edges, 6.0, 6, precision="fp32", periodic=True, boxsize=60.0)
    assert g.stats["tuned"] == "tuned" and g.stats["waves"] == 4
    assert (wp[0].ravel() == g.npairs.ravel()).all() and (wp[1] == wp[0]).all()
    text = json.loads(cache.read_text())
    single = [v for k, v in text.items() if k.startswith("wp/")]
    assert len(single) == 1 and single[0]["waves"] == 4, text
