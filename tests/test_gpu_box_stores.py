"""The box kernel's cached stores (states beyond the L2 caches): bitwise the
sweep's state."""
import numpy as np
import pytest

from paper_2206_11524_amd import inputs, lbm

pytestmark = pytest.mark.gpu


# each above the bound from which the box stores through the caches
@pytest.mark.parametrize("storage,forcing,ncomp,c_ns,shape", [
    ("f16s", "shan-chen", 2, 1, (57, 57, 57)), ("bf16s", "guo", 2, 2, (59, 60, 55)), ("f32", "shan-chen", 2, 2, (50, 51, 49)),
    ("f32", "guo", 2, 1, (46, 45, 47)), ("f64", "shan-chen", 2, 2, (42, 42, 42)), ("f64", "guo", 1, 1, (61, 50, 50)),
    ("f32", "shan-chen", 1, 1, (261, 65, 19))])
def test_cached_box_stores_equal_the_sweep_bitwise(monkeypatch, storage, forcing, ncomp, c_ns, shape):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    w = inputs.random_state(shape, 980, ncomp=ncomp, c_ns=c_ns, ns_choices=[0.0, 0.4, 1.0], rho_range=(0.3, 0.7))
    w.G, w.G_ads, w.F_ext = (0.7 if ncomp == 2 else 0.0), (0.2, -0.15), (2e-4, -1e-4, 3e-4)
    got = []
    for box in ("0", None):
        monkeypatch.setenv("LBM_BOX", box) if box else monkeypatch.delenv("LBM_BOX")
        sim = lbm.from_workload(w, storage=storage, forcing=forcing)
        sim.step(5)
        got.append(sim.populations())
        sim.close()
    assert np.isfinite(got[0]).all() and np.array_equal(*got)
