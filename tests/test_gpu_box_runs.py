"""Results of the box kernel on domains and boxes that are known to run it
(_box_cases.py), and of the sweeps, which it has taken small domains from, against
the FP64 oracle."""
import numpy as np
import pytest

from paper_2206_11524_amd import inputs, lbm

import _box_cases
from _common import oracle_for, rel_max_err

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    yield


def _workload(shape, ncomp, c_ns):
    w = inputs.random_state(shape, 985, ncomp=ncomp, c_ns=c_ns, ns_choices=[0.0, 0.05, 0.4, 0.9, 1.0],
                            rho_range=(0.3, 0.7))
    w.tau = (0.8, 1.3)
    w.G, w.G_ads, w.F_ext = (0.7 if ncomp == 2 else 0.0), (0.2, -0.15), (2e-4, -1e-4, 3e-4)
    if shape[0] >= 4:
        w.reservoirs = [(0, 1, 2, (0.6, 0.4))] + ([(2, shape[2] - 1, shape[2], (0.4, 0.6))] if shape[2] >= 4 else [])
    return w


@pytest.mark.parametrize("fmt", _box_cases.CASES, ids=lambda f: "-".join(map(str, f)))
def test_box_equals_the_sweep_bitwise(monkeypatch, fmt):
    storage, ncomp, c_ns, forcing = fmt

    def run(w, box):
        monkeypatch.setenv("LBM_BOX", box) if box else monkeypatch.delenv("LBM_BOX", raising=False)
        sim = lbm.from_workload(w, storage=storage, forcing=forcing)
        sim.step(4)
        f = sim.populations()
        sim.close()
        return f

    shapes, boxes = _box_cases.CASES[fmt]
    for shape in shapes:
        w = _workload(shape, ncomp, c_ns)
        assert np.array_equal(run(w, None), run(w, "0")), shape
    w = _workload(_box_cases.BOXED, ncomp, c_ns)
    ref = run(w, "0")
    assert np.isfinite(ref).all()
    for box in boxes:
        assert np.array_equal(run(w, "%d,%d,%d" % box), ref), box


@pytest.mark.parametrize("forcing", ["shan-chen", "guo"])
@pytest.mark.parametrize("ncomp,c_ns", [(1, 1), (2, 1), (2, 2)])
@pytest.mark.parametrize("shape", [(1, 20, 2), (17, 19, 23), (70, 13, 11), (100, 30, 1), (130, 3, 6)])
def test_sweep_equals_the_oracle(monkeypatch, shape, ncomp, c_ns, forcing):
    """FP64 to 1e-10; the densities in FP32 to 1e-4, the bar of its parity."""
    monkeypatch.setenv("LBM_BOX", "0")
    w = _workload(shape, ncomp, c_ns)
    o = oracle_for(w, forcing=forcing)
    f = o.run(o.init(w.rho), 20)
    for storage in ("f64", "f32"):
        sim = lbm.from_workload(w, storage=storage, forcing=forcing)
        sim.step(20)
        if storage == "f64":
            assert rel_max_err(sim.populations(), f) <= 1e-10
        else:
            assert rel_max_err(sim.populations().sum(axis=1), f.sum(axis=1)) <= 1e-4
        sim.close()
