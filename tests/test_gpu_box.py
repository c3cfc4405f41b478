"""The box kernel of small domains: bitwise the sweep's state (every kernel
evaluates the same expressions per cell), and the FP64 oracle's."""
import numpy as np
import pytest

from paper_2206_11524_amd import inputs, lbm

from _common import oracle_for, rel_max_err

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    yield


def _workload(shape, ncomp, c_ns, seed=900):
    w = inputs.random_state(shape, seed, ncomp=ncomp, c_ns=c_ns, ns_choices=[0.0, 0.05, 0.4, 0.9, 1.0],
                            rho_range=(0.3, 0.7))
    w.tau = (0.8, 1.3)
    w.G, w.G_ads, w.F_ext = (0.7 if ncomp == 2 else 0.0), (0.2, -0.15), (2e-4, -1e-4, 3e-4)
    if shape[0] >= 4:  # slots along x and, where deep enough, z
        w.reservoirs = [(0, 1, 2, (0.6, 0.4))] + ([(2, shape[2] - 1, shape[2], (0.4, 0.6))] if shape[2] >= 4 else [])
    return w


# one cell; neighbours that wrap onto the cell itself; remainders on every
# axis; one plane; a row longer than a wave; boxes of the largest domains
SHAPES = [(1, 1, 1), (1, 20, 2), (2, 2, 2), (3, 5, 1), (7, 1, 3), (130, 3, 1), (17, 19, 23), (70, 13, 11),
          (33, 45, 71), (100, 90, 1)]


def _run(w, monkeypatch, box, steps, **kw):
    if box is None:
        monkeypatch.delenv("LBM_BOX", raising=False)
    else:
        monkeypatch.setenv("LBM_BOX", box)
    sim = lbm.from_workload(w, **kw)
    sim.step(steps)
    f = sim.populations()
    sim.close()
    return f


@pytest.mark.parametrize("forcing", ["shan-chen", "guo"])
@pytest.mark.parametrize("storage,rounding", [("f64", None), ("f32", None), ("f16s", "stochastic"),
                                              ("f16s", "nearest"), ("bf16s", "stochastic")])
def test_box_equals_the_sweep_bitwise(monkeypatch, storage, rounding, forcing):
    for shape in SHAPES:
        for ncomp, c_ns in ((1, 1), (2, 1), (2, 2)):
            w = _workload(shape, ncomp, c_ns)
            kw = dict(storage=storage, rounding=rounding, forcing=forcing)
            ref = _run(w, monkeypatch, "0", 5, **kw)
            assert np.array_equal(_run(w, monkeypatch, None, 5, **kw), ref), (shape, ncomp, c_ns)


@pytest.mark.parametrize("box", ["1,1,1", "4,3,2", "8,4,4", "13,5,3"])
def test_box_shape_does_not_change_results(monkeypatch, box):
    for storage, forcing in (("f64", "shan-chen"), ("f32", "guo"), ("f16s", "shan-chen")):
        w = _workload((37, 14, 9), 2, 2)
        ref = _run(w, monkeypatch, "0", 4, storage=storage, forcing=forcing)
        assert np.array_equal(_run(w, monkeypatch, box, 4, storage=storage, forcing=forcing), ref), storage


@pytest.mark.parametrize("shape", [(1, 20, 2), (17, 19, 23), (100, 30, 1)])
def test_box_equals_the_oracle(shape):
    w = _workload(shape, 2, 2)
    o = oracle_for(w)
    sim = lbm.from_workload(w, storage="f64")
    sim.step(25)
    assert rel_max_err(sim.populations(), o.run(o.init(w.rho), 25)) <= 1e-10
    sim.close()
