"""Domains of at most four rows, whose sweep runs smaller blocks: bitwise the
state of the large ones, and the FP64 oracle's."""
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


def _workload(shape, ncomp, c_ns):
    w = inputs.random_state(shape, 970, ncomp=ncomp, c_ns=c_ns, ns_choices=[0.0, 0.4, 1.0], rho_range=(0.3, 0.7))
    w.G, w.G_ads, w.F_ext = (0.7 if ncomp == 2 else 0.0), (0.2, -0.15), (2e-4, -1e-4, 3e-4)
    w.reservoirs = [(0, 0, 2, (0.6, 0.4))]
    return w


# one row whose neighbours are itself, two that are each other's, full and
# ragged last tiles, one plane
SHAPES = [(130, 4, 9), (65, 3, 1), (200, 1, 5), (7, 2, 40), (64, 4, 1), (128, 4, 6)]


@pytest.mark.parametrize("storage,ncomp,c_ns,forcing", [
    ("f64", 1, 1, "shan-chen"), ("f64", 2, 2, "guo"), ("f32", 1, 1, "guo"), ("f32", 2, 1, "shan-chen"),
    ("f32", 2, 2, "guo"), ("f16s", 1, 1, "shan-chen"), ("f16s", 2, 2, "guo"), ("bf16s", 2, 1, "shan-chen")])
def test_small_blocks_equal_large_ones_bitwise(monkeypatch, storage, ncomp, c_ns, forcing):
    def run(w, rounding, **env):
        for k in ("LBM_BOX", "LBM_TILE_X", "LBM_TILE_Y", "LBM_ZCHUNK"):
            monkeypatch.delenv(k, raising=False)
        for k, v in env.items():
            monkeypatch.setenv(k, str(v))
        sim = lbm.from_workload(w, storage=storage, forcing=forcing, rounding=rounding)
        sim.step(5)
        f = sim.populations()
        sim.close()
        return f

    big = dict(LBM_TILE_X=64, LBM_TILE_Y=4 if (storage, ncomp) == ("f64", 2) else 8)
    for shape in SHAPES:
        w = _workload(shape, ncomp, c_ns)
        for rounding in ((None, "nearest") if storage == "f16s" else (None,)):
            ref = run(w, rounding, **big)
            assert np.isfinite(ref).all()
            assert np.array_equal(run(w, rounding, LBM_BOX="0"), ref), shape  # the planned tile
            assert np.array_equal(run(w, rounding, LBM_TILE_X=33, LBM_TILE_Y=min(shape[1], 3), LBM_ZCHUNK=2), ref), shape


@pytest.mark.parametrize("ncomp", [1, 2])
@pytest.mark.parametrize("shape", [(130, 4, 9), (65, 3, 1), (40, 1, 7)])
def test_small_blocks_equal_the_oracle(monkeypatch, shape, ncomp):
    monkeypatch.setenv("LBM_BOX", "0")
    w = _workload(shape, ncomp, ncomp)
    o = oracle_for(w)
    sim = lbm.from_workload(w, storage="f64")
    sim.step(25)
    assert rel_max_err(sim.populations(), o.run(o.init(w.rho), 25)) <= 1e-10
    sim.close()
