"""The sweeps' run-time tiles and both store policies: bitwise the state of
64-wide tiles, alone and in a group, on domains whose rows and columns leave
remainders."""
import numpy as np
import pytest

from paper_2206_11524_amd import inputs, lbm

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    yield


def _workload(shape, c_ns, ncomp=2):
    w = inputs.random_state(shape, 950, ncomp=ncomp, c_ns=c_ns, ns_choices=[0.0, 0.4, 1.0], rho_range=(0.3, 0.7))
    w.G, w.G_ads, w.F_ext = (0.7 if ncomp == 2 else 0.0), (0.2, -0.15), (2e-4, -1e-4, 3e-4)
    w.reservoirs = [(0, 0, 2, (0.6, 0.4)), (2, shape[2] - 1, shape[2], (0.4, 0.6))]
    return w


def _run(w, monkeypatch, env, **kw):
    for k in ("LBM_BOX", "LBM_TILE_X", "LBM_TILE_Y", "LBM_ZCHUNK"):
        monkeypatch.delenv(k, raising=False)
    for k, v in env.items():
        monkeypatch.setenv(k, str(v))
    sim = lbm.from_workload(w, **kw)
    sim.step(5)
    f = sim.populations()
    sim.close()
    return f


# widths below, at and above 32 and 64; a one-cell and a two-cell last column;
# nx a multiple of a 128-byte line (non-temporal stores) and not (cached)
@pytest.mark.parametrize("storage,forcing", [("f16s", "shan-chen"), ("bf16s", "guo"), ("f32", "shan-chen")])
@pytest.mark.parametrize("shape", [(33, 17, 9), (64, 16, 6), (65, 31, 7), (130, 9, 11), (128, 24, 5)])
def test_tile_does_not_change_results(monkeypatch, storage, forcing, shape):
    for c_ns in (1, 2):
        w = _workload(shape, c_ns)
        kw = dict(storage=storage, forcing=forcing)
        ref = _run(w, monkeypatch, dict(LBM_TILE_X=64, LBM_TILE_Y=8), **kw)
        assert np.isfinite(ref).all()
        assert np.array_equal(_run(w, monkeypatch, dict(LBM_BOX="0"), **kw), ref)  # the planned tile
        for tx, ty, zc in ((32, 16, 2), (33, 15, 3), (64, 1, 1), (5, 16, 4), (44, 11, shape[2])):
            f = _run(w, monkeypatch, dict(LBM_TILE_X=tx, LBM_TILE_Y=ty, LBM_ZCHUNK=zc), **kw)
            assert np.array_equal(f, ref), (c_ns, tx, ty)


# the split layout: FP64 (tiles of 256 cells in at most five rows), the GS-WBS in
# FP32 (ten rows, eight with two n_s fields), one component (sixteen rows)
@pytest.mark.parametrize("storage,forcing,ncomp,rows", [("f64", "shan-chen", 2, 5), ("f64", "guo", 2, 5),
                                                        ("f32", "guo", 2, 8), ("f32", "shan-chen", 1, 16),
                                                        ("f16s", "shan-chen", 1, 16), ("f64", "guo", 1, 16)])
@pytest.mark.parametrize("shape", [(33, 17, 9), (65, 31, 7), (130, 9, 11), (128, 24, 5)])
def test_split_tile_does_not_change_results(monkeypatch, storage, forcing, ncomp, rows, shape):
    for c_ns in (1, 2)[:ncomp]:
        w = _workload(shape, c_ns, ncomp)
        kw = dict(storage=storage, forcing=forcing)
        ref = _run(w, monkeypatch, dict(LBM_TILE_X=64, LBM_TILE_Y=4), **kw)
        assert np.isfinite(ref).all()
        assert np.array_equal(_run(w, monkeypatch, dict(LBM_BOX="0"), **kw), ref)  # the planned tile
        for tx, ty, zc in ((32, rows, 2), (43, 5, 3), (64, 1, 1), (5, rows, shape[2])):
            f = _run(w, monkeypatch, dict(LBM_TILE_X=tx, LBM_TILE_Y=ty, LBM_ZCHUNK=zc), **kw)
            assert np.array_equal(f, ref), (c_ns, tx, ty)


@pytest.mark.parametrize("storage", ["f16s", "f32", "f64"])
@pytest.mark.parametrize("shapes", [[(33, 17, 9), (67, 40, 21), (130, 9, 11)], [(64, 16, 20), (128, 24, 9)]])
def test_group_tiles_do_not_change_results(monkeypatch, storage, shapes):
    import torch
    ws = [_workload(s, 1) for s in shapes]
    ref = [_run(w, monkeypatch, dict(LBM_TILE_X=64, LBM_TILE_Y=8), storage=storage) for w in ws]
    monkeypatch.delenv("LBM_TILE_X")
    monkeypatch.delenv("LBM_TILE_Y")
    with torch.cuda.stream(torch.cuda.Stream()):
        sims = [lbm.from_workload(w, storage=storage) for w in ws]
        g = lbm.Group(sims)
        g.step(5)
        for s, f in zip(sims, ref):
            assert np.array_equal(s.populations(), f)
        g.step(16)  # a graph replay
        for s in sims:
            assert np.isfinite(s.populations()).all()
        g.close()
        for s in sims:
            s.close()
