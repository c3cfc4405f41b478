"""What groups and servers launch, seen on a device that is not there
(tests/plan_driver/group_driver.cpp): tiles, store policies, graphs."""
import pytest

from paper_2206_11524_amd import lbm

import _plan


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    return _plan.build_driver("group_driver", tmp_path_factory.mktemp("plan") / "group_driver")


def _tiles(lines):
    return {tuple(map(int, x.split()[1:3])) for x in lines if x.startswith("tile")}


def _server(driver, storage, ncomp, tile, *shapes):
    return _plan.run_driver(driver, ["server", lbm.STORAGE[storage], ncomp, 1, *tile, *sum(shapes, ())])


def _group(driver, storage, ncomp, steps, *shapes, **env):
    return _plan.run_driver(driver, ["group", lbm.STORAGE[storage], ncomp, 1, steps, *sum(shapes, ())], env=env)


# two components in FP64 hold 256 cells in five rows: as many of the rows as that
@pytest.mark.parametrize("storage,ncomp,asked,got", [
    ("f64", 2, (64, 8), (64, 4)), ("f64", 2, (32, 8), (32, 5)), ("f64", 1, (32, 8), (32, 8)), ("f32", 1, (64, 8), (64, 8)),
    ("f32", 2, (64, 8), (64, 8)), ("f16s", 2, (64, 0), (64, 8))])
def test_an_asked_tile_is_used(driver, storage, ncomp, asked, got):
    assert _tiles(_server(driver, storage, ncomp, asked, (40, 40, 40), (131, 50, 20))) == {got}
    env = {"LBM_BATCH_TILE_X": asked[0]}
    if asked[1]:
        env["LBM_BATCH_TILE_Y"] = asked[1]
    assert _tiles(_group(driver, storage, ncomp, 20, (40, 40, 40), (131, 50, 20), **env)) == {got}


def _after_creation(lines):
    return lines[lines.index("created") + 1:]


@pytest.mark.parametrize("storage", ["f64", "f32", "f16s"])
def test_server_captures_its_graphs_when_it_is_created(driver, storage):
    """Requests of whole lines and of ragged rows, so of both store policies:
    every full tick replays a graph, none is captured on the way."""
    out = _server(driver, storage, 2, (0, 0), (64, 64, 16), (67, 67, 67), (128, 16, 16), (70, 69, 65))
    ticks = _after_creation(out)
    assert not [x for x in ticks if x.startswith(("capture", "launch"))]
    policies = {x.split()[1] for x in ticks if x.startswith("graph")}
    assert policies == ({"1"} if storage == "f64" else {"0", "1"})
    assert {x.split()[2] for x in out if x.startswith("capture")} == policies


@pytest.mark.parametrize("env", [{}, {"LBM_BATCH_TILE_X": 32}, {"LBM_BATCH_TILE_X": 64}], ids=str)
def test_group_captures_the_policy_that_it_launches(driver, env):
    # one component in FP16: rows of 64 cells are whole lines, of 32 are not
    out = _group(driver, "f16s", 1, 36, (64, 48, 200), (128, 32, 20), **env)
    steps = _after_creation(out)
    assert not [x for x in steps if x.startswith("capture")]
    policy = {x.split()[2] for x in out if x.startswith("capture")}
    assert len(policy) == 1
    assert [x for x in steps if not x.startswith(("tile", "time"))] == (
        2 * ["graph " + min(policy)] + 4 * ["launch " + min(policy)])


@pytest.mark.parametrize("failing", [1, 2, 3, 4])
def test_a_failed_capture_leaves_the_other_graphs(driver, failing):
    out = _plan.run_driver(driver, ["server", lbm.STORAGE["f16s"], 2, 1, 0, 0, *(64, 64, 16, 67, 67, 67) * 3],
                           env=dict(FAKE_FAIL_CAPTURE=failing))
    ticks = _after_creation(out)
    assert sum(x.startswith("capture") for x in out) == 3
    graphs, launches = (sum(x.startswith(k) for x in ticks) for k in ("graph", "launch"))
    # twelve ticks of four steps, alternately from two tables, six of each policy:
    # three of them lost their graph
    assert (graphs, launches) == (9, 3 * 4)


# us a step, fitted / 64-wide tiles
@pytest.mark.parametrize("storage,ncomp,edge,n,got", [
    ("f32", 2, 32, 8, (64, 8)),    # 35 / 31
    ("f32", 1, 32, 8, (64, 8)),    # 26 / 22
    ("f16s", 1, 24, 16, (64, 8)),  # 25 / 23
    ("f32", 2, 24, 16, (24, 12)),  # 31 / 34: some blocks would get a second tile
    ("f32", 1, 16, 5, (16, 16)),   # 14 / 20: some CUs would
    ("f32", 2, 40, 12, (40, 10)),  # enough tiles
    ("f16s", 2, 128, 8, (64, 8)),
])
def test_small_batches_spread_over_the_device(driver, storage, ncomp, edge, n, got):
    assert _tiles(_group(driver, storage, ncomp, 16, *[(edge, edge, edge)] * n)) == {got}


# us a step, non-temporal / cached stores
@pytest.mark.parametrize("storage,ncomp,shape,n,policy", [
    ("f32", 2, (300, 50, 1), 4, "1"),   # 9 MB: 15.0 / 16.6
    ("f16s", 2, (28, 28, 28), 8, "1"),  # 13 MB: 24.3 / 25.9
    ("f32", 2, (33, 33, 33), 6, "0"),   # 33 MB: 34.7 / 30.8
    ("f32", 1, (62, 61, 60), 3, "0"),
    ("f32", 2, (64, 64, 64), 4, "1"),   # whole lines
])
def test_small_batches_store_past_the_caches(driver, storage, ncomp, shape, n, policy):
    out = _group(driver, storage, ncomp, 20, *[shape] * n)
    assert {x.split()[-1] for x in out if x.startswith(("capture", "graph", "launch"))} == {policy}
