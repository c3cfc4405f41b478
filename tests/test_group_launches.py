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
