"""Launch plans, chosen on the host (no device): what a domain's kernel, tile
and chunk may be, from times measured on an MI355X."""
import pytest

import _box_cases
import _plan


@pytest.fixture(scope="module")
def planner(tmp_path_factory):
    return _plan.build_driver("plan_driver", tmp_path_factory.mktemp("plan") / "plan_driver")


# us a step of (tile, planes per block); each plan has to be one of those within
# 6 % of the best
TIMES = {
    # the caches hold the domain: idle lanes cost little, planes a round trip each
    ((63, 63, 63), "f64", 2): {(63, 4, 4): 38.3, (63, 3, 6): 45.1, (63, 2, 8): 53.7},
    ((58, 209, 11), "f64", 2): {(58, 3, 4): 30.6, (58, 4, 4): 31.4, (58, 2, 6): 38.6},
    ((268, 22, 51), "f64", 2): {(64, 4, 7): 53.7, (64, 3, 9): 61.3},
    ((64, 64, 129), "f64", 2): {(64, 4, 9): 75.9, (64, 3, 12): 85.2},
    ((64, 64, 129), "f32", 2): {(64, 8, 5): 39.7, (64, 6, 6): 43.5},
    ((64, 64, 129), "f16s", 2): {(64, 8, 5): 29.2, (64, 6, 6): 32.8},
    # rows of whole lines, beyond the caches: a tile that splits them
    ((160, 242, 96), "f32", 1): {(64, 6, 48): 119.1, (32, 15, 32): 107.7, (54, 9, 32): 172.3},
    ((200, 200, 100), "f64", 1): {(64, 8, 20): 260.0, (40, 12, 34): 247.0, (50, 10, 34): 321.0},
    ((200, 200, 200), "f64", 1): {(64, 8, 40): 499.7, (40, 12, 67): 471.9, (50, 10, 67): 652.4},
    # flat: a chunk's halo and pipeline fill cost less than idle lanes' planes
    ((254, 268, 30), "f16s", 2): {(64, 8, 10): 106.3, (64, 7, 10): 107.6, (64, 5, 30): 128.0, (64, 8, 30): 128.7},
    ((160, 160, 160), "f16s", 2): {(32, 16, 32): 167.3, (64, 8, 40): 176.9},
    ((224, 224, 224), "f16s", 2): {(64, 8, 112): 418.9, (64, 8, 25): 440.3, (32, 16, 45): 442.3},
    # rows that split lines anyway keep the fitted tiles
    ((131, 131, 131), "f16s", 2): {(44, 11, 19): 108.2, (64, 8, 27): 124.8},
    ((131, 131, 131), "f64", 2): {(44, 5, 44): 363.9, (64, 4, 27): 407.1},
    ((150, 150, 150), "f32", 1): {(50, 9, 30): 114.8, (50, 10, 30): 119.8, (64, 8, 38): 148.6},
}


@pytest.mark.parametrize("domain", TIMES, ids=lambda d: "x".join(map(str, d[0])) + "-" + d[1] + "-%d" % d[2])
def test_planned_tile_is_near_the_best_measured(planner, domain):
    shape, storage, ncomp = domain
    p = _plan.plans(planner, [(shape, storage, ncomp, 1, "shan-chen")])[0]
    times = TIMES[domain]
    assert p.box is None
    assert times[(*p.tile, p.zchunk)] <= 1.06 * min(times.values())


@pytest.mark.parametrize("storage,ncomp,c_ns,forcing", [("f64", 1, 1, "shan-chen"), ("f32", 1, 1, "guo"),
                                                        ("f32", 2, 2, "guo"), ("f32", 2, 1, "shan-chen"),
                                                        ("f16s", 2, 2, "guo"), ("bf16s", 1, 1, "shan-chen")])
def test_thin_domains_take_small_blocks(planner, storage, ncomp, c_ns, forcing):
    """Four rows fill 256 lanes of a block at most; beyond them 512 are the
    faster ones."""
    fmt = (storage, ncomp, c_ns, forcing)
    thin = [((nx, ny, nz), *fmt) for nx, nz in ((40000, 1), (400, 400), (100, 2000)) for ny in (1, 2, 3, 4)]
    for p in _plan.plans(planner, thin, env=dict(LBM_BOX="0")):
        assert p.cells == 256 and p.tile[1] <= 4
    for p in _plan.plans(planner, [((40000, 5, 1), *fmt), ((400, 7, 400), *fmt)], env=dict(LBM_BOX="0")):
        assert p.cells == 512
    # a tile that does not fit the small block keeps the large one
    for ty, cells in ((4, 256), (8, 512)):
        p = _plan.plans(planner, [((400, 4, 400), *fmt)], env=dict(LBM_TILE_X=64, LBM_TILE_Y=ty))[0]
        assert (p.tile, p.cells) == ((64, ty), cells)


def test_box_stores_are_cached_beyond_the_l2(planner):
    """Domains of the box kernel, us a step with cached / non-temporal stores."""
    cached = [((261, 95, 19), "f32", 1), ((261, 95, 19), "f64", 1), ((57, 57, 57), "f16s", 2),  # 17 / 22, 32 / 38, 15 / 17
              ((42, 42, 42), "f64", 2)]  # 18 / 21
    nt = [((41, 41, 41), "f32", 2), ((247, 111, 8), "f32", 1), ((36, 36, 36), "f32", 2)]  # 9.3 / 8.7, 12 / 10, 8.1 / 7.2
    for d, want in [(d, False) for d in cached] + [(d, True) for d in nt]:
        p = _plan.plans(planner, [(*d, 1, "shan-chen")])[0]
        assert p.box and p.nt is want, d


def test_served_and_grouped_domains_have_the_same_tile(planner):
    """Cubes of edge 2 to 192 and flat, thin and uneven domains, in every
    format of the batched kernel."""
    shapes = [(e, e, e) for e in range(2, 193)]
    shapes += [(x, y, z) for x in (5, 17, 40, 63, 100, 127) for y in (3, 12, 40, 77) for z in (1, 6, 50)]
    fmts = [(st, nc, cn, "shan-chen") for st in ("f64", "f32", "f16s", "bf16s") for nc, cn in ((1, 1), (2, 1), (2, 2))]
    domains = [(s, *f) for s in shapes for f in fmts]
    for d, p in zip(domains, _plan.plans(planner, domains)):
        assert p.group == p.server, d
        assert p.group[0] <= max(d[0][0], 64)


@pytest.mark.parametrize("tile", [dict(LBM_TILE_X=32), dict(LBM_TILE_Y=2), dict(LBM_TILE_X=20, LBM_TILE_Y=5)],
                         ids=lambda e: "-".join("%s=%d" % i for i in e.items()))
def test_sweep_tile_settings_stay_out_of_groups_and_servers(planner, tile):
    domains = [(s, st, nc, 1, "shan-chen") for s in ((40, 40, 40), (131, 50, 20), (96, 96, 96), (300, 50, 1))
               for st in ("f64", "f32", "f16s") for nc in (1, 2)]
    for d, p, q in zip(domains, _plan.plans(planner, domains), _plan.plans(planner, domains, env=tile)):
        assert (p.group, p.server) == (q.group, q.server), d
        assert q.tile[0] == tile.get("LBM_TILE_X", 64) and q.box is None


@pytest.mark.parametrize("fmt", _box_cases.CASES, ids=lambda f: "-".join(map(str, f)))
def test_box_cases_take_the_box_kernel(planner, fmt):
    shapes, boxes = _box_cases.CASES[fmt]
    assert all(p.box for p in _plan.plans(planner, [(s, *fmt) for s in shapes]))
    for box in boxes:
        p = _plan.plans(planner, [(_box_cases.BOXED, *fmt)], env=dict(LBM_BOX="%d,%d,%d" % box))[0]
        assert p.box == box
    for env in (dict(LBM_BOX="0"), dict(LBM_TILE_X=64), dict(LBM_BOX="64,64,64")):  # the last fits no format
        assert not any(p.box for p in _plan.plans(planner, [(s, *fmt) for s in shapes], env=env))


def test_box_rows_of_whole_lines_are_stored_past_the_caches(planner):
    """Beyond the L2 as well: 64 x 64 x 128 with one component in FP32 15.7 us a
    step, 15.9 with cached stores."""
    for shape, nt in (((64, 64, 128), True), ((66, 62, 128), False)):
        p = _plan.plans(planner, [(shape, "f32", 1, 1, "shan-chen")])[0]
        assert p.box and p.nt is nt


def test_one_component_fp64_stores_split_rows_through_the_caches(planner):
    """us a step, cached / non-temporal: 317 x 125 x 210 528 / 605, 133 x 117 x 181
    194 / 273, 234 x 42 x 355 240 / 307.  Rows of whole 64 bytes (160^3, 200^3 in
    40-wide tiles) and two components stay non-temporal."""
    for shape, ncomp, nt in (((317, 125, 210), 1, False), ((133, 117, 181), 1, False), ((234, 42, 355), 1, False),
                             ((160, 160, 160), 1, True), ((200, 200, 200), 1, True), ((150, 150, 150), 2, True)):
        p = _plan.plans(planner, [(shape, "f64", ncomp, 1, "shan-chen")])[0]
        assert p.box is None and p.nt is nt, shape
