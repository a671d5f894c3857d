"""Settings of the projection and expansion forms on host-only plans: whatever
the order in which they are made, a plan with supports keeps the tables of the
form that will run."""
import ctypes
import itertools

import pytest

from paper_1905_00480_amd import binding as bd
from paper_1905_00480_amd import workloads as wl

KINDS = {"f64": 0, "det": bd.FLAG_DETERMINISTIC, "f32": bd.FLAG_FP32, "bloch": bd.FLAG_BLOCH,
         "stored": bd.FLAG_STORED, "per_atom": bd.FLAG_PER_ATOM}


def _plan(flags, nbands=32, natoms=12):
    s = wl.small_periodic(natoms=natoms, nbands=nbands)
    return bd.Plan(s.n, s.h, s.periodic, s.pos, s.sigma, s.numax, s.nbands,
                   flags=flags | bd.FLAG_HOST_ONLY)


def _info(p):  # as it is now (Plan.info is what it was at creation)
    info = bd.sho_plan_info()
    assert bd.load_library().sho_plan_get_info(p._h, ctypes.byref(info)) == bd.SHO_OK
    return {k: getattr(info, k) for k, _ in bd.sho_plan_info._fields_}


def _setters(p):
    mode, rows, x = p.expand_form()
    return {
        "expand rows": lambda: p.set_expand(bd.EXPAND_ROWS),
        "expand blocks": lambda: p.set_expand(bd.EXPAND_BLOCKS),
        "expand blocks 4x8": lambda: p.set_expand(bd.EXPAND_BLOCKS, 4, 8),
        "expand owner": lambda: p.set_expand(bd.EXPAND_OWNER),
        "expand owner 16": lambda: p.set_expand(bd.EXPAND_OWNER, 0, 16),
        "expand as given": lambda: p.set_expand(mode, rows, x),
        "tile 0": lambda: p.set_expand_tile(0),
        "tile 8": lambda: p.set_expand_tile(8),
        "tile 16": lambda: p.set_expand_tile(16),
        "schedule": lambda: p.set_schedule(bd.SCHED_SINGLE_LPT, 0, 4096),
        "project items": lambda: p.set_project(bd.PROJECT_ITEMS),
        "project blocks": lambda: p.set_project(bd.PROJECT_BLOCKS),
    }


@pytest.mark.parametrize("kind", sorted(KINDS))
def test_no_setting_leaves_an_empty_form(kind):
    names = list(_setters(_plan(KINDS[kind])))
    for seq in itertools.chain(itertools.permutations(names, 2), [(n,) for n in names]):
        p = _plan(KINDS[kind])
        setters = _setters(p)
        for n in seq:
            try:
                setters[n]()
            except bd.ShoError as e:  # a form that plans of this kind refuse
                assert e.code == bd.SHO_E_INVALID
        info = _info(p)
        if p.expand_form()[0] != bd.EXPAND_ROWS:  # (which has tables of its own)
            assert info["expand_blocks"] > 0 and info["expand_entries"] > 0, seq
        p.close()


def test_band_tile_leaves_deterministic_plans_their_form():
    """The band tile is the block form's, which deterministic plans never take."""
    for tile in (0, 8, 16, 32):
        p = _plan(bd.FLAG_DETERMINISTIC)
        before = _info(p)
        p.set_expand_tile(tile)
        assert _info(p) == before
        p.close()


def _state(p):
    info = _info(p)
    return (p.forms(), p.schedule(), p.expand_form(), p.expand_tile(), info["expand_blocks"],
            info["expand_entries"], info["expand_points"])


@pytest.mark.parametrize("kind", sorted(KINDS))
def test_settings_survive_a_round_trip(kind):
    """What the getters return, set again at once or after other settings, gives
    the state that it was read in."""
    stored = kind == "stored"
    base = bd.SCHED_SINGLE if kind == "bloch" else bd.SCHED_SINGLE_LPT
    p = _plan(KINDS[kind])
    fresh = _state(p)
    sc, ex, tile, pr = p.schedule(), p.expand_form(), p.expand_tile(), p.project_form()
    if kind in ("f64", "det", "bloch"):
        assert fresh[0] == (bd.FORM_PLANES, 4, bd.FORM_TILES)

    def give_back():
        p.set_schedule(*sc)
        if not stored:
            p.set_expand_tile(tile)
        p.set_expand(*ex)
        p.set_project(*pr)

    give_back()
    assert _state(p) == fresh
    p.set_schedule(base, 0, 4096)
    assert p.forms()[:2] == (bd.PROJECT_ITEMS, 0)
    kept = _state(p)
    p.set_schedule(*p.schedule())
    assert _state(p) == kept
    for tile2 in () if stored else (8, 16):
        p.set_expand_tile(tile2)
        kept = _state(p)
        p.set_expand_tile(p.expand_tile())
        assert _state(p) == kept
    form = (bd.EXPAND_OWNER, 0, 16) if kind == "det" else (bd.EXPAND_BLOCKS, 2, 8)
    p.set_expand(*form)
    assert p.forms()[2] == form[0]
    kept = _state(p)
    p.set_expand(*p.expand_form())
    assert _state(p) == kept
    give_back()
    if stored:  # (in the row form here, which takes no shape)
        assert _state(p)[:2] == fresh[:2]
    else:
        assert _state(p) == fresh
    p.close()


def test_project_blocks_and_back():
    p = _plan(0)
    fresh = _state(p)
    p.set_project(bd.PROJECT_BLOCKS)
    assert p.forms()[0] == bd.PROJECT_BLOCKS
    p.set_project(bd.PROJECT_ITEMS)
    assert _state(p) == fresh
    p.close()


@pytest.mark.parametrize("kind", ["f64", "det", "f32", "bloch"])
def test_expand_points_of_tiles_and_blocks(kind):
    """Tiles move the points that a support holds, blocks whole blocks, whatever
    ran before."""
    p = _plan(KINDS[kind])
    first = _info(p)
    assert p.forms()[2] == bd.FORM_TILES
    assert first["expand_points"] == first["union_points"]
    mode = p.expand_form()[0]
    p.set_expand(mode, *((0, 16) if kind == "det" else (2, 8)))
    assert p.forms()[2] == mode
    assert _info(p)["expand_points"] >= first["union_points"]
    p.set_expand(mode)
    assert _info(p)["expand_points"] == first["union_points"]
    p.close()


def test_launches_too_large_for_tiles_stay_with_blocks():
    """64 planes of a 4 x 4 column are 64 tiles; a launch of 64 x 2^18 band groups
    of 256 threads would be 2^32."""
    for nbands, form in ((1 << 22, bd.FORM_TILES), (1 << 23, bd.EXPAND_BLOCKS)):
        p = bd.Plan((4, 4, 64), 0.3, (False,) * 3, [[0.5, 0.5, 9.5]], [1.0], [1], nbands,
                    rbox=[12.0], flags=bd.FLAG_HOST_ONLY)
        assert p.forms()[2] == form
        assert _info(p)["expand_blocks"] > 0
        p.close()
