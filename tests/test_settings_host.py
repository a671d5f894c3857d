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
