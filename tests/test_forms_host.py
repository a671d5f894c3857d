"""Which forms the rules choose for the systems of the GPU tests and the
workloads: a change of a rule that takes the plane or tile kernels out of their
own tests fails here."""
import pytest

from paper_1905_00480_amd import binding as bd
from paper_1905_00480_amd import workloads as wl

import test_gpu_plane_waves as waves
import test_gpu_planes as planes
import test_gpu_tiles as tiles

ITEMS = {"nu0", "nu1", "one_column"}  # few or small: they run as work items


def _forms(s, flags=0):
    p = bd.Plan.from_system(s, flags=flags | bd.FLAG_HOST_ONLY)
    f = p.forms()
    p.close()
    return f


@pytest.mark.parametrize("name", sorted(planes.CASES))
def test_plane_cases(name):
    s = planes.CASES[name]()
    for flags in (0, bd.FLAG_DETERMINISTIC):
        want = (bd.PROJECT_ITEMS, 0) if name in ITEMS else (bd.FORM_PLANES, 4)
        assert _forms(s, flags)[:2] == want


@pytest.mark.parametrize("name", sorted(waves.CASES))
def test_plane_wave_cases(name):
    nu, nbands, w = waves.CASES[name]
    for flags in (0, bd.FLAG_DETERMINISTIC, bd.FLAG_BLOCH):
        assert _forms(waves.system(nu, nbands, w), flags)[:2] == (bd.FORM_PLANES, w)
    if w == 1 and nbands % 2 == 0:
        assert _forms(waves.system(nu, nbands, w), bd.FLAG_FP32)[:2] == (bd.FORM_PLANES, w)


@pytest.mark.parametrize("name", sorted(tiles.CASES))
def test_tile_cases(name):
    s = tiles.CASES[name]()
    assert _forms(s, bd.FLAG_DETERMINISTIC)[2] == bd.FORM_TILES
    few = name in ("bands1", "bands2", "one_column")
    assert _forms(s)[2] == (bd.EXPAND_BLOCKS if few else bd.FORM_TILES)


def test_workloads():
    assert _forms(wl.scale()) == (bd.FORM_PLANES, 2, bd.FORM_TILES)
    assert _forms(wl.scale(), bd.FLAG_FP32) == (bd.PROJECT_ITEMS, 0, bd.FORM_TILES)
    assert _forms(wl.scale(), bd.FLAG_BLOCH) == (bd.FORM_PLANES, 2, bd.FORM_TILES)
    assert _forms(wl.scale(), bd.FLAG_DETERMINISTIC) == (bd.FORM_PLANES, 2, bd.FORM_TILES)
