"""A deterministic plan gives the same bits in every call: also on a stream that
the caller is capturing, where the projection may not use the plan's scratch,
and after that scratch was released.  Systems for every cut-off, one, two and
four waves per atom plane, one and two bands per lane, and odd band counts."""
import numpy as np
import pytest

import oracle
from paper_1905_00480_amd import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _bd():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1905_00480_amd import binding
    binding.load_library()
    return binding


def _case(nu, nbands, n=(26, 23, 21), periodic=(True, True, False), natoms=4, sigma=0.6):
    return wl.make_system("cap", n, 0.2, periodic, natoms, sigma, nu, nbands, 700 + nu + nbands)


CASES = {"nu%d" % nu: (lambda nu=nu: _case(nu, 20, natoms=12)) for nu in range(11)}
CASES.update({"nu%d_bands13" % nu: (lambda nu=nu: _case(nu, 13, natoms=12)) for nu in (2, 5, 8)})
CASES["bands33"] = lambda: _case(4, 33)
# units enough for two waves each (little overlap) and for one
CASES["two_waves"] = lambda: _case(5, 33, n=(72, 72, 66), natoms=50, periodic=(True,) * 3)
CASES["one_wave"] = lambda: _case(6, 35, n=(36, 33, 40), natoms=60, periodic=(True, False, True))
CASES["mixed"] = wl.small_mixed


def _outside():  # an atom that misses the grid
    s = wl.make_system("out", (40, 30, 30), 0.2, (False,) * 3, 5, 0.6, 4, 18, 7)
    s.pos[0] = (-9.0, 1.0, 1.0)
    return s


CASES["outside"] = _outside


def _bits(t):
    return t.view(torch.int64)


@pytest.mark.parametrize("name", sorted(CASES))
def test_captured_calls_give_the_bits_of_eager_ones(name):
    bd = _bd()
    s = CASES[name]()
    psi, w = wl.psi_for(s), wl.coeffs_for(s)
    d_psi, d_w = torch.from_numpy(psi).cuda(), torch.from_numpy(w).cuda()
    plan = bd.Plan.from_system(s, flags=bd.FLAG_DETERMINISTIC)
    c0 = plan.project(d_psi).clone()
    e0 = plan.expand(d_w, d_psi.clone())
    ref, ab = oracle.project(*s.geometry(), psi, with_abs=True)
    assert np.all(np.abs(c0.cpu().numpy() - ref.ravel()) <= 1e-12 * ab.ravel() + 1e-300)
    c, e = torch.empty_like(c0), torch.empty_like(d_psi)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        plan.project(d_psi, c)
        plan.expand(d_w, e)
    for _ in range(3):
        c.fill_(float("nan"))
        e.copy_(d_psi)
        g.replay()
        eager = plan.project(d_psi)
        torch.cuda.synchronize()
        assert torch.equal(_bits(c), _bits(c0)) and torch.equal(_bits(e), _bits(e0))
        assert torch.equal(_bits(eager), _bits(c0))
    plan.close()


def test_projection_captured_without_scratch():
    """The captured projection uses none: it replays after the plan's scratch
    is released, and so does the next eager call, which allocates it again."""
    bd = _bd()
    s = CASES["nu5"]()
    d_psi = torch.from_numpy(wl.psi_for(s)).cuda()
    plan = bd.Plan.from_system(s, flags=bd.FLAG_DETERMINISTIC)
    c0 = plan.project(d_psi).clone()
    c = torch.empty_like(c0)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        plan.project(d_psi, c)
    plan.release_scratch()
    for _ in range(2):
        c.fill_(float("nan"))
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(_bits(c), _bits(c0))
        assert torch.equal(_bits(plan.project(d_psi)), _bits(c0))
    plan.close()
