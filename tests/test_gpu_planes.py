"""The plane form of the projection (the default: one wave per atom plane and
band group on FP64 matrix cores, then a z pass) where its kernels can go
wrong: every cut-off (function groups of four and their remainders), band
counts around the 16- and 32-band groups and odd ones, cells smaller than the
supports (runs cut at both faces, many images), atoms that miss the grid, and
large supports.  Against the oracle at the abs-sum bound of the other parity
tests, |c - c_oracle| <= 1e-12 A; the item form (set_schedule) must agree with
the oracle on the same inputs."""
import numpy as np
import pytest

import oracle
from paper_1905_00480_amd import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

RTOL = 1e-12


def _bd():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1905_00480_amd import binding
    binding.load_library()
    return binding


def _check(t, ref, ab, what):
    torch.cuda.synchronize()
    err = np.abs(t.cpu().numpy().ravel() - ref.ravel())
    bound = RTOL * ab.ravel() + 1e-300
    assert np.all(err <= bound), "%s: %d entries off, max |d| %.3e" % (
        what, int((err > bound).sum()), float(err.max()))


def _case(nu, nbands, n=(26, 23, 21), periodic=(True, True, False), natoms=4, h=0.2, sigma=0.6):
    return wl.make_system("planes", n, h, periodic, natoms, sigma, nu, nbands, 100 + nu + nbands)


CASES = {"nu%d" % nu: (lambda nu=nu: _case(nu, 20)) for nu in range(11)}
CASES.update({"bands%d" % b: (lambda b=b: _case(4, b)) for b in (1, 15, 16, 17, 31, 32, 33, 70)})
# (four small atoms run as work items: these have planes enough for the form)
CASES.update({"many_nu%d" % nu: (lambda nu=nu: _case(nu, 34, natoms=12)) for nu in range(4)})
CASES["bands21_nu9"] = lambda: _case(9, 21)
CASES["small_cell"] = lambda: _case(5, 18, n=(5, 7, 4), periodic=(True,) * 3, h=0.25)
CASES["one_column"] = lambda: _case(3, 3, n=(1, 9, 8), periodic=(True,) * 3, h=0.25)
CASES["mixed"] = wl.small_mixed
CASES["large"] = lambda: _case(6, 5, n=(70, 40, 12), periodic=(True, False, True), natoms=2,
                               sigma=1.3)


@pytest.mark.parametrize("name", sorted(CASES))
def test_plane_form_matches_oracle(name):
    bd = _bd()
    s = CASES[name]()
    psi = wl.psi_for(s)
    d_psi = torch.from_numpy(psi).cuda()
    ref, ab = oracle.project(*s.geometry(), psi, with_abs=True)
    for flags in (0, bd.FLAG_DETERMINISTIC):
        plan = bd.Plan.from_system(s, flags=flags)
        c = torch.full((plan.coeff_doubles,), float("nan"), dtype=torch.float64, device="cuda")
        _check(plan.project(d_psi, c), ref, ab, name)
        if flags:  # what a deterministic plan promises
            first = c.clone()
            plan.project(d_psi, c)
            assert torch.equal(first, c)
        plan.set_schedule(*plan.schedule())  # the caller's work items
        _check(plan.project(d_psi, c.fill_(float("nan"))), ref, ab, name + " items")
        plan.close()


def test_plane_form_atoms_outside_and_nan():
    """An atom that misses an isolated grid gets zeros; a NaN in one band stays
    in that band's coefficients and out of the atoms that do not hold it."""
    bd = _bd()
    s = wl.make_system("out", (40, 30, 30), 0.2, (False,) * 3, 5, 0.6, 4, 18, 7)
    s.pos[0] = (-9.0, 1.0, 1.0)
    s.pos[1] = (1.0, 3.0, 3.0)
    s.pos[2] = (7.0, 3.0, 3.0)
    psi = wl.psi_for(s)
    ref, ab = oracle.project(*s.geometry(), psi, with_abs=True)
    plan = bd.Plan.from_system(s)
    _check(plan.project(torch.from_numpy(psi).cuda()), ref, ab, "outside")
    psi[15, 15, 5, 3] = np.nan  # next to atom 1
    c = plan.project(torch.from_numpy(psi).cuda()).cpu().numpy()
    off = wl.coeff_offsets(s)
    hit = np.isnan(c[off[1]:off[2]].reshape(-1, s.nbands))
    assert hit[:, 3].all() and not np.delete(hit, 3, axis=1).any()
    assert not np.isnan(c[off[2]:off[3]]).any()
    plan.close()


def test_projection_captured_by_the_caller():
    """A caller's own capture records no use of the plan's scratch: replays
    beside eager calls of the plan keep their results."""
    bd = _bd()
    s = _case(5, 20)
    psi = wl.psi_for(s)
    d_psi = torch.from_numpy(psi).cuda()
    ref, ab = oracle.project(*s.geometry(), psi, with_abs=True)
    plan = bd.Plan.from_system(s)
    c = torch.empty(plan.coeff_doubles, dtype=torch.float64, device="cuda")
    plan.project(d_psi, c)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        plan.project(d_psi, c)
    eager = torch.empty_like(c)
    for _ in range(3):
        c.fill_(float("nan"))
        g.replay()
        plan.project(d_psi, eager)
        _check(c, ref, ab, "replay")
        _check(eager, ref, ab, "eager")
    plan.close()
