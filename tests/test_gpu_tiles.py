"""The tile form of the expansion (the default: plane partials, then one
workgroup per 16 rows x 16 points and 16 or 32 bands, matrix cores along y and
vector FMAs along x) where its kernels can go wrong: every cut-off (function
groups of four and their remainders), band counts around the 16- and 32-band
groups and odd ones, grids that are no multiple of a tile, cells smaller than
the supports (runs cut at both faces, many images), atoms that miss the grid.
Deterministic plans take the form at every size; the others by a rule, so that
their default is compared as well and the block form (an explicit shape) must
agree with the same oracle.  Bounds of the other parity tests: FP64
|psi - psi_oracle| <= 1e-12 A; FP32 2 k u A with k = 3 (nu_max + 1) + 4 +
overlaps, A = |psi_in| + sum |c P|.
"""
import numpy as np
import pytest

import oracle
from paper_1905_00480_amd import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

RTOL = 1e-12
U32 = 2.0 ** -24


def _bd():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1905_00480_amd import binding
    binding.load_library()
    return binding


def _check(t, ref, ab, what, k=None):
    torch.cuda.synchronize()
    d = t.cpu().numpy().ravel() - ref.ravel()
    err = np.maximum(np.abs(d.real), np.abs(d.imag))
    bound = (RTOL * ab.ravel() if k is None else 2.0 * k * U32 * ab.ravel()) + 1e-300
    assert np.all(err <= bound), "%s: %d entries off, max |d| %.3e" % (
        what, int((err > bound).sum()), float(err.max()))


def _small(nu, nbands, n=(26, 23, 21), periodic=(True, True, False), natoms=4, h=0.2, sigma=0.6):
    return wl.make_system("tiles", n, h, periodic, natoms, sigma, nu, nbands, 300 + nu + nbands)


def _many(nu, nbands):  # tiles enough for two bands per lane
    return _small(nu, nbands, n=(37, 33, 70), natoms=40 if nu < 4 else 14,
                  periodic=(True, False, True))


CASES = {"nu%d" % nu: (lambda nu=nu: _small(nu, 20)) for nu in range(11)}
CASES.update({"bands%d" % b: (lambda b=b: _small(4, b)) for b in (1, 2, 15, 16, 17, 33)})
CASES.update({"many_nu%d" % nu: (lambda nu=nu: _many(nu, 32)) for nu in range(11)})
CASES.update({"many_bands%d" % b: (lambda b=b: _many(4, b)) for b in (17, 31, 33, 70)})
CASES["bands21_nu9"] = lambda: _small(9, 21)
CASES["small_cell"] = lambda: _small(5, 18, n=(5, 7, 4), periodic=(True,) * 3, h=0.25)
CASES["one_column"] = lambda: _small(3, 3, n=(1, 9, 8), periodic=(True,) * 3, h=0.25)
CASES["mixed"] = wl.small_mixed
CASES["large"] = lambda: _small(6, 5, n=(70, 40, 12), periodic=(True, False, True), natoms=2,
                                sigma=1.3)


@pytest.mark.parametrize("name", sorted(CASES))
def test_tile_form_matches_oracle(name):
    bd = _bd()
    s = CASES[name]()
    psi, w = wl.psi_for(s), wl.coeffs_for(s)
    d_psi, d_w = torch.from_numpy(psi).cuda(), torch.from_numpy(w).cuda()
    ref, ab = oracle.expand(*s.geometry(), w, psi, with_abs=True)
    for flags in (bd.FLAG_DETERMINISTIC, 0):
        plan = bd.Plan.from_system(s, flags=flags)
        out = plan.expand(d_w, d_psi.clone())
        _check(out, ref, ab, name)
        same = oracle.expand(*s.geometry(), np.zeros_like(w), psi, with_abs=True)[1] == ab
        assert np.array_equal(out.cpu().numpy()[same], psi[same])  # points of no atom
        if flags:
            if name.startswith("many"):
                assert plan.info["expand_blocks"] * ((s.nbands + 31) // 32) >= 512
            assert torch.equal(out, plan.expand(d_w, d_psi.clone()))
        mode, rows, x = plan.expand_form()
        plan.set_expand(mode, rows, x)  # the named form
        _check(plan.expand(d_w, d_psi.clone()), ref, ab, name + " by its shape")
        plan.set_expand(mode)  # and the default again
        _check(plan.expand(d_w, d_psi.clone()), ref, ab, name + " default again")
        plan.close()


@pytest.mark.parametrize("nu,nbands", [(0, 70), (1, 62), (2, 66), (3, 34), (4, 14), (5, 18), (6, 32),
                                       (7, 20), (8, 22), (9, 34), (10, 12)])
def test_tile_form_fp32_and_bloch(nu, nbands):
    bd = _bd()
    s = _many(nu, nbands)
    rng = np.random.default_rng(nu)
    cnt = np.zeros(int(np.prod(s.n)))
    for a in range(s.natoms):
        _, mem = oracle.support(s.n, s.h, s.periodic, s.pos[a],
                                oracle.box_radius(s.sigma[a], s.numax[a], s.h))
        cnt += np.bincount(mem, minlength=cnt.size)
    k = np.repeat(3 * (nu + 1) + 4 + cnt, nbands)
    psi, w = wl.psi_for(s, dtype=np.float32), wl.coeffs_for(s).astype(np.float32)
    ref, ab = oracle.expand(*s.geometry(), w.astype(np.float64), psi.astype(np.float64),
                            with_abs=True)
    plan = bd.Plan.from_system(s, flags=bd.FLAG_FP32)
    _check(plan.expand(torch.from_numpy(w).cuda(), torch.from_numpy(psi).cuda()), ref, ab,
           "fp32", k)
    plan.close()
    kp = (0.9, -0.4, 1.7)
    zpsi = rng.standard_normal(s.psi_shape) + 1j * rng.standard_normal(s.psi_shape)
    zw = rng.standard_normal(w.size) + 1j * rng.standard_normal(w.size)
    ref, ab = oracle.expand_k(*s.geometry(), zw, zpsi, kp, with_abs=True)
    plan = bd.Plan.from_system(s, flags=bd.FLAG_BLOCH)
    plan.set_kpoint(kp)
    _check(plan.expand(torch.from_numpy(zw).cuda(), torch.from_numpy(zpsi).cuda()), ref, ab,
           "bloch")
    plan.close()


def test_tile_form_nan_and_capture():
    """A NaN coefficient reaches the points of its atom in its band alone; a
    caller's capture replays beside eager calls."""
    bd = _bd()
    s = _small(5, 20, n=(48, 20, 18), periodic=(False,) * 3, natoms=3)
    s.pos[0], s.pos[1], s.pos[2] = (1.5, 2.0, 1.8), (8.0, 2.0, 1.8), (5.0, 2.0, 1.8)
    psi, w = wl.psi_for(s), wl.coeffs_for(s)
    d_psi, d_w = torch.from_numpy(psi).cuda(), torch.from_numpy(w).cuda()
    ref, ab = oracle.expand(*s.geometry(), w, psi, with_abs=True)
    plan = bd.Plan.from_system(s, flags=bd.FLAG_DETERMINISTIC)
    bad = d_w.clone()
    bad[7] = float("nan")  # atom 0, band 7
    hit = torch.isnan(plan.expand(bad, d_psi.clone())).cpu().numpy()
    mem = oracle.support(s.n, s.h, s.periodic, s.pos[0],
                         oracle.box_radius(s.sigma[0], s.numax[0], s.h))[1]
    want = np.zeros((psi.size // s.nbands, s.nbands), dtype=bool)
    want[mem, 7] = True
    assert np.array_equal(hit.reshape(want.shape), want)
    out = d_psi.clone()
    plan.expand(d_w, out)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        plan.expand(d_w, out)
    for _ in range(3):
        out.copy_(d_psi)
        g.replay()
        eager = plan.expand(d_w, d_psi.clone())
        _check(out, ref, ab, "replay")
        _check(eager, ref, ab, "eager")
    plan.close()
