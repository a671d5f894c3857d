"""Infinities pass through the expansion and the projection as the sums that
they are terms of give them: a coefficient of +-Inf makes +-Inf (the sign of
c P) of the points of its atom in its band and leaves everything else finite,
and a point of +-Inf makes +-Inf of the coefficients of the atoms that hold it.
Band b carries its infinity at function b mod N_SHO or at a random one, so that
every remainder of the function groups of four is met."""
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


def _system(nu, wide):
    if wide:  # tiles enough for two bands per lane
        return wl.make_system("inf", (37, 33, 70), 0.2, (True, False, True),
                              40 if nu < 4 else 14, 0.6, nu, 34, 500 + nu)
    # (cells wider than the supports: two images of an infinity could cancel)
    return wl.make_system("inf", (36, 23, 21), 0.2, (True, False, False), 4, 0.6, nu, 13, 600 + nu)


def _functions(nu, nbands, rng):
    N = oracle.nsho(nu)
    return np.where(rng.random(nbands) < 0.5, np.arange(nbands) % N,
                    rng.integers(0, N, size=nbands))


def _values(plan, s, n, sign):
    """Of the functions n[b] of atom 0 in band b, on the grid (oracle)."""
    one = s.subset(np.array([0]))
    c = np.zeros((oracle.nsho(int(s.numax[0])), s.nbands))
    c[n, np.arange(s.nbands)] = sign
    return oracle.expand(*one.geometry(), c.ravel(), np.zeros(s.psi_shape))


@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("nu", range(11))
def test_infinite_coefficient(nu, wide):
    bd = _bd()
    s = _system(nu, wide)
    rng = np.random.default_rng(nu)
    n = _functions(nu, s.nbands, rng)
    sign = rng.choice([-1.0, 1.0], size=s.nbands)
    psi, w = wl.psi_for(s), wl.coeffs_for(s)
    off = oracle.coeff_offsets(s.numax, s.nbands)
    w[off[0]:off[1]].reshape(-1, s.nbands)[n, np.arange(s.nbands)] = sign * np.inf
    for flags in (bd.FLAG_DETERMINISTIC, 0):
        plan = bd.Plan.from_system(s, flags=flags)
        val = _values(plan, s, n, sign)
        got = plan.expand(torch.from_numpy(w).cuda(), torch.from_numpy(psi).cuda())
        torch.cuda.synchronize()
        got = got.cpu().numpy().reshape(val.shape)
        plan.close()
        assert np.all(got[val > 0] == np.inf) and np.all(got[val < 0] == -np.inf)
        assert np.isfinite(got[val == 0]).all()


@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("nu", range(11))
def test_infinite_point(nu, wide):
    bd = _bd()
    s = _system(nu, wide)
    rng = np.random.default_rng(nu)
    sign = rng.choice([-1.0, 1.0], size=s.nbands)
    mem = oracle.support(s.n, s.h, s.periodic, s.pos[0],
                         oracle.box_radius(s.sigma[0], s.numax[0], s.h))[1]
    psi = wl.psi_for(s)
    at = rng.choice(mem, size=s.nbands)  # a point per band
    spike = np.zeros(s.psi_shape)
    spike.reshape(-1, s.nbands)[at, np.arange(s.nbands)] = sign
    psi.reshape(-1, s.nbands)[at, np.arange(s.nbands)] = sign * np.inf
    val = oracle.project(*s.geometry(), spike)
    for flags in (bd.FLAG_DETERMINISTIC, 0):
        plan = bd.Plan.from_system(s, flags=flags)
        got = plan.project(torch.from_numpy(psi).cuda())
        torch.cuda.synchronize()
        got = got.cpu().numpy()
        plan.close()
        assert np.all(got[val > 0] == np.inf) and np.all(got[val < 0] == -np.inf)
        assert np.isfinite(got[val == 0]).all()
