"""The plane form of the projection with one and two waves to an atom plane (1024
and more units; little and much overlap), over the cut-offs, one and two bands
per lane, odd band counts: FP64, deterministic and Bloch plans, and FP32 where
it takes the form.  Against the oracle, |c - c_oracle| <= 1e-12 A, in FP32
2 k u A with k = 3 (points along an axis) + 12 (+ 4 for the Bloch phases)."""
import numpy as np
import pytest

import oracle
from paper_1905_00480_amd import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# cut-off, bands, waves
CASES = {"nu%d_bands%d_waves%d" % c: c for c in
         [(nu, b, 2) for nu, b in ((0, 70), (1, 65), (2, 97), (3, 66), (4, 101), (5, 98), (6, 99),
                                   (7, 101), (8, 102), (9, 129), (10, 130), (4, 13), (7, 16))] +
         [(nu, b, 1) for nu, b in ((0, 66), (1, 67), (2, 98), (3, 101), (4, 102), (5, 99), (6, 130),
                                   (7, 97), (8, 98), (9, 101), (10, 66), (3, 15), (5, 16), (8, 14))]}


def system(nu, nbands, waves):
    groups = -(-nbands // 32) if nbands > 16 else 1
    planes = 2 * int((0.6 * np.sqrt(2 * nu + 3) + 0.4) / 0.2)
    natoms = 2 + -(-1100 // (groups * planes))
    if waves == 1:  # supports overlap four times and more
        r3 = 4.19 * (planes / 2 + 0.3) ** 3
        n = int(min(40, max(planes + 2, (natoms * r3 / 6.5) ** (1 / 3))))
        natoms = max(natoms, int(5.5 * n ** 3 / r3) + 1)
        return wl.make_system("waves", (n, n - 1, n), 0.2, (True, True, True), natoms, 0.6, nu,
                              nbands, 900 + nu + nbands)
    n = 34 if natoms < 20 and nu < 8 else 42 if natoms < 20 else 52
    return wl.make_system("waves", (n + 3, n, n - 1), 0.2, (True, True, True), natoms, 0.6, nu,
                          nbands, 900 + nu + nbands)


def _bd():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1905_00480_amd import binding
    binding.load_library()
    return binding


def _check(got, ref, bound, what):
    d = got.ravel() - ref.ravel()
    err = np.maximum(np.abs(d.real), np.abs(d.imag))
    assert np.all(err <= bound.ravel() + 1e-300), "%s: max |d| %.3e" % (what, float(err.max()))


@pytest.mark.parametrize("name", sorted(CASES))
def test_plane_form_by_its_waves(name):
    bd = _bd()
    nu, nbands, waves = CASES[name]
    s = system(nu, nbands, waves)
    atoms = np.array([0, s.natoms // 2, s.natoms - 1])
    sub = s.subset(atoms)
    off = oracle.coeff_offsets(s.numax, s.nbands)
    psi = wl.psi_for(s)
    ref, ab = oracle.project(*sub.geometry(), psi, with_abs=True)

    def run(flags, d_psi, kpoint=None):
        plan = bd.Plan.from_system(s, flags=flags)
        assert plan.forms()[:2] == (bd.FORM_PLANES, waves)
        if kpoint:
            plan.set_kpoint(kpoint)
        c = plan.project(d_psi)
        torch.cuda.synchronize()
        plan.close()
        return np.concatenate([c.cpu().numpy()[off[a]:off[a + 1]] for a in atoms])

    d_psi = torch.from_numpy(psi).cuda()
    got = run(0, d_psi)
    _check(got, ref, 1e-12 * ab, "f64")
    assert np.array_equal(got, run(bd.FLAG_DETERMINISTIC, d_psi))
    k = 3 * (2 * int(np.ceil((0.6 * np.sqrt(2 * nu + 3) + 0.4) / 0.2)) + 2) + 12
    if waves == 1 and nbands % 2 == 0:
        p32 = psi.astype(np.float32)
        r32, a32 = oracle.project(*sub.geometry(), p32.astype(np.float64), with_abs=True)
        _check(run(bd.FLAG_FP32, torch.from_numpy(p32).cuda()), r32, 2.0 ** -23 * k * a32, "f32")
    zpsi = psi[..., ::-1] * 1j + psi
    kp = (0.7, -0.3, 1.1)
    rk, ak = oracle.project_k(*sub.geometry(), zpsi, kp, with_abs=True)
    _check(run(bd.FLAG_BLOCH, torch.from_numpy(zpsi).cuda(), kp), rk, 1e-12 * ak, "bloch")
