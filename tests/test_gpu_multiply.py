"""The atomic-matrix product d_a = D_a c_a where its kernel's split can go
wrong: every cut-off alone (row blocks of 16 and their remainders, waves with
no part of m), bands around the tile of 32, and mixed cut-offs (row blocks that
an atom does not have).  Against the product in numpy: both sum N <= 286 terms,
|d - d_ref| <= 2 * 286 * 2^-53 * (|D| |c|), below the 1e-12 taken here."""
import numpy as np
import pytest

import oracle
from paper_1905_00480_amd import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("numax,nbands", [([nu], b) for nu in range(11) for b in (1, 21)] +
                         [([6], b) for b in (15, 16, 17, 31, 32, 33, 65)] +
                         [([0, 10, 3, 0, 7], 34), ([2, 1, 0], 5), ([2, 0, 3, 1] * 300, 3)],
                         ids=lambda v: None if isinstance(v, int) else "%d_%d" % (len(v), max(v)))
def test_multiply_splits(numax, nbands):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1905_00480_amd import binding as bd
    s = wl.make_system("mul", (12, 11, 10), 0.3, (True,) * 3, len(numax), 0.5, 0, nbands, 5)
    s.numax = np.array(numax, dtype=np.int32)
    rng = np.random.default_rng(nbands)
    off = oracle.matrix_offsets(s.numax)
    D, c = rng.standard_normal(int(off[-1])), wl.coeffs_for(s)
    plan = bd.Plan.from_system(s)
    d = torch.full((c.size,), float("nan"), dtype=torch.float64, device="cuda")
    plan.multiply(torch.from_numpy(D).cuda(), torch.from_numpy(c).cuda(), d)
    torch.cuda.synchronize()
    d = d.cpu().numpy()
    coff = oracle.coeff_offsets(s.numax, s.nbands)
    for a in range(s.natoms):
        N = oracle.nsho(int(s.numax[a]))
        Da = D[off[a]:off[a + 1]].reshape(N, N)
        ca = c[coff[a]:coff[a + 1]].reshape(N, nbands)
        err = np.abs(d[coff[a]:coff[a + 1]].reshape(N, nbands) - Da @ ca)
        assert np.all(err <= 1e-12 * (np.abs(Da) @ np.abs(ca)))
    plan.close()
