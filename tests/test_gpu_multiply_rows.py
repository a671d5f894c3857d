"""The atomic-matrix product by row blocks, which many (atom, 32-band tile) pairs
take (more than 1024, from cut-off 8 on more than 4096): the loop over the row
blocks of a wave, blocks past the fourth wave's, second band tiles and mixed
cut-offs.  Sampled atoms against numpy: both sum N <= 286 terms,
|d - d_ref| <= 2 * 286 * 2^-53 * (|D| |c|), below the 1e-12 taken here."""
import numpy as np
import pytest

import oracle
from paper_1905_00480_amd import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("numax,natoms,nbands", [((5, 5), 520, 33), ((6, 6), 530, 64),
                                                 ((7, 7), 350, 90), ((0, 7), 1100, 17),
                                                 ((8, 8), 170, 790), ((9, 9), 130, 1030),
                                                 ((10, 10), 100, 1320), ((0, 10), 600, 230)])
def test_multiply_by_row_blocks(numax, natoms, nbands):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1905_00480_amd import binding as bd
    assert natoms * -(-nbands // 32) > (4096 if numax[1] >= 8 else 1024)
    s = wl.make_system("rows", (12, 11, 10), 0.3, (True,) * 3, natoms, 0.5, 0, nbands, 5)
    rng = np.random.default_rng(nbands)
    s.numax = rng.integers(numax[0], numax[1] + 1, size=natoms).astype(np.int32)
    s.numax[0] = numax[1]
    off, coff = oracle.matrix_offsets(s.numax), oracle.coeff_offsets(s.numax, s.nbands)
    gen = torch.Generator(device="cuda").manual_seed(nbands)
    D = torch.randn(int(off[-1]), generator=gen, dtype=torch.float64, device="cuda")
    c = torch.randn(int(coff[-1]), generator=gen, dtype=torch.float64, device="cuda")
    d = torch.full_like(c, float("nan"))
    plan = bd.Plan.from_system(s)
    plan.multiply(D, c, d)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(d).all())
    for a in np.unique(np.concatenate([[0, natoms - 1], rng.choice(natoms, 6, replace=False)])):
        N = oracle.nsho(int(s.numax[a]))
        Da = D[off[a]:off[a + 1]].cpu().numpy().reshape(N, N)
        ca = c[coff[a]:coff[a + 1]].cpu().numpy().reshape(N, nbands)
        err = np.abs(d[coff[a]:coff[a + 1]].cpu().numpy().reshape(N, nbands) - Da @ ca)
        assert np.all(err <= 1e-12 * (np.abs(Da) @ np.abs(ca)))
    plan.close()
