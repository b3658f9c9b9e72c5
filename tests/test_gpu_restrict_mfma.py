"""The MFMA restriction over its tile counts: basis columns below, at and above
16, right-hand sides at the edges of the eight-column tiles and of the 32 a
launch takes, fifth dimensions that fill its row groups and that do not, blocks
of few rows; against the oracle's R on the installed basis, and the block
orthonormality that its Gram matrices give."""
import numpy as np
import pytest
import torch

from inputs import gaussian_fermion, prepare_gauge, random_starts
from oracle import transfer as ot

pytestmark = pytest.mark.gpu

TOL = {"f64": 1e-13, "f32": 2e-6}  # the bars of the transfer tests


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


@pytest.mark.parametrize("L,block,Ls,nvec", [((4, 4, 4, 2), (2, 2, 2, 1), 8, 24), ((4, 2, 6, 4), (2, 2, 3, 2), 6, 16),
                                             ((2, 4, 2, 4), (1, 2, 1, 2), 5, 17), ((4, 4, 2, 2), (4, 2, 2, 2), 4, 32),
                                             ((3, 2, 2, 2), (1, 1, 1, 1), 2, 3)])
def test_restrict_tiles(cuda, L, block, Ls, nvec):
    import paper_1205_2933_amd as mg
    h = mg.Handle(L, Ls, 1.8, 0.02)
    mg.mgdwf_set_gauge(h, dev(prepare_gauge(L, 0.4, 91)))
    mg.mgdwf_set_nullvecs(h, block, dev(random_starts(L, Ls, nvec, 92)), nvec)
    Vh = torch.empty((nvec,) + h.fermion_shape, dtype=torch.complex128, device="cuda")
    mg.mgdwf_get_basis(h, Vh)
    Vn = Vh.cpu().numpy()
    # <v_i, v_j> on every block and chirality through R itself: the identity
    c = torch.empty((nvec, h.ncoarse), dtype=torch.complex128, device="cuda")
    mg.mgdwf_restrict(h, Vh, c, nrhs=nvec)
    G = c.reshape(nvec, -1, 2, nvec)
    eye = torch.eye(nvec, dtype=torch.complex128, device="cuda")[:, None, None, :]
    assert float((G - eye).abs().max()) < 1e-12
    for n in (2, 8, 9, 17, 25, 33):
        x = gaussian_fermion(L, Ls, 93, n=n)
        want = np.stack([ot.restrict(x[r], Vn, block) for r in range(n)]).reshape(n, -1)
        for prec in ("f64", "f32"):
            got = torch.full((n, h.ncoarse), float("nan"), dtype=torch.complex128, device="cuda")
            mg.mgdwf_restrict(h, dev(x), got, nrhs=n, prec=prec)
            e = np.linalg.norm(got.cpu().numpy() - want) / np.linalg.norm(want)
            assert e < TOL[prec], (n, prec, e)
    h.close()
