"""The FP64 tile Dslash on the internal layout, as solves use it (D, D^+, the residual
form and the norms that it leaves): enough fields or sites for it (2^20 5D sites),
against the plain kernel on one field at a time, and against CG written out over
mgdwf_apply_dwf."""
import numpy as np
import pytest
import torch

from inputs import gaussian_fermion, prepare_gauge, random_starts

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


# 256 tiles times fields and more: whole t-ranges, dealt to the XCDs by field and z-slab;
# 52 fields: t in two chunks
@pytest.mark.parametrize("L,Ls,block,n,bc", [((8, 4, 4, 10), 16, (4, 2, 2, 5), 64, (-1, 1, 1, -1)),
                                             ((8, 4, 4, 10), 16, (4, 2, 2, 5), 52, (1, 1, 1, -1)),
                                             ((4, 4, 8, 13), 14, (2, 2, 4, 13), 64, (1, -1, -1, 1))])
def test_batched_solve_equals_single(cuda, L, Ls, block, n, bc):
    """Two steps of a squared FP64 solve (smoothers, residuals, coarse CG of a fixed length)
    on a batch, tile kernel, and on one field, plain kernel.  Bar 1e-9: a
    cycle turns one rounding into 1e-11 at most; one field's norm in another's place
    would change it by order one."""
    import paper_1205_2933_amd as mg
    nvec = 4
    assert L[0] * L[1] * L[2] * L[3] * Ls * n >= 2**20
    h = mg.Handle(L, Ls, 1.8, 0.05, bc=bc)
    mg.mgdwf_set_gauge(h, dev(prepare_gauge(L, 0.4, 61)))
    mg.mgdwf_set_nullvecs(h, block, dev(random_starts(L, Ls, nvec, 62)), nvec)
    mg.mgdwf_build_coarse_squared(h)
    mg.mgdwf_set_mg_params(h, mg.make_mg_params(block, nvec, nu_pre=2, nu_post=2, coarse_tol=1e-30, coarse_maxiter=7,
                                                fine_prec="f64", coarse_prec="f64", squared=True))
    b = dev(gaussian_fermion(L, Ls, 63, n=n) * (1.0 + np.arange(n)).reshape((n,) + (1,) * 7))
    x = torch.zeros_like(b)
    mg.mgdwf_solve(h, b, x, nrhs=n, tol=1e-13, max_outer=2, restart=8, allow_not_converged=True)
    for r in (0, 1, n // 2, n - 1):
        one = torch.zeros_like(b[r])
        mg.mgdwf_solve(h, b[r].contiguous(), one, nrhs=1, tol=1e-13, max_outer=2, restart=8, allow_not_converged=True)
        assert float(one.norm()) > 0
        assert float((one - x[r]).norm() / one.norm()) < 1e-9, r
    h.close()


def test_cgne_steps_in_t_chunks(cuda):
    """Five CG steps on D D^+ y = b, x = D^+ y, one field of 2^20 sites: t in chunks.  The
    same steps over mgdwf_apply_dwf (canonical fields, checked against the oracle
    elsewhere) with torch's sums.  Bar 1e-12: five steps, rounding 1e-16, condition of
    the steps' scalars of order one."""
    import paper_1205_2933_amd as mg
    L, Ls, bc, steps = (8, 16, 8, 64), 16, (1, 1, 1, -1), 5
    h = mg.Handle(L, Ls, 1.8, 0.02, bc=bc)
    mg.mgdwf_set_gauge(h, dev(prepare_gauge(L, 0.4, 85)))
    b = dev(gaussian_fermion(L, Ls, 86))

    def D(v, dagger=False):
        out = torch.empty_like(v)
        mg.mgdwf_apply_dwf(h, v, out, dagger=dagger, nrhs=1)
        return out

    x = torch.zeros_like(b)
    with pytest.raises(mg.MgdwfError):
        mg.mgdwf_cgne(h, b, x, tol=1e-14, max_iter=steps)
    want, r = torch.zeros_like(b), b.clone()
    p, rr = D(r, True), (r.abs() ** 2).sum()
    for _ in range(steps):
        a = rr / (p.abs() ** 2).sum()
        want += a * p
        r -= a * D(p)
        new = (r.abs() ** 2).sum()
        p = D(r, True) + (new / rr) * p
        rr = new
    assert float((x - want).norm() / want.norm()) < 1e-12
    h.close()
