"""Fine-operator calls on canonical fields (one launch) and through the packed
internal layout: both against the oracle, on site counts that fill no
workgroup, odd ones among them."""
import numpy as np
import pytest
import torch

from inputs import gaussian_fermion, prepare_gauge
from oracle import dwf

pytestmark = pytest.mark.gpu

TOL = {"f64": 1e-13, "f32": 2e-6}  # the bars of the operator tests


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


# (lattice, Ls, fields): FP32 above 2^20 numbers is packed; V5 odd, V5 even but no
# multiple of 128, fewer sites than one workgroup, antiperiodic faces
@pytest.mark.parametrize("L,Ls,n,bc", [((9, 7, 5, 11), 5, 6, (1, 1, 1, -1)), ((6, 5, 7, 9), 10, 5, (-1, 1, 1, 1)),
                                       ((2, 3, 2, 2), 1, 1, (1, -1, 1, -1)), ((3, 2, 5, 2), 7, 2, (1, 1, -1, 1))])
@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_canonical_and_packed(cuda, L, Ls, n, bc, prec):
    import paper_1205_2933_amd as mg
    U = prepare_gauge(L, 0.4, 81)
    h = mg.Handle(L, Ls, 1.7, 0.03, bc=bc)
    mg.mgdwf_set_gauge(h, dev(U))
    psi = gaussian_fermion(L, Ls, 82, n=n)
    x = dev(psi)
    for dagger in (False, True):
        y = torch.full_like(x, float("nan"))
        mg.mgdwf_apply_dwf(h, x, y, dagger=dagger, prec=prec, nrhs=n)
        want = dwf.apply_dwf(psi[n - 1], U, 1.7, 0.03, dagger=dagger, bc=bc)
        e = np.linalg.norm(y[n - 1].cpu().numpy() - want) / np.linalg.norm(want)
        assert e < TOL[prec], e
        for k in range(n):  # one field at a time takes the canonical path
            one = torch.empty_like(x[k])
            mg.mgdwf_apply_dwf(h, x[k].contiguous(), one, dagger=dagger, prec=prec, nrhs=1)
            e = float((one - y[k]).norm() / one.norm())
            assert e < TOL[prec], (k, e)
    h.close()


@pytest.mark.parametrize("L,Ls,n,bc", [((8, 4, 4, 10), 16, 52, (-1, 1, 1, -1)), ((4, 4, 2, 13), 14, 181, (1, -1, -1, 1))])
def test_fp64_tile_kernel_against_plain(cuda, L, Ls, n, bc):
    """Enough fields for the FP64 tile kernel (2^20 sites) against the plain
    kernel on one field at a time and the oracle: one tile wide in a direction,
    odd t, antiperiodic faces; canonical fields (apply_dwf)."""
    import paper_1205_2933_amd as mg
    U = prepare_gauge(L, 0.4, 83)
    h = mg.Handle(L, Ls, 1.8, 0.02, bc=bc)
    mg.mgdwf_set_gauge(h, dev(U))
    psi = gaussian_fermion(L, Ls, 84, n=n)
    x = dev(psi)
    for dagger in (False, True):
        y = torch.full_like(x, float("nan"))
        mg.mgdwf_apply_dwf(h, x, y, dagger=dagger, nrhs=n)
        want = dwf.apply_dwf(psi[n - 1], U, 1.8, 0.02, dagger=dagger, bc=bc)
        assert np.linalg.norm(y[n - 1].cpu().numpy() - want) / np.linalg.norm(want) < TOL["f64"]
        for k in range(n):
            one = torch.empty_like(x[k])
            mg.mgdwf_apply_dwf(h, x[k].contiguous(), one, dagger=dagger, nrhs=1)
            assert float((one - y[k]).norm() / one.norm()) < TOL["f64"], k
    h.close()


def test_fp64_tile_kernel_t_chunks(cuda):
    """One field of 2^20 sites: t in chunks, against the oracle; canonical fields
    and (CGNE, which stops at once) the residual form on the internal layout."""
    import paper_1205_2933_amd as mg
    L, Ls, bc = (8, 16, 8, 64), 16, (1, 1, 1, -1)
    U = prepare_gauge(L, 0.4, 85)
    h = mg.Handle(L, Ls, 1.8, 0.02, bc=bc)
    mg.mgdwf_set_gauge(h, dev(U))
    psi = gaussian_fermion(L, Ls, 86)
    x = dev(psi)
    y = torch.empty_like(x)
    mg.mgdwf_apply_dwf(h, x, y, nrhs=1)
    want = dwf.apply_dwf(psi, U, 1.8, 0.02, bc=bc)
    assert np.linalg.norm(y.cpu().numpy() - want) / np.linalg.norm(want) < TOL["f64"]
    z = torch.empty_like(x)
    mg.mgdwf_apply_dwf(h, x, z, dagger=True, nrhs=1)
    # <D x, y> = <x, D^+ y> with y = D x, and D^+ x through D: <x, D x> = <D^+ x, x>
    a = torch.vdot(x.reshape(-1), y.reshape(-1))
    b = torch.vdot(z.reshape(-1), x.reshape(-1))
    assert abs(complex(a - b)) < 1e-12 * float(x.norm() * y.norm())
    sol = x.clone()
    rep = mg.mgdwf_cgne(h, y, sol, tol=1e-12)  # x solves D x = y: residual at rounding on entry
    assert rep["outer_iters"] == 0 and torch.equal(sol, x)
    assert rep["true_relres"] < 1e-13
    h.close()
