"""FP64 results against 80-bit arithmetic on the host, where a kernel's order of
sums decides the last bits, and what non-finite inputs leave behind."""
import numpy as np
import pytest
import torch

from inputs import gaussian_fermion, prepare_gauge, random_starts
from oracle import dwf
from oracle.transfer import block_split

pytestmark = pytest.mark.gpu

LD = np.clongdouble


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


def rel(a, b):
    return float(np.sqrt((np.abs(a - b) ** 2).sum() / (np.abs(b) ** 2).sum()))


def handle_with_basis(L, Ls, block, nvec):
    import paper_1205_2933_amd as mg
    h = mg.Handle(L, Ls, 1.8, 0.02)
    mg.mgdwf_set_gauge(h, dev(prepare_gauge(L, 0.4, 91)))
    mg.mgdwf_set_nullvecs(h, block, dev(random_starts(L, Ls, nvec, 92)), nvec)
    V = torch.empty((nvec,) + h.fermion_shape, dtype=torch.complex128, device="cuda")
    mg.mgdwf_get_basis(h, V)
    return h, V


def panels(f, block):
    """(n, field) -> (n, coarse sites, chirality, rows) in 80 bits."""
    g = block_split(f, block)
    g = np.stack([g[..., :2, :], g[..., 2:, :]], axis=5)
    return g.reshape(f.shape[0], int(np.prod(g.shape[1:5])), 2, -1).astype(LD)


# right-hand sides below and above the four tiles that decide how often the sum is
# compensated, two and one rows per lane, blocks of one row group and of many
@pytest.mark.parametrize("L,Ls,block,nvec,n", [((4, 4, 8, 4), 8, (4, 4, 4, 4), 16, 2), ((4, 4, 4, 4), 16, (4, 4, 4, 4), 32, 9),
                                               ((4, 4, 4, 4), 16, (4, 4, 4, 4), 24, 27), ((8, 8, 4, 4), 4, (2, 2, 2, 2), 8, 12),
                                               ((4, 4, 4, 8), 5, (2, 2, 2, 2), 12, 3), ((4, 4, 4, 4), 10, (2, 2, 2, 2), 24, 5)])
def test_restrict_f64_rounding(cuda, L, Ls, block, nvec, n):
    """Bar: 2.2e-16 (two roundings).  The sums leave the rounding of chains of 8 or 16
    products, each chain's end exact to second order, and of one sum per workgroup."""
    import paper_1205_2933_amd as mg
    h, V = handle_with_basis(L, Ls, block, nvec)
    x = gaussian_fermion(L, Ls, 93, n=n)
    c = torch.empty((n, h.ncoarse), dtype=torch.complex128, device="cuda")
    mg.mgdwf_restrict(h, dev(x), c, nrhs=n)
    Vb, xb = panels(V.cpu().numpy(), block), panels(x, block)
    got = c.cpu().numpy().reshape(n, -1, 2, nvec).astype(LD)
    for r in (0, n - 1):
        want = np.stack([(np.conj(Vb[k]) * xb[r]).sum(-1) for k in range(nvec)], axis=-1)
        assert rel(got[r], want) < 2.2e-16, r
    h.close()


# row groups that fill blocks (a sum that is not finite is taken twice) and that do
# not (lanes past the block read its first row), FP64 and FP32
@pytest.mark.parametrize("L,Ls,block,prec", [((4, 4, 4, 4), 16, (4, 4, 4, 4), "f64"), ((3, 2, 2, 2), 5, (3, 1, 1, 1), "f64"),
                                             ((3, 2, 2, 2), 6, (3, 1, 1, 1), "f32"), ((4, 4, 4, 4), 8, (4, 4, 4, 4), "f32")])
@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan")])
def test_restrict_non_finite(cuda, L, Ls, block, prec, value):
    """One infinite entry in a block's first row makes that block's coefficients of one
    chirality and one right-hand side infinite (never NaN), and nothing else."""
    import paper_1205_2933_amd as mg
    nvec = 3
    h, V = handle_with_basis(L, Ls, block, nvec)
    x = gaussian_fermion(L, Ls, 94, n=3)
    x[1, 0, 0, 0, 0, 0, 0, 0] = complex(value, 0.25)
    c = torch.empty((3, h.ncoarse), dtype=torch.complex128, device="cuda")
    mg.mgdwf_restrict(h, dev(x), c, nrhs=3, prec=prec)
    got = c.cpu().numpy().reshape(3, -1, 2, nvec)
    hit = got[1, 0, 0].copy()
    got[1, 0, 0] = 0
    assert np.isfinite(got.view(np.float64)).all()
    parts = hit.view(np.float64)
    assert (np.isnan(parts) if np.isnan(value) else np.isinf(parts)).all(), hit
    h.close()


@pytest.mark.parametrize("dagger", [False, True])
def test_fp64_tile_kernel_rounding(cuda, dagger):
    """The tile kernel (enough fields for 2^20 sites) is no further from 80 bits than the
    plain kernel (one field).  Bar: 1.1 times; 2.5e5 entries fix the ratio to 1 %."""
    import paper_1205_2933_amd as mg
    L, Ls, n, bc = (8, 4, 4, 10), 16, 52, (1, 1, 1, -1)
    U = prepare_gauge(L, 0.4, 83)
    h = mg.Handle(L, Ls, 1.75, 0.02, bc=bc)  # 5 - M5 is exact
    mg.mgdwf_set_gauge(h, dev(U))
    psi = gaussian_fermion(L, Ls, 84)
    x = dev(np.broadcast_to(psi, (n,) + psi.shape))
    y = torch.empty_like(x)
    mg.mgdwf_apply_dwf(h, x, y, dagger=dagger, nrhs=n)
    one = torch.empty_like(x[0])
    mg.mgdwf_apply_dwf(h, x[0].contiguous(), one, dagger=dagger, nrhs=1)
    want = dwf.apply_dwf(psi.astype(LD), U.astype(LD), 1.75, 0.02, dagger=dagger, bc=bc)
    plain = rel(one.cpu().numpy().astype(LD), want)
    for k in (0, n - 1):
        assert rel(y[k].cpu().numpy().astype(LD), want) < 1.1 * plain, (k, plain)
    assert plain < 1.2e-16
    h.close()
