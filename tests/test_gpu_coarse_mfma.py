"""The MFMA coarse kernels over every dof count they are compiled for: the
D_c and D_c^+ apply against the stencil sum of the FP64 operator, and the coarse
CGNE steps of a batch of right-hand sides against the same right-hand sides
one at a time (another grid, and above 8192 partials another way of adding
them)."""
import numpy as np
import pytest
import torch

from inputs import gaussian_fermion, prepare_gauge, random_starts

pytestmark = pytest.mark.gpu

# FP32: 2e-6, the bar of the FP32 apply elsewhere.  16 bits: the operator and
# the vector each carry half a unit roundoff (2^-11, 2^-8) of their block or
# site maximum, about three times an entry's own size at these dof counts.
TOL = {"f32": 2e-6, "f16": 3 * 2.0 ** -11, "bf16": 3 * 2.0 ** -8}


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


def stencil(Dc, x, Lc, dagger):
    """sum_d Dc[X][d] x(X + delta_d), or its adjoint; arrays [t][z][y][x][...]."""
    y = torch.zeros_like(x)
    for d in range(9):
        mu, sg = (d - 1) >> 1, 1 if d & 1 else -1
        M = Dc[..., d, :, :]
        ax = 3 - mu
        if dagger:
            v = (M.conj().transpose(-1, -2).resolve_conj().contiguous() @ x.unsqueeze(-1)).squeeze(-1)
            y += v if d == 0 else torch.roll(v, sg, ax)
        else:
            v = x if d == 0 else torch.roll(x, -sg, ax)
            y += (M @ v.unsqueeze(-1)).squeeze(-1)
    return y


@pytest.mark.parametrize("nvec", [8, 16, 24, 32, 12])
def test_apply_every_dof_count(cuda, nvec):
    import paper_1205_2933_amd as mg
    L, Ls, block = (4, 4, 6, 2), 4, (2, 2, 2, 2)
    Lc = tuple(L[m] // 2 for m in range(4))
    h = mg.Handle(L, Ls, 1.8, 0.02)
    mg.mgdwf_set_gauge(h, dev(prepare_gauge(L, 0.4, 71)))
    mg.mgdwf_set_nullvecs(h, block, dev(random_starts(L, Ls, nvec, 72)), nvec)
    mg.mgdwf_build_coarse(h)
    n2 = 2 * nvec
    Dc = torch.empty(Lc[::-1] + (9, n2, n2), dtype=torch.complex128, device="cuda")
    mg.mgdwf_get_coarse_op(h, Dc)
    rng = np.random.default_rng(73)
    precs = ("f32", "f16", "bf16") if nvec % 8 == 0 else ("f32",)
    for nr in (1, 10, 16, 17):
        shp = (nr,) + Lc[::-1] + (n2,)
        x = dev(rng.standard_normal(shp) + 1j * rng.standard_normal(shp))
        for dagger in (False, True):
            want = torch.stack([stencil(Dc, x[r], Lc, dagger) for r in range(nr)])
            for prec in precs:
                for shape in (0, 1):
                    mg.mgdwf_set_coarse_tiling(h, shape)
                    y = torch.empty_like(x)
                    mg.mgdwf_apply_coarse(h, x, y, dagger=dagger, prec=prec, nrhs=nr)
                    e = float((y - want).norm() / want.norm())
                    assert e < TOL[prec], (nvec, nr, dagger, prec, shape, e)
    h.close()


@pytest.mark.parametrize("nvec,cprec,t", [(8, "f32", 18), (24, "f16", 2), (24, "f32", 2), (32, "bf16", 2), (16, "f16", 18)])
def test_batched_coarse_solve_equals_single(cuda, nvec, cprec, t):
    """Coarse CGNE fixed at 16 iterations: 17 right-hand sides (two column
    groups; with t = 18, 576 coarse sites, their sums go through the
    finalising launch) against two of them alone."""
    import paper_1205_2933_amd as mg
    L, Ls, block = (8, 8, 8, t), 2, (2, 2, 2, 2)
    h = mg.Handle(L, Ls, 1.8, 0.05)
    mg.mgdwf_set_gauge(h, dev(prepare_gauge(L, 0.3, 74)))
    mg.mgdwf_set_nullvecs(h, block, dev(random_starts(L, Ls, nvec, 75)), nvec)
    mg.mgdwf_build_coarse(h)
    mg.mgdwf_set_mg_params(h, mg.make_mg_params(block, nvec, nu_pre=1, nu_post=1, coarse_tol=1e-30, coarse_maxiter=16,
                                                fine_prec="f32", coarse_prec=cprec))
    b = dev(gaussian_fermion(L, Ls, 76, n=17))
    z = torch.empty_like(b)
    for _ in range(2):  # eager, then graph replays
        mg.mgdwf_apply_vcycle(h, b, z, nrhs=17)
        for r in (0, 16):
            one = torch.empty_like(b[r])
            mg.mgdwf_apply_vcycle(h, b[r].contiguous(), one, nrhs=1)
            e = float((one - z[r]).norm() / one.norm())
            # FP32 sums in another order, through 16 CG steps: the V-cycle's own bars
            assert e < {"f32": 1e-5, "f16": 0.1 * 2.0 ** -11, "bf16": 0.1 * 2.0 ** -8}[cprec], (r, e)
    h.close()
