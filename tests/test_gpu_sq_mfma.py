"""The squared coarse operator's MFMA kernels over their dof counts, row splits and
right-hand-side groups: the apply against the sum over the 33 offsets of the FP64
operator, and the coarse CG inside a V-cycle on a batch against the same fields
one at a time (another grid and another grouping)."""
import numpy as np
import pytest
import torch

from inputs import gaussian_fermion, prepare_gauge, random_starts

pytestmark = pytest.mark.gpu

TOL = {"f64": 1e-13, "f32": 2e-6}  # the bars of the squared operator's tests


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


def offsets():
    out = [(0, 0, 0, 0)]
    unit = lambda mu, s: tuple(s if m == mu else 0 for m in range(4))
    for mu in range(4):
        out += [unit(mu, 1), unit(mu, -1)]
    for mu in range(4):
        for nu in range(mu + 1, 4):
            for s in (1, -1):
                for r in (1, -1):
                    out.append(tuple(s if m == mu else (r if m == nu else 0) for m in range(4)))
    return out


# coarse sites x groups below and above 256 (a site's rows split or together), 256
# sites or more with 9 right-hand sides (two column tiles); nvec 12: the scalar kernel
@pytest.mark.parametrize("L,nvec", [((4, 4, 6, 4), 8), ((4, 4, 6, 4), 24), ((4, 4, 4, 4), 32), ((4, 4, 4, 4), 12),
                                    ((8, 8, 8, 8), 16), ((8, 8, 8, 8), 24), ((8, 8, 8, 4), 32)])
def test_apply_matches_stencil(cuda, L, nvec):
    import paper_1205_2933_amd as mg
    Ls, block = 2, (2, 2, 2, 2)
    Lc = tuple(n // 2 for n in L)
    h = mg.Handle(L, Ls, 1.8, 0.05)
    mg.mgdwf_set_gauge(h, dev(prepare_gauge(L, 0.4, 95)))
    mg.mgdwf_set_nullvecs(h, block, dev(random_starts(L, Ls, nvec, 96)), nvec)
    mg.mgdwf_build_coarse_squared(h)
    n2 = 2 * nvec
    A = torch.empty(Lc[::-1] + (33, n2, n2), dtype=torch.complex128, device="cuda")
    mg.mgdwf_get_coarse_op(h, A)
    rng = np.random.default_rng(97)
    for nr in (1, 8, 9, 17):
        shp = (nr,) + Lc[::-1] + (n2,)
        x = dev(rng.standard_normal(shp) + 1j * rng.standard_normal(shp))
        want = torch.zeros_like(x)
        for o, d in enumerate(offsets()):
            y = torch.roll(x, tuple(-d[3 - ax] for ax in range(4)), dims=(1, 2, 3, 4))
            M = A[..., o, :, :].contiguous()
            for r in range(nr):
                want[r] += (M @ y[r].unsqueeze(-1)).squeeze(-1)
        for prec in ("f64", "f32"):
            got = torch.full_like(x, float("nan"))
            mg.mgdwf_apply_coarse(h, x, got, prec=prec, nrhs=nr)
            e = float((got - want).norm() / want.norm())
            assert e < TOL[prec], (nr, prec, e)
    h.close()


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("L,nvec", [((4, 4, 4, 4), 24), ((8, 8, 8, 8), 8)])
def test_batched_coarse_cg_equals_single(cuda, L, nvec, prec):
    import paper_1205_2933_amd as mg
    Ls, block = 4, (2, 2, 2, 2)
    h = mg.Handle(L, Ls, 1.8, 0.1)
    mg.mgdwf_set_gauge(h, dev(prepare_gauge(L, 0.3, 98)))
    mg.mgdwf_set_nullvecs(h, block, dev(random_starts(L, Ls, nvec, 99)), nvec)
    mg.mgdwf_build_coarse_squared(h)
    mg.mgdwf_set_mg_params(h, mg.make_mg_params(block, nvec, nu_pre=1, nu_post=1, coarse_tol=1e-30, coarse_maxiter=12,
                                                fine_prec=prec, coarse_prec=prec, squared=True))
    b = dev(gaussian_fermion(L, Ls, 94, n=17))
    z = torch.empty_like(b)
    mg.mgdwf_apply_vcycle(h, b, z, nrhs=17)
    for r in (0, 8, 16):
        one = torch.empty_like(b[r])
        mg.mgdwf_apply_vcycle(h, b[r].contiguous(), one, nrhs=1)
        # twelve CG steps on sums in another order (the V-cycle's own bars)
        assert float((one - z[r]).norm() / one.norm()) < {"f64": 1e-10, "f32": 1e-5}[prec]
    h.close()
