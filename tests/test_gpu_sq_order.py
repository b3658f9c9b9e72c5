"""Squared mixed-precision solves, whose coarse sums keep one order: every dof count
and every number of right-hand sides per workgroup of the ordered FP32 apply, a last
group that is partly empty, and dof counts of the general kernel (nvec 12)."""
import numpy as np
import pytest
import torch

from inputs import gaussian_fermion, prepare_gauge, random_starts

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


# 16 coarse sites: one right-hand side per workgroup; 256 sites: 1, 2, 4 and 8
@pytest.mark.parametrize("L,nvec,counts", [((4, 4, 4, 4), 8, (1, 3)), ((4, 4, 4, 4), 32, (5,)), ((4, 4, 4, 4), 12, (3,)),
                                           ((8, 8, 8, 8), 16, (2, 3)), ((8, 8, 8, 8), 24, (1, 5, 9))])
def test_one_mixed_step_follows_fp64(cuda, L, nvec, counts):
    """The first iterate of a solve (one cycle, seven coarse CG steps without a test in
    between) in mixed precision against FP64.  Bar: seven CG steps and eight smoother
    steps of FP32 rounding (6e-8 each, largest amplification per step about ten) stay
    below 1e-4; a row, column or right-hand side out of place changes it by order one."""
    import paper_1205_2933_amd as mg
    Ls, block = 4, (2, 2, 2, 2)
    h = mg.Handle(L, Ls, 1.8, 0.05)
    mg.mgdwf_set_gauge(h, dev(prepare_gauge(L, 0.4, 95)))
    params = lambda prec: mg.make_mg_params(block, nvec, sweeps=1, sweep0_iters=30, nu_pre=4, nu_post=4, coarse_tol=0.1,
                                            coarse_maxiter=7, fine_prec=prec, coarse_prec=prec, squared=True)
    mg.mgdwf_setup(h, params("f64"), dev(random_starts(L, Ls, nvec, 96)))
    for n in counts:
        b = torch.stack([dev(gaussian_fermion(L, Ls, 97 + r)) for r in range(n)])
        x = {}
        for prec in ("f64", "f32"):
            mg.mgdwf_set_mg_params(h, params(prec))
            x[prec] = torch.zeros_like(b)
            mg.mgdwf_solve(h, b, x[prec], nrhs=n, tol=1e-9, max_outer=1, restart=8, allow_not_converged=True)
        for r in range(n):
            e = float((x["f32"][r] - x["f64"][r]).norm() / x["f64"][r].norm())
            assert e < 1e-4, (n, r, e)
    h.close()
