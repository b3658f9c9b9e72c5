"""Squared setups, the third level and squared mixed-precision solves repeat, bit for
bit, the results of the library's first kernels for them: the checksums in
golden/squared_order.json (written by golden/make_squared_order.py with the library of
commit 095df9d).  A solve stops at a residual that leaves 1e-9 or more of error in D's
lowest modes, and one other order of sums redraws it.

Links and vectors are made with exact or single-rounding operations, so that every
host makes the same ones."""
import hashlib
import json
from pathlib import Path

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

GOLDEN = Path(__file__).with_name("golden") / "squared_order.json"

# every dof count of the ordered FP32 apply (and 24, the general kernel's), right-hand
# sides alone, in one group and in several; four sites to 256; the third level; enough
# FP64 sites for the tile kernel that such solves do not take
CASES = {
    "4c4x4_nv8": dict(L=(4, 4, 4, 4), Ls=4, block=2, nvec=8, counts=(1, 3)),
    "4c4x4_nv16": dict(L=(4, 4, 4, 4), Ls=4, block=2, nvec=16, counts=(1, 20)),
    "4c4x4_nv24": dict(L=(4, 4, 4, 4), Ls=4, block=2, nvec=24, counts=(3,)),
    "4c4x4_nv32": dict(L=(4, 4, 4, 4), Ls=4, block=2, nvec=32, counts=(5,)),
    "4c4x4_nv12": dict(L=(4, 4, 4, 4), Ls=4, block=2, nvec=12, counts=(3,)),
    "8c8x4_nv16": dict(L=(8, 8, 8, 8), Ls=4, block=2, nvec=16, counts=(1, 2, 6)),
    "8c8x4_nv24": dict(L=(8, 8, 8, 8), Ls=4, block=2, nvec=24, counts=(1, 4, 5, 12)),
    "8x8x8x4x4_nv24": dict(L=(8, 8, 8, 4), Ls=4, block=2, nvec=24, counts=(2, 8, 12)),
    "4c8x6_l2_nv8": dict(L=(4, 4, 4, 8), Ls=6, block=2, nvec=8, counts=(1, 3), level2=dict(block=(2, 2, 1, 2), nvec=8)),
    "8c8x4_l2_nv24": dict(L=(8, 8, 8, 8), Ls=4, block=2, nvec=24, counts=(2,), level2=dict(block=(2, 2, 2, 2), nvec=16)),
    "8c16x16_nv8": dict(L=(8, 8, 8, 16), Ls=16, block=4, nvec=8, counts=(8,)),
}


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


def exact_links(L, seed):
    """Unitary to rounding: plane rotations with Pythagorean cosines and phases of i."""
    rng = np.random.Generator(np.random.PCG64(seed))
    shp = tuple(L[::-1]) + (4,)
    cos, sin = np.array([3 / 5, 15 / 17, 21 / 29, 1.0]), np.array([4 / 5, 8 / 17, 20 / 29, 0.0])
    re = np.zeros(shp + (3, 3))
    re[..., 0, 0] = re[..., 1, 1] = re[..., 2, 2] = 1.0
    for i, j in ((0, 1), (1, 2), (0, 2)):
        k = rng.integers(0, 4, shp)
        c, s = cos[k][..., None], sin[k][..., None]
        a, b = re[..., i, :].copy(), re[..., j, :].copy()
        u, v = c * a, s * b
        p, q = s * a, c * b
        re[..., i, :], re[..., j, :] = u - v, p + q
    k = rng.integers(0, 4, shp + (3,))[..., None, :]
    unit_re, unit_im = np.array([1.0, 0.0, -1.0, 0.0])[k], np.array([0.0, 1.0, 0.0, -1.0])[k]
    U = np.zeros(shp + (3, 3), dtype=np.complex128)
    U.real, U.imag = re * unit_re, re * unit_im
    return U


def exact_vectors(shape, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    v = np.zeros(shape, dtype=np.complex128)
    v.real, v.imag = rng.integers(-2**20, 2**20, shape) / 2**19, rng.integers(-2**20, 2**20, shape) / 2**19
    return v


def digest(t):
    return hashlib.sha256(np.ascontiguousarray(t.cpu().numpy()).tobytes()).hexdigest()[:16]


def results(mg, case):
    """Checksums of the setup's basis, of the third level's parts and of the solutions."""
    L, Ls, nvec, block = case["L"], case["Ls"], case["nvec"], (case["block"],) * 4
    field = tuple(L[::-1]) + (Ls, 4, 3)
    h = mg.Handle(L, Ls, 1.75, 0.03125)
    mg.mgdwf_set_gauge(h, dev(exact_links(L, 11)))
    params = lambda prec: mg.make_mg_params(block, nvec, sweeps=2, sweep0_iters=6, sweep_iters=2, nu_pre=2, nu_post=2,
                                            coarse_tol=0.05, coarse_maxiter=24, fine_prec=prec, coarse_prec=prec,
                                            squared=True)
    mg.mgdwf_setup(h, params("f64"), dev(exact_vectors((nvec,) + field, 12)))
    V = torch.empty((nvec,) + field, dtype=torch.complex128, device="cuda")
    mg.mgdwf_get_basis(h, V)
    out = {"basis": digest(V)}
    if "level2" in case:
        p = mg.make_level2_params(case["level2"]["block"], case["level2"]["nvec"], null_iters=6, nu=2, coarse_tol=0.05,
                                  coarse_maxiter=24, gamma=2)
        W0 = exact_vectors((p.nvec,) + tuple(n // case["block"] for n in L[::-1]) + (2, nvec), 13)
        mg.mgdwf_setup_level2(h, p, dev(W0))
        out["level2"] = [digest(t) for t in mg.mgdwf_get_level2(h)]
    mg.mgdwf_set_mg_params(h, params("f32"))
    for n in case["counts"]:
        b = dev(exact_vectors((n,) + field, 14))
        x = torch.zeros_like(b)
        mg.mgdwf_solve(h, b, x, nrhs=n, tol=1e-12, max_outer=3, restart=8, allow_not_converged=True)
        out[f"solve{n}"] = digest(x)
    h.close()
    return out


@pytest.mark.parametrize("name", list(CASES))
def test_results_repeat_bit_for_bit(cuda, name):
    import paper_1205_2933_amd as mg
    assert results(mg, CASES[name]) == json.loads(GOLDEN.read_text())[name]
