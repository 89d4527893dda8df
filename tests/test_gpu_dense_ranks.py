"""CP-ALS and the GD gradient at the ranks where the dense steps change
kernels, against the oracle: the block Gauss-Jordan (33 to 128, register tiles
of 2, 3 and 4) and the one past it, the spread lambda step (above 40), the
Grams of 5 to 16 column tiles (above 64), the row maps of any rank up to 128
(tiles of 1 to 8, one or two per wave) and the per-element ones past them.

N(0,1) factors and a ridge of 1 keep kappa(H) at a few dozen, so the flat
tolerance of the parity tests holds: relative Frobenius error 1e-5 in FP32
(kappa times the 1e-7 of the FP32 sums), one BF16 unit with BF16 storage.
"""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import build, factors_to_dev, rel_fro, say, to_host64, DEV
from paper_1406_4519_amd import dfacto, gen

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def problem():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ctx = dfacto.Context(0)
    coo = gen.zipf_distinct((701, 403, 257), 40_000, 1.1, seed=9)  # no row count a multiple of 16
    t = build(ctx, coo)
    yield ctx, coo, t
    torch.cuda.synchronize()
    t.close()
    ctx.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("R", [2, 15, 17, 31, 33, 41, 49, 65, 81, 96, 97, 113, 128, 129, 192])
def test_als_gd(problem, R, dtype):
    ctx, coo, t = problem
    rng = np.random.default_rng(R)
    F0 = [rng.standard_normal((d, R)) for d in coo.dims]
    tol = 1e-5 if dtype == "f32" else 2.0 ** -8
    say(f"  R={R} {dtype}")
    Fd, Fw = factors_to_dev(F0, dtype)
    lam = torch.zeros(R, dtype=torch.float64, device=DEV)
    fit = torch.zeros(1, dtype=torch.float64, device=DEV)
    dfacto.als_iter(ctx, t, Fd, lam, fit, reg=1.0)
    A, B, C, lam_ref, info = oracle.als_iter(*coo.arrays64(), coo.dims, Fw, 1.0,
                                             store="f64" if dtype == "f32" else "bf16")
    assert max(rel_fro(to_host64(x), ref) for x, ref in zip(Fd, (A, B, C))) <= tol
    assert rel_fro(lam.cpu().numpy(), lam_ref) <= tol
    assert abs(fit.item() - info["fit"]) <= (1e-6 if dtype == "f32" else 1e-4)
    Fd, Fw = factors_to_dev(F0, dtype)
    grads = [torch.empty((d, R), device=DEV) for d in coo.dims]
    f = torch.zeros(1, dtype=torch.float64, device=DEV)
    dfacto.gd_grad(ctx, t, Fd, grads, f, reg=0.5)
    gref, fref = oracle.gd_grad(*coo.arrays64(), coo.dims, Fw, 0.5)
    assert max(rel_fro(to_host64(g), ref) for g, ref in zip(grads, gref)) <= 1e-5
    assert abs(f.item() - fref) <= 1e-6 * abs(fref)


@pytest.mark.parametrize("R", [36, 70])
def test_singular_gram(problem, R):
    """Two equal columns: the block Gauss-Jordan meets a zero pivot and the
    pseudo-inverse takes over (the tolerance of the parity tests' own case)."""
    ctx, coo, t = problem
    rng = np.random.default_rng(R)
    F0 = [rng.standard_normal((d, R)) for d in coo.dims]
    for m in (1, 2):
        F0[m][:, R - 2] = F0[m][:, 1]
    Fd, Fw = factors_to_dev(F0, "f32")
    lam = torch.zeros(R, dtype=torch.float64, device=DEV)
    fit = torch.zeros(1, dtype=torch.float64, device=DEV)
    dfacto.als_iter(ctx, t, Fd, lam, fit)
    A, B, C, lam_ref, info = oracle.als_iter(*coo.arrays64(), coo.dims, Fw)
    assert info["pinv_mask"] & 1
    assert max(rel_fro(to_host64(x), ref) for x, ref in zip(Fd, (A, B, C))) <= 1e-4
