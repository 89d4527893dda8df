"""Joint ALS rows of at most 7 ratings whose own system fails the pivot test:
they are solved from P^-1 where P = mu H + lam I passes its test, mode by mode,
and are a named failure where it does not."""
import numpy as np
import pytest
import torch

from gpu_util import build, say, to_host64, DEV
from paper_1406_4519_amd import dfacto, gen

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -52


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = dfacto.Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


def _ratings(ctx, dims, yi, yj, yv):
    d = [torch.from_numpy(np.asarray(a).astype(np.int32)).to(DEV) for a in (yi, yj)]
    return dfacto.build_ratings(ctx, dims, d[0], d[1], torch.from_numpy(np.asarray(yv, dtype=np.float32)).to(DEV))


def _users_fail_items_hold(ctx, unrated):
    """R = 2, lam = 1e-17, the word factor's second column zero.  User 0 has
    one rating: its system vv^T + P fails the test and P = diag(~2e-17, lam)
    passes.  With the large ratings the items' P = diag(> 1, lam) fails, but
    every rated item's own system is that of 11 generic users.  `unrated` more
    items have no rating, so their system is P itself."""
    I, J, K, lam = 12, 9 + unrated, 3, 1e-17
    rng = np.random.default_rng(5)
    yi, yj = np.meshgrid(np.arange(1, I), np.arange(9), indexing="ij")
    yi, yj = np.append(yi.ravel(), 0), np.append(yj.ravel(), 0)
    yv = (1e9 * rng.uniform(0.5, 1.5, len(yi))).astype(np.float32)
    F = [rng.uniform(0.5, 1.5, (d, 2)).astype(np.float32) for d in (I, J, K)]
    F[2] = np.stack([np.full(K, 5e-10), np.zeros(K)], 1).astype(np.float32)
    X = gen.uniform_distinct((I, J, K), 40, seed=6)
    # the pivot test is d > R eps max diag
    H0 = (F[1].astype(np.float64).T @ F[1]) * (F[2].astype(np.float64).T @ F[2])
    assert lam > 100 * 2 * EPS * H0[0, 0] and 3 * (H0[0, 0] + lam) < 2 * EPS * 0.25
    return (I, J), lam, (yi, yj, yv), F, build(ctx, X)


def test_modes_decide_for_themselves(ctx):
    """A user row that needs P^-1 does not send the item rows, whose P fails
    its test but which all pass theirs, the same way."""
    dims, lam, y, F, X = _users_fail_items_hold(ctx, 0)
    Y = _ratings(ctx, dims, *y)
    Fd = [torch.from_numpy(f).to(DEV) for f in F]
    dfacto.joint_als_iter(ctx, X, Y, Fd, 1.0, lam)
    torch.cuda.synchronize()
    A, B = to_host64(Fd[0]), to_host64(Fd[1])
    C = F[2].astype(np.float64)
    M = to_host64(dfacto.mttkrp(ctx, X, 1, [Fd[0], torch.from_numpy(F[1]).to(DEV), torch.from_numpy(F[2]).to(DEV)]))
    H = (A.T @ A) * (C.T @ C)
    assert 2 * EPS * H[0, 0] > 10 * lam
    for j in range(dims[1]):
        e = np.flatnonzero(y[1] == j)
        V = A[y[0][e]]
        S = H + lam * np.eye(2) + V.T @ V
        x = np.linalg.solve(S, V.T @ y[2][e].astype(np.float64) + M[j])
        # stored in FP32; the solve is backward stable in FP64
        tol = 1.01 * 2.0 ** -24 + 128 * EPS * np.linalg.cond(S)
        assert np.linalg.norm(B[j] - x) <= tol * np.linalg.norm(x), j
    X.close()
    Y.close()


def test_short_row_without_a_valid_inverse_is_a_failure(ctx):
    """An unrated item's system is P, which fails: nothing can solve it."""
    dims, lam, y, F, X = _users_fail_items_hold(ctx, 1)
    Y = _ratings(ctx, dims, *y)
    with pytest.raises(dfacto.DfactoError) as err:
        dfacto.joint_als_iter(ctx, X, Y, [torch.from_numpy(f).to(DEV) for f in F], 1.0, lam)
    assert err.value.status == dfacto.E_NUMERIC
    X.close()
    Y.close()


@pytest.mark.parametrize("mu", [0.0, 1.0])
@pytest.mark.parametrize("R", [6, 16, 32])
def test_short_rows_have_the_ridge_solution(ctx, R, mu):
    """Rows of fewer than min(8, R) ratings with P of about 1e-17 (mu = 0: lam I;
    mu = 1: word factors of 1e-10): S = P + V^T V fails the test, and x is
    z0 + P^-1 V^T K^-1 (y - V z0), z0 = mu P^-1 M[row], K = I + V P^-1 V^T
    (S^-1 V^T = P^-1 V^T K^-1), nothing of which is ill-conditioned."""
    I, J, K, lam = 151, 211, 20, 1e-17
    rng = np.random.default_rng(5)
    n = [r % 8 if r % 8 < R else 0 for r in range(I)]
    yi = np.repeat(np.arange(I), n)
    yj = np.arange(len(yi)) % J  # no item more than 3 times
    yv = rng.integers(1, 6, len(yi)).astype(np.float64)
    Y = _ratings(ctx, (I, J), yi, yj, yv)
    coo = gen.uniform_distinct((I, J, K), 6000, seed=72)
    coo.val *= np.float32(1e-7)
    X = build(ctx, coo)
    F = [rng.uniform(0, 1, (d, R)).astype(np.float32) for d in (I, J, K)]
    F[2] *= np.float32(1e-10)
    Fd = [torch.from_numpy(f).to(DEV) for f in F]
    dfacto.joint_als_iter(ctx, X, Y, Fd, mu, lam)
    torch.cuda.synchronize()
    new, C, worst = [to_host64(f) for f in Fd], F[2].astype(np.float64), 0.0
    seen = [torch.from_numpy(f).to(DEV) for f in F]
    for m, own, oth in ((0, yi, yj), (1, yj, yi)):
        O = to_host64(seen[1 - m])
        P = mu * ((O.T @ O) * (C.T @ C)) + lam * np.eye(R)
        M = to_host64(dfacto.mttkrp(ctx, X, m, seen))
        for r in range(len(new[m])):
            e = np.flatnonzero(own == r)
            V = O[oth[e]]
            z0, U = np.linalg.solve(P, mu * M[r]), np.linalg.solve(P, V.T).T
            Kr = np.eye(len(e)) + V @ U.T
            d = U.T @ np.linalg.solve(Kr, yv[e] - V @ z0) if len(e) else np.zeros(R)
            x = z0 + d
            # stored in FP32; P^-1, K and their products in FP64
            cond = np.linalg.cond(P) * (np.linalg.cond(Kr) if len(e) else 1.0)
            tol = 1.01 * 2.0 ** -24 * np.linalg.norm(x) + \
                64 * R * EPS * cond * (np.linalg.norm(z0) + np.linalg.norm(d))
            err = np.linalg.norm(new[m][r] - x)
            assert err <= tol, (m, r, len(e), err, tol)
            worst = max(worst, err / max(tol, 1e-300))
        seen[m] = Fd[m]
    say(f"  joint short rows R={R} mu={mu}: worst error / bound {worst:.3f}")
    X.close()
    Y.close()
