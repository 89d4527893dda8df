"""The row solves of the joint ALS at the sizes where they can go wrong:
row lengths around the batches of 4, 16 and 32 entries and around the split
into segments, numbers of rows that are no multiple of 4, ranks around the
4-column blocks and the two block counts, rows that start off their
alignment, and systems close to singular.  mu = 0 leaves the ratings alone,
so each row is a ridge least squares of its ratings, solved here in float64
from the factor the device used."""
import numpy as np
import pytest
import torch

from gpu_util import build, say, to_host64, DEV
from paper_1406_4519_amd import dfacto, gen

pytestmark = pytest.mark.gpu

I, J = 151, 2203
LENGTHS = [0, 1, 2, 3, 4, 5, 7, 8, 15, 16, 17, 31, 32, 33, 63, 64, 65, 126, 127, 128, 129, 130, 253, 254, 255, 256,
           257, 1100, 2030, 2033, 2100, 2203]


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = dfacto.Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


def _ratings(ctx, lengths, seed):
    rng = np.random.default_rng(seed)
    yi = np.concatenate([np.full(n, r) for r, n in enumerate(lengths)])
    yj = np.concatenate([rng.choice(J, n, replace=False) for n in lengths])
    yv = rng.integers(1, 6, len(yi)).astype(np.float32)
    dv = [torch.from_numpy(a.astype(np.int32)).to(DEV) for a in (yi, yj)]
    return (yi, yj, yv.astype(np.float64)), dfacto.build_ratings(ctx, (I, J), dv[0], dv[1],
                                                                 torch.from_numpy(yv).to(DEV))


@pytest.fixture(scope="module")
def problem(ctx):
    rng = np.random.default_rng(71)
    lengths = LENGTHS + list(rng.integers(0, 40, I - len(LENGTHS) - 3)) + [0, 0, 9]
    X = build(ctx, gen.zipf_distinct((I, J, 20), 500, 0.5, seed=72))
    y, Y = _ratings(ctx, lengths, 73)
    return X, y, Y


def _factors(R, dtype, off, seed):
    """Factors that start `off` elements into their allocation."""
    t = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator().manual_seed(seed)
    out = []
    for d in (I, J, 20):
        buf = torch.zeros(d * R + off, dtype=t, device=DEV)
        buf[off:].copy_(torch.rand(d * R, generator=g))
        out.append(buf[off:].view(d, R))
    return out


@pytest.mark.parametrize("R,dtype,off", [(1, "f32", 0), (3, "bf16", 0), (4, "f32", 0), (5, "f32", 0), (8, "bf16", 0),
                                         (15, "f32", 0), (16, "f32", 0), (16, "bf16", 0), (16, "bf16", 1),
                                         (17, "f32", 0), (20, "bf16", 0), (28, "f32", 0), (31, "bf16", 0),
                                         (32, "f32", 0), (32, "f32", 1), (32, "bf16", 0)])
def test_rows_are_ridge_least_squares(ctx, problem, R, dtype, off):
    X, (yi, yj, yv), Y = problem
    lam = 0.1
    F = _factors(R, dtype, off, 74 + R)
    B0 = to_host64(F[1])
    dfacto.joint_als_iter(ctx, X, Y, F, 0.0, lam)
    torch.cuda.synchronize()
    A, B = to_host64(F[0]), to_host64(F[1])
    # stored to half a unit in the last place of each element (24 and 8
    # significant bits); the solve itself is backward stable in float64
    unit = 2.0 ** -24 if dtype == "f32" else 2.0 ** -8
    worst = 0.0
    for new, other, own, oth in ((A, B0, yi, yj), (B, A, yj, yi)):
        order = np.argsort(own, kind="stable")
        start = np.searchsorted(own[order], np.arange(new.shape[0] + 1))
        for r in range(new.shape[0]):
            e = order[start[r]:start[r + 1]]
            V = other[oth[e]]
            S = V.T @ V + lam * np.eye(R)
            x = np.linalg.solve(S, V.T @ yv[e])
            tol = 1.01 * unit + 64 * R * 2.0 ** -53 * np.linalg.cond(S)
            err = np.linalg.norm(new[r] - x) / max(np.linalg.norm(x), 1e-30) if len(e) else np.abs(new[r]).max()
            assert err <= tol, (r, len(e), err, tol)
            worst = max(worst, err / tol)
    say(f"  joint rows R={R} {dtype}: worst error / bound {worst:.3f}")


@pytest.mark.parametrize("R", [6, 16, 32])
def test_short_rows_near_singular_are_solved(ctx, problem, R):
    """A lam below the pivot test: rows of at most 7 ratings are solved from
    P^-1 = I / lam all the same; a longer row with fewer ratings than R is a
    failure that names itself."""
    X, _, _ = problem
    lengths = [0, 1, 2, 3, 4, 5, 5] + [0] * (I - 7)
    (yi, yj, yv), Y = _ratings(ctx, lengths, 75)
    F = _factors(R, "f32", 0, 76)
    dfacto.joint_als_iter(ctx, X, Y, F, 0.0, 1e-17)
    torch.cuda.synchronize()
    assert all(np.isfinite(to_host64(f)).all() for f in F)
    Y.close()
    if R > 8:
        _, Y = _ratings(ctx, [8] + [0] * (I - 1), 77)
        with pytest.raises(dfacto.DfactoError) as e:
            dfacto.joint_als_iter(ctx, X, Y, _factors(R, "f32", 0, 78), 0.0, 1e-17)
        assert e.value.status == dfacto.E_NUMERIC
        Y.close()
