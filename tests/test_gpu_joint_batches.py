"""Rows of more ratings than one wave takes are solved in batches of segments,
so that the workspace of a joint ALS iteration does not grow with the number of
such rows: 20,000 users of 260 ratings (a segment each, three batches) and
2,000 items of 2,600 (three segments each)."""
import numpy as np
import pytest
import torch

from gpu_util import build, to_host64, DEV
from paper_1406_4519_amd import dfacto, gen

pytestmark = pytest.mark.gpu

I, J, PER = 20_000, 2_000, 260


@pytest.mark.parametrize("R,dtype", [(4, "f32"), (17, "f32"), (32, "bf16")])
def test_rows_in_batches(R, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ctx = dfacto.Context(0, allocator="torch")
    row = np.repeat(np.arange(I, dtype=np.int64), PER)
    col = (row * 13 + np.tile(np.arange(PER), I) * 7) % J  # distinct within a row: 7 and 2000 are coprime
    val = (1 + (row * 31 + col * 17) % 5).astype(np.float32)
    Y = dfacto.build_ratings(ctx, (I, J), torch.from_numpy(row.astype(np.int32)).to(DEV),
                             torch.from_numpy(col.astype(np.int32)).to(DEV), torch.from_numpy(val).to(DEV))
    X = build(ctx, gen.uniform_distinct((I, J, 20), 1000, seed=41))
    g = torch.Generator().manual_seed(42)
    t = torch.float32 if dtype == "f32" else torch.bfloat16
    F = [torch.rand((d, R), generator=g).to(t).to(DEV) for d in (I, J, 20)]
    B0, lam = to_host64(F[1]), 0.1
    torch.cuda.synchronize()
    before = torch.cuda.memory_allocated()
    dfacto.joint_als_iter(ctx, X, Y, F, 0.0, lam)
    torch.cuda.synchronize()
    added = torch.cuda.memory_allocated() - before
    # 8192 partial systems of 14 or 44 blocks of 16 doubles; the rows' FP32
    # products; R x R matrices and their partial sums; an eighth of slack
    most = 8192 * 16 * 8 * (14 if R <= 16 else 44) + 4 * R * I + 8 * (2 * 256 + 64) * R * R + (1 << 20)
    assert added <= 1.125 * most, (added, most)
    A, B = to_host64(F[0]), to_host64(F[1])
    unit = 2.0 ** -24 if dtype == "f32" else 2.0 ** -8
    users = [0, 1, 2, 3, 8190, 8191, 8192, 8193, 16382, 16383, 16384, 16385, I - 2, I - 1]
    for new, other, own, oth, rows in ((A, B0, row, col, users), (B, A, col, row, [0, 1, 999, 1000, J - 2, J - 1])):
        for r in rows:
            e = np.flatnonzero(own == r)
            V = other[oth[e]]
            S = V.T @ V + lam * np.eye(R)
            x = np.linalg.solve(S, V.T @ val[e].astype(np.float64))
            # stored to half a unit in the last place; the solve is backward stable in FP64
            tol = 1.01 * unit + 64 * R * 2.0 ** -53 * np.linalg.cond(S)
            assert np.linalg.norm(new[r] - x) <= tol * np.linalg.norm(x), (r, len(e))
    for x in (X, Y):
        x.close()
    torch.cuda.synchronize()
    ctx.close()
