"""The MTTKRP's two kernels against each other, bitwise.

A tensor with few work chunks is computed by one block per chunk, one with
many by lane groups.  The large tensor here is the small one plus nonzeros
whose indices lie beyond it in every mode: the small one's rows come first in
each stream and are cut into the same chunks, so both kernels form the same
sums in the same order and the shared rows must agree to the last bit (the
parity tests compare the small tensors' results with the oracle).
"""
import numpy as np
import pytest
import torch

from gpu_util import build, factors_to_dev, say, DEV
from paper_1406_4519_amd import dfacto, gen

pytestmark = pytest.mark.gpu


def _small():
    """Fibers of 1 to 300 nonzeros (a segment holds 128, a mask word 64),
    one row of many fibers over several chunks, rows of one nonzero, empty
    rows at the start, in between and at the end."""
    rng = np.random.default_rng(77)
    I, J, K = 90, 400, 120
    ii, jj, kk = [], [], []

    def fiber(i, k, n):
        ii.extend([i] * n)
        kk.extend([k] * n)
        jj.extend(rng.choice(J, n, replace=False))

    for q, n in enumerate((1, 2, 62, 63, 64, 65, 126, 127, 128, 129, 130, 192, 256, 257, 300)):
        fiber(2 + q, 3 * q, n)
    for k in range(110):  # a row over several chunks
        fiber(30, k, int(rng.integers(1, 40)))
    for i in range(40, 80):
        fiber(i, int(rng.integers(K)), 1)
    for k in range(0, 120, 2):  # the last row: single-nonzero fibers
        fiber(87, k, 1)
    u = lambda a: np.asarray(a, np.uint32)
    return gen.Coo((I, J, K), u(ii), u(jj), u(kk),
                   rng.standard_normal(len(ii)).astype(np.float32))


@pytest.fixture(scope="module")
def pair():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ctx = dfacto.Context(0)
    a = _small()
    n, I, J, K = 2_000_000, *a.dims
    rng = np.random.default_rng(78)
    ext = [rng.integers(0, 1000, n).astype(np.uint32) for _ in range(3)]
    b = gen.Coo((I + 1000, J + 1000, K + 1000), np.concatenate([a.i, ext[0] + np.uint32(I)]),
                np.concatenate([a.j, ext[1] + np.uint32(J)]),
                np.concatenate([a.k, ext[2] + np.uint32(K)]),
                np.concatenate([a.val, rng.standard_normal(n).astype(np.float32)]))
    ta, tb = build(ctx, a), build(ctx, b)
    say(f"  chunks {ta.info()['nchunk']} and {tb.info()['nchunk']}")
    assert max(ta.info()["nchunk"]) * 16 < 4096 and min(tb.info()["nchunk"]) > 5120
    yield ctx, a, b, ta, tb
    torch.cuda.synchronize()
    ta.close()
    tb.close()
    ctx.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("R", [1, 2, 4, 7, 8, 9, 10, 12, 16, 17, 24, 31, 32, 33, 48, 64, 100, 130, 255, 256])
def test_kernels_agree(pair, R, dtype):
    ctx, a, b, ta, tb = pair
    rng = np.random.default_rng(R)
    Fb, _ = factors_to_dev([rng.standard_normal((d, R)) for d in b.dims], dtype)
    Fa = [f[:d].contiguous() for f, d in zip(Fb, a.dims)]
    for m in range(3):
        say(f"  mode {m} R={R} {dtype}")
        x = dfacto.mttkrp(ctx, ta, m, Fa, torch.full((a.dims[m], R), float("nan"), device=DEV))
        y = dfacto.mttkrp(ctx, tb, m, Fb, torch.full((b.dims[m], R), float("nan"), device=DEV))
        assert torch.equal(x, y[:a.dims[m]]), f"mode {m}"


def test_kernels_agree_nonfinite(pair):
    """Inf and NaN factor entries reach the same outputs from both kernels."""
    ctx, a, b, ta, tb = pair
    R = 10
    rng = np.random.default_rng(5)
    F = [rng.standard_normal((d, R)) for d in b.dims]
    for m, d in enumerate(a.dims):
        F[m][d // 3, 2], F[m][d // 2, 5], F[m][d // 4, 7] = np.inf, -np.inf, np.nan
    Fb, _ = factors_to_dev(F, "f32")
    Fa = [f[:d].contiguous() for f, d in zip(Fb, a.dims)]
    for m in range(3):
        x = dfacto.mttkrp(ctx, ta, m, Fa)
        y = dfacto.mttkrp(ctx, tb, m, Fb)[:a.dims[m]]
        assert torch.equal(torch.isnan(x), torch.isnan(y)) and not torch.isfinite(x).all()
        assert torch.equal(torch.nan_to_num(x), torch.nan_to_num(y))
