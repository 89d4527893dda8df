"""The builder's passes at the sizes where they change, against numpy: exact
structure, and every value the FP32 sum of its duplicates in input order.

Sorts of one tile, of few tiles and of many (4096 pairs each; 256 tiles and
more take other offsets); indices that fit one 64-bit key and ones that do
not; dimensions of 1 (no digits to sort); duplicate runs around the length
that a wave takes over (16), beyond its batch (1024) and across tiles (2048
entries); fibers longer than a tile and around the 128-nonzero segments; rows
split over short and long runs of chunks.
"""
import numpy as np
import pytest
import torch

from gpu_util import say, DEV
from paper_1406_4519_amd import dfacto

pytestmark = pytest.mark.gpu

ROLES = ((0, 2, 1), (1, 0, 2), (2, 1, 0))  # (root, mid, leaf) axis of each mode


def reference(idx, val, mode):
    r, m, l = (idx[a].astype(np.int64) for a in ROLES[mode])
    o = np.lexsort((l, m, r))  # stable: input order among equal coordinates
    r, m, l, v = r[o], m[o], l[o], val[o]
    new = np.ones(len(r), bool)
    new[1:] = (r[1:] != r[:-1]) | (m[1:] != m[:-1]) | (l[1:] != l[:-1])
    at = np.flatnonzero(new)
    end = np.append(at[1:], len(r))
    # np.add.accumulate adds one element after the other in FP32
    s = np.array([v[a] if b == a + 1 else np.add.accumulate(v[a:b])[-1] for a, b in zip(at, end)],
                 np.float32)
    r, m, l = r[at], m[at], l[at]
    fib = np.ones(len(r), bool)
    fib[1:] = (r[1:] != r[:-1]) | (m[1:] != m[:-1])
    fa = np.flatnonzero(fib)
    root = np.ones(len(fa), bool)
    root[1:] = r[fa][1:] != r[fa][:-1]
    ra = np.flatnonzero(root)
    return dict(root_id=r[fa][ra], root_ptr=np.append(ra, len(fa)), fib_mid=m[fa],
                fib_ptr=np.append(fa, len(r)), leaf=l, val=s)


def _uniform(rng, dims, n):
    return [rng.integers(0, d, n).astype(np.uint32) for d in dims]


def _runs(rng):
    """coordinates drawn 1 to 5000 times each, in mixed order"""
    reps = [1, 2, 3, 15, 16, 17, 18, 63, 64, 65, 66, 1023, 1024, 1025, 2047, 2048, 2049, 5000] + [1] * 3000
    base = _uniform(rng, (900, 800, 700), len(reps))
    o = rng.permutation(np.repeat(np.arange(len(reps)), reps))
    return [b[o] for b in base]


def _fibers(rng):
    """fibers of 1 to 9000 nonzeros, one row over many chunks"""
    ii, jj, kk = [], [], []
    for q, n in enumerate((9000, 1, 127, 128, 129, 256, 257, 2047, 2048, 2049, 4096, 3)):
        ii += [q // 2] * n
        kk += [q] * n
        jj += list(rng.choice(10_000, n, replace=False))
    for k in range(60):
        n = int(rng.integers(1, 400))
        ii += [40] * n
        kk += [k] * n
        jj += list(rng.choice(10_000, n, replace=False))
    o = rng.permutation(len(ii))
    return [np.asarray(a, np.uint32)[o] for a in (ii, jj, kk)]


CASES = {
    "one": ((5, 4, 3), lambda r: [np.array([x], np.uint32) for x in (4, 0, 2)]),
    "tile": ((300, 200, 100), lambda r: _uniform(r, (300, 200, 100), 4096)),
    "tile+1": ((300, 200, 100), lambda r: _uniform(r, (300, 200, 100), 4097)),
    "flat": ((1, 5000, 1), lambda r: _uniform(r, (1, 5000, 1), 20_000)),
    "column": ((1, 1, 3000), lambda r: _uniform(r, (1, 1, 3000), 5_000)),
    "many tiles": ((5000, 300, 4000), lambda r: _uniform(r, (5000, 300, 4000), 257 * 4096)),
    "runs": ((900, 800, 700), _runs),
    "fibers": ((64, 10_000, 64), _fibers),
    "64 bits": ((1 << 30, 1 << 17, 1 << 17), lambda r: _uniform(r, (1 << 30, 1 << 17, 1 << 17), 30_000)),
    "65 bits": ((1 << 30, 1 << 18, 1 << 17), lambda r: _uniform(r, (1 << 30, 1 << 18, 1 << 17), 30_000)),
    "wide runs": ((1 << 28, 1 << 28, 1 << 28),
                  lambda r: [x * np.uint32(290_000) for x in _runs(r)]),
}


@pytest.mark.parametrize("relabel", [False, True])
@pytest.mark.parametrize("case", list(CASES))
def test_build(case, relabel):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dims, draw = CASES[case]
    if relabel and max(dims) > 1 << 20:
        pytest.skip("the rank tables of 2^28 rows are not the point here")
    rng = np.random.default_rng(len(case))
    idx = draw(rng)
    val = rng.standard_normal(len(idx[0])).astype(np.float32)
    say(f"  {case} relabel={relabel} n={len(val)}")
    ctx = dfacto.Context(0)
    t = dfacto.build_flattenings(ctx, dims, *[torch.from_numpy(x.view(np.int32)).to(DEV) for x in idx],
                                 torch.from_numpy(val).to(DEV), relabel=relabel)
    inf = t.info()
    for mode in range(3):
        ref, got = reference(idx, val, mode), dfacto.tensor_export(ctx, t, mode)
        assert inf["nnz"] == len(ref["leaf"]) and inf["nfib"][mode] == len(ref["fib_mid"])
        for key, want in ref.items():
            np.testing.assert_array_equal(got[key], want, err_msg=f"mode {mode} {key}")
    exact = float(np.sum(ref["val"].astype(np.float64) ** 2))
    assert abs(inf["normsq"] - exact) <= 1e-12 * exact
    t.close()
    ctx.close()
