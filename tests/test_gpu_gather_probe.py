"""The gather probe loads what it says: pattern 0 the row of every stream entry
and no other, pattern 7 leaf rows by buffer loads, 3 nothing; the others, whose
rows are drawn, means of the tables.  Ranks over one to two columns per lane,
whole waves, odd ones, and rows padded by a relabeled mode."""
import numpy as np
import pytest
import torch

from gpu_util import build, factors_to_dev, DEV
from paper_1406_4519_amd import dfacto, gen

pytestmark = pytest.mark.gpu

DIMS = (900, 700, 500)


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = dfacto.Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


@pytest.mark.parametrize("R,dtype,relabel", [(8, "f32", False), (16, "f32", False), (32, "f32", False),
                                             (32, "bf16", False), (64, "f32", False), (128, "f32", False),
                                             (256, "f32", False), (10, "f32", True), (10, "bf16", True),
                                             (32, "bf16", True), (64, "bf16", True)])
def test_probe_sums(ctx, R, dtype, relabel):
    coo = gen.zipf_distinct(DIMS, 60_000, 0.4, seed=61)
    t = build(ctx, coo, relabel=relabel)
    rng = np.random.default_rng(62)
    Fd, F = factors_to_dev([rng.uniform(0.5, 1.5, (d, R)) for d in DIMS], dtype)
    info = t.info()
    for m in range(3):
        e = dfacto.tensor_export(ctx, t, m)
        leaf, mid = F[(m + 1) % 3], F[(m + 2) % 3]
        headers = info["nentry"][m] - info["nnz"]
        assert headers == len(e["fib_mid"])  # no fiber is split: a header each
        own = leaf[e["leaf"]].sum() + mid[e["fib_mid"]].sum()
        # FP32 sums of at most 640 positive terms per lane, added up in FP64
        tol = 700 * 2.0 ** -24
        for pat in range(10):
            if pat in (5, 8, 9) and R > 64:
                continue
            sink = torch.zeros(64 * info["nchunk"][m], device=DEV)
            dfacto.gather_probe(ctx, t, m, Fd, pat, sink)
            torch.cuda.synchronize()
            s = sink.double().sum().item()
            if pat == 0:
                assert abs(s - own) <= tol * own, (m, s, own)
            elif pat in (3, 6):
                assert np.isfinite(s)
            elif pat == 7 and not relabel:  # (a relabeled header's index is a rank)
                ref = own - mid[e["fib_mid"]].sum() + leaf[e["fib_mid"] % DIMS[(m + 1) % 3]].sum()
                # the first header of a chunk opens it without a gather
                slack = info["nchunk"][m] * R * 1.5
                assert ref - slack - tol * ref <= s <= ref + tol * ref, (m, s, ref)
            else:
                n = info["nentry"][m] * R
                assert 0.4 * n <= s <= 1.6 * n, (m, pat, s / n)
    t.close()
