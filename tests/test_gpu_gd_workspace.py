"""What a GD step adds to a context's device memory: the trial factors and one
dims[0] x R FP32 buffer (or one Gram's partial sums where those are larger), not
a fixed amount that small tensors would pay too."""
import pytest
import torch

from gpu_util import build, factors_to_dev, DEV
from paper_1406_4519_amd import dfacto, gen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,R", [((300, 200, 100), 64), ((100, 300, 200), 64), ((40, 30, 20), 32), ((70, 90, 80), 8),
                                    ((90, 80, 70), 100), ((40_000, 300, 70_000), 48)])
def test_gd_step_workspace_follows_the_sizes(dims, R):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ctx = dfacto.Context(0, allocator="torch")
    t = build(ctx, gen.zipf_distinct(dims, 3000, 0.5, seed=31))
    F, _ = factors_to_dev(gen.init_factors(dims, R, seed=32))
    G = [torch.empty((d, R), device=DEV) for d in dims]
    f = torch.zeros(1, dtype=torch.float64, device=DEV)
    dfacto.gd_grad(ctx, t, F, G, f)
    torch.cuda.synchronize()
    before = torch.cuda.memory_allocated()
    first = dfacto.gd_step(ctx, t, F, G, max_trials=80)
    torch.cuda.synchronize()
    added = torch.cuda.memory_allocated() - before
    factors = 4 * R * sum(dims)
    least = 8 * R * R * max(1, min(dims) // 128 + 1)
    # workspaces are allocated an eighth larger than asked for, each part on 256 bytes
    assert added <= 1.125 * (factors + max(4 * R * dims[0], least) + 4 * 256) + 512, added
    # the Grams' partial sums there change nothing: f at the accepted point is f0 of the next gradient
    assert first["accepted"]
    dfacto.gd_grad(ctx, t, F, G, f)
    torch.cuda.synchronize()
    assert abs(f.item() - first["f"]) <= 1e-12 * abs(first["f0"])
    t.close()
    torch.cuda.synchronize()
    ctx.close()
