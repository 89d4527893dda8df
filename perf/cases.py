"""The work that programs have this library do, as cases that can be timed.

A case is a dict of plain values.  `op` says which entry points a pass calls:

  mttkrp   the three MTTKRPs of a built tensor (a solver of the caller's own)
  als      the start of a CP-ALS solve: the factors set to their starting
           values, then `iters` iterations
  gd       one GD gradient with the objective (an optimizer of the caller's)
  gdstep   the start of a GD solve: `iters` iterations with the line search,
           the first trial step 1, then twice the step taken
  group    the start of many CP-ALS solves at once, as one group whose
           iteration is replayed as a graph
  build    a tensor built from COO arrays and its three first MTTKRPs
  joint    one ALS iteration of the joint ratings and tensor model

Coordinates follow a Zipf law per mode over a seeded permutation (s = 0:
uniform), values are |N(0,1)|, factors U(0,1), as in the repository's own
benchmark and tests.  Sizes are those of its workloads, or spread between
them.
"""
import math
import random

import torch

from paper_1406_4519_amd import dfacto, gen

DEV = "cuda:0"
LEAF = (1, 2, 0)  # mode n gathers factor LEAF[n] per nonzero and MID[n] per fiber
MID = (2, 0, 1)


def listed():
    return [
        # the smallest calls: a parity-sized tensor, where launches and latency count
        dict(name="mttkrp-20k-r8", op="mttkrp", I=200, J=150, K=100, nnz=20_000, s=0.0, R=8, dtype="f32"),
        # a tenth of the paper's 1.2 billion nonzeros in each size, BF16 storage
        # (few rows, each gathered often: the library relabels it)
        dict(name="mttkrp-100m-r32-bf16", op="mttkrp", I=650_000, J=250_000, K=150_000, nnz=100_000_000,
             s=1.2, R=32, dtype="bf16"),
        # solves: the small configuration, the paper's synthetic sweeps
        # (1e6 nonzeros, R = 10), the 50M-nonzero review-like tensor, and a
        # high rank with ridge and BF16 storage
        dict(name="als-20k-r8", op="als", I=200, J=150, K=100, nnz=20_000, s=0.0, R=8, dtype="f32", reg=0.0, iters=5),
        dict(name="als-1m-r10", op="als", I=100_000, J=100_000, K=100_000, nnz=1_000_000, s=0.6, R=10, dtype="f32",
             reg=0.0, iters=3),
        dict(name="als-50m-r32", op="als", I=1_000_000, J=500_000, K=200_000, nnz=50_000_000, s=1.1, R=32,
             dtype="f32", reg=0.0, iters=1),
        dict(name="als-4m-r100-bf16", op="als", I=120_011, J=61_001, K=23_003, nnz=4_000_000, s=1.1, R=100,
             dtype="bf16", reg=0.1, iters=1),
        # gradients: the tenth of the paper's shape at the rank of its runs, and a
        # whole gradient descent with its line search on a sweep's tensor
        dict(name="gd-100m-r10", op="gd", I=650_000, J=250_000, K=150_000, nnz=100_000_000, s=1.2, R=10,
             dtype="f32", reg=0.0),
        dict(name="gdstep-1m-r10", op="gdstep", I=100_000, J=100_000, K=100_000, nnz=1_000_000, s=0.6, R=10,
             dtype="f32", reg=0.0, iters=3),
        # many solves at once: 32 tensors of 1e3 to 1e5 rows per mode, 1e4 to
        # 5e6 nonzeros, ranks 8, 16 and 32
        dict(name="group-32", op="group", members=32, most=5_000_000, dtype="f32", iters=2),
        # new tensors: one of a served burst, and the review-like one (raw
        # draws in no order: some coordinates twice), each with its first products
        dict(name="build-1m-r16", op="build", I=70_000, J=30_000, K=9_000, nnz=1_000_000, s=1.1, R=16, dtype="f32",
             memory="library"),
        dict(name="build-50m-r32", op="build", I=1_000_000, J=500_000, K=200_000, nnz=50_000_000, s=1.1, R=32,
             dtype="f32", memory="torch"),
        # ratings and a tensor together: users and items of a review site
        dict(name="joint-10m-r32", op="joint", I=400_000, J=200_000, K=80_000, nnz=10_000_000, ratings=4_000_000,
             s=1.1, R=32, dtype="f32", mu=1.0, lam=0.1),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    op = rng.choice(("mttkrp", "mttkrp", "als", "als", "gd", "gdstep", "group", "build", "joint"))
    dtype = rng.choice(("f32", "f32", "bf16"))
    if op == "group":
        return dict(op=op, members=rng.randint(4, 32), most=_log_uniform(rng, 100_000, 4_000_000), dtype=dtype,
                    iters=rng.randint(1, 2))
    most = dict(mttkrp=60e6, als=30e6, gd=60e6, gdstep=1e6, build=40e6, joint=8e6)[op]
    nnz = _log_uniform(rng, 20_000, most)
    R = rng.choice((4, 8, 10, 12, 16, 20, 24, 31, 32, 48, 64, 100))
    if op == "joint":
        R = min(R, 32)
    if nnz > 4_000_000:  # no more than the listed ones cost
        R = min(R, 32)
    if op == "gdstep":
        R = min(R, 16)
    # rows per mode from a few nonzeros per row to a thousand
    lo, hi = max(100, nnz // 1000), min(1_000_000, max(200, nnz // 3))
    c = dict(op=op, I=_log_uniform(rng, lo, hi), J=_log_uniform(rng, lo, hi), K=_log_uniform(rng, lo, hi), nnz=nnz,
             s=rng.choice((0.0, 0.6, 1.1, 1.2)), R=R, dtype=dtype)
    cells = c["I"] * c["J"] * c["K"]
    c["nnz"] = min(nnz, cells // 20)
    if c["s"] > 0.6:  # distinct coordinates of a steep law run out sooner
        c["nnz"] = min(c["nnz"], cells // 20_000 + 20_000)
    if op in ("als", "gd", "gdstep"):
        c["reg"] = rng.choice((0.0, 0.1))
    if op in ("als", "gdstep"):
        c["iters"] = 1 if nnz > 1_000_000 else rng.randint(1, 3)
    if op == "build":
        c["memory"] = rng.choice(("library", "torch"))
    if op == "joint":
        c["ratings"] = max(1000, min(c["nnz"] // 3, c["I"] * c["J"] // 50))
        c.update(mu=rng.choice((0.5, 1.0)), lam=0.1)
    return c


# ---- inputs ---------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _raw(dims, n, s, g):
    """n draws in no order; a coordinate may come more than once."""
    idx = []
    for d in dims:
        cdf = torch.from_numpy(gen.zipf_cdf(d, s)).to(DEV)
        perm = torch.randperm(d, generator=g, device=DEV)
        u = torch.rand(n, generator=g, device=DEV, dtype=torch.float64)
        idx.append(perm[torch.searchsorted(cdf, u, right=True).clamp_(max=d - 1)].to(torch.int32))
    val = torch.randn(n, generator=g, device=DEV).abs_()
    return idx + [val]


def _coo(dims, nnz, s, seed, raw=False):
    if raw:
        return _raw(dims, nnz, s, _gen(seed))
    batch = max(1 << 16, min(1 << 27, 2 * nnz))
    return list(gen.zipf_distinct_torch(dims, nnz, s, seed, device=DEV, batch=batch))


def _dims(case):
    return (case["I"], case["J"], case["K"])


def _factors(dims, R, dtype, g):
    t = torch.float32 if dtype == "f32" else torch.bfloat16
    return [torch.rand((d, R), generator=g, device=DEV).to(t) for d in dims]


def _members(case):
    """(dims, nnz, s, R) of a group's members, as different in size as the
    solves that come together in a batch."""
    rng = random.Random(case["most"] * 1000 + case["members"])
    out = []
    for _ in range(case["members"]):
        dims = tuple(_log_uniform(rng, 1_000, 100_000) for _ in range(3))
        nnz = _log_uniform(rng, 10_000, case["most"])
        cells = dims[0] * dims[1] * dims[2]
        out.append((dims, min(nnz, cells // 20_000 + 10_000), 1.1, rng.choice((8, 16, 32))))
    # the whole group's nonzeros are bounded by `most`
    total, want = sum(m[1] for m in out), case["members"] * case["most"] / 6.5
    f = min(1.0, want / total)
    return [(d, max(1_000, int(n * f)), s, R) for d, n, s, R in out]


def _group_inputs(case, seed):
    t = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    mem = _members(case)
    coos = [_coo(d, n, s, seed * 64 + q) for q, (d, n, s, _) in enumerate(mem)]
    # one buffer for every member's factors (each on a 16-byte boundary)
    sizes = [(d * R + 7) // 8 * 8 for dims, _, _, R in mem for d in dims]
    flat = torch.rand(sum(sizes), generator=_gen(seed), device=DEV).to(t)
    return mem, coos, flat, sizes


def _views(mem, flat, sizes):
    at, out, q = 0, [], 0
    for dims, _, _, R in mem:
        F = []
        for d in dims:
            F.append(flat[at:at + d * R].view(d, R))
            at += sizes[q]
            q += 1
        out.append(F)
    return out


def prepare(case, seed):
    op = case["op"]
    if op == "group":
        ctx = dfacto.Context(0)
        mem, coos, start, sizes = _group_inputs(case, seed)
        tensors = [dfacto.build_flattenings(ctx, m[0], *c) for m, c in zip(mem, coos)]
        flat = start.clone()
        lam = torch.zeros(sum(m[3] for m in mem), dtype=torch.float64, device=DEV)
        lams = list(torch.split(lam, [m[3] for m in mem]))
        fits = torch.zeros(len(mem), dtype=torch.float64, device=DEV)
        g = dfacto.Group(ctx, tensors, _views(mem, flat, sizes), lams, fits, graph=True)
        return dict(case=case, ctx=ctx, tensors=tensors, start=start, flat=flat, lam=lam, fits=fits, group=g)
    dims, R, g = _dims(case), case["R"], _gen(seed + 7)
    st = dict(case=case, dims=dims)
    st["start"] = _factors(dims, R, case["dtype"], g)
    st["F"] = [f.clone() for f in st["start"]]
    if op == "build":
        st["ctx"] = dfacto.Context(0, allocator="torch" if case["memory"] == "torch" else None)
        st["coo"] = _coo(dims, case["nnz"], case["s"], seed, raw=True)
    else:
        st["ctx"] = dfacto.Context(0)
        st["T"] = dfacto.build_flattenings(st["ctx"], dims, *_coo(dims, case["nnz"], case["s"], seed))
    if op in ("mttkrp", "build"):
        st["M"] = [torch.empty((d, R), device=DEV) for d in dims]
    if op == "als":
        st["lam"] = torch.zeros(R, dtype=torch.float64, device=DEV)
        st["fit"] = torch.zeros(1, dtype=torch.float64, device=DEV)
    if op in ("gd", "gdstep"):
        st["G"] = [torch.empty((d, R), device=DEV) for d in dims]
        st["f"] = torch.zeros(1, dtype=torch.float64, device=DEV)
    if op == "joint":
        i, j, _, y = _coo((dims[0], dims[1], 1), case["ratings"], case["s"], seed + 3)
        st["Y"] = dfacto.build_ratings(st["ctx"], dims[:2], i, j, y)
    return st


# ---- one pass -------------------------------------------------------------

def run(st):
    case, ctx = st["case"], st["ctx"]
    op = case["op"]
    if op == "group":
        st["flat"].copy_(st["start"])
        st["group"].als(case["iters"])
        return dict(factors=st["flat"], lam=st["lam"], fit=st["fits"])
    if op == "mttkrp":
        return [dfacto.mttkrp(ctx, st["T"], m, st["F"], st["M"][m]) for m in range(3)]
    if op == "build":
        T = dfacto.build_flattenings(ctx, st["dims"], *st["coo"])
        M = [dfacto.mttkrp(ctx, T, m, st["F"], st["M"][m]) for m in range(3)]
        inf = T.info()
        T.close()
        return dict(M=M, nnz=inf["nnz"], nfib=list(inf["nfib"]), nroot=list(inf["nroot"]),
                    nentry=list(inf["nentry"]), normsq=inf["normsq"])
    if op == "gd":
        dfacto.gd_grad(ctx, st["T"], st["F"], st["G"], st["f"], reg=case["reg"])
        return dict(G=st["G"], f=st["f"])
    for x, x0 in zip(st["F"], st["start"]):
        x.copy_(x0)
    if op == "als":
        for _ in range(case["iters"]):
            dfacto.als_iter(ctx, st["T"], st["F"], st["lam"], st["fit"], reg=case["reg"])
        return dict(F=st["F"], lam=st["lam"], fit=st["fit"])
    if op == "joint":
        dfacto.joint_als_iter(ctx, st["T"], st["Y"], st["F"], case["mu"], case["lam"])
        return st["F"]
    alpha, steps = 1.0, []
    for _ in range(case["iters"]):
        r = dfacto.gd_step(ctx, st["T"], st["F"], st["G"], reg=case["reg"], alpha0=alpha, max_trials=60)
        alpha = 2.0 * r["alpha"] if r["accepted"] else alpha
        steps.append([r["f0"], r["f"], r["gnorm2"], r["trials"]])
    return dict(F=st["F"], G=st["G"], steps=steps)


# ---- what a pass cannot do without ----------------------------------------

def _mttkrp_work(dims, nnz, R, es):
    """Three MTTKRPs: per mode each nonzero's index and value once, the two
    gathered factors once, the output once; a multiply and an add per nonzero
    and column, and another per nonzero's fiber at the most compressed (none
    counted)."""
    b = sum(8 * nnz + es * R * (dims[LEAF[m]] + dims[MID[m]]) + 4 * R * dims[m] for m in range(3))
    return b, 3 * 2.0 * R * nnz


def work(case):
    op, es = case["op"], 4 if case["dtype"] == "f32" else 2
    if op == "group":
        b = f = 0
        for dims, nnz, _, R in _members(case):
            x, y = _mttkrp_work(dims, nnz, R, es)
            b += x + es * R * sum(dims)
            f += y + 4.0 * R * R * sum(dims)
        return dict(bytes=case["iters"] * b, flops=case["iters"] * f)
    dims, nnz, R = _dims(case), case["nnz"], case["R"]
    rows = sum(dims)
    b, f = _mttkrp_work(dims, nnz, R, es)
    if op == "mttkrp":
        return dict(bytes=b, flops=f)
    if op == "build":  # the COO read once, three flattenings written once
        return dict(bytes=b + 16 * nnz + 3 * 8 * nnz, flops=f + 2.0 * nnz)
    if op == "als":  # the products, each new factor's rows written, Gram and update
        return dict(bytes=case["iters"] * (b + es * R * rows), flops=case["iters"] * (f + 4.0 * R * R * rows))
    if op == "gd":  # the products, the factors' own rows, Grams and F H
        return dict(bytes=b + es * R * rows, flops=f + 4.0 * R * R * rows)
    if op == "gdstep":  # a gradient, and one accepted trial: trial factors and its objective
        b1, f1 = b / 3 + 2 * es * R * rows, f / 3 + 2.0 * R * R * rows
        return dict(bytes=case["iters"] * (b + es * R * rows + b1), flops=case["iters"] * (f + 4.0 * R * R * rows + f1))
    # joint: the products; per rating one rank-one update of its user's and its
    # item's system, and those systems solved
    y = case["ratings"]
    return dict(bytes=b + 2 * 8 * y + 2 * es * R * rows,
                flops=f + 2.0 * y * (R * R + 2 * R) + (dims[0] + dims[1]) * (R ** 3 / 3 + 2.0 * R * R))


# ---- 64-bit values --------------------------------------------------------

class _Sorted:
    """COO sorted by each mode's row, for row sums in 64 bits."""

    def __init__(self, coo):
        self.idx, self.val = [x.long() for x in coo[:3]], coo[3].double()
        self.order = [torch.argsort(x, stable=True) for x in self.idx]

    def mttkrp(self, m, F, rows):
        R = F[LEAF[m]].shape[1]
        out = torch.zeros((rows, R), dtype=torch.float64, device=DEV)
        step = max(1 << 14, (1 << 25) // R)
        for a in range(0, self.val.numel(), step):
            o = self.order[m][a:a + step]
            t = F[LEAF[m]][self.idx[LEAF[m]][o]] * F[MID[m]][self.idx[MID[m]][o]] * self.val[o, None]
            r, n = torch.unique_consecutive(self.idx[m][o], return_counts=True)
            c = torch.cumsum(t, 0)[torch.cumsum(n, 0) - 1]
            c[1:] = c[1:] - c[:-1].clone()
            out[r] += c  # a row appears once among r
        return out

    def normsq(self):
        key = (self.idx[0] << 42) | (self.idx[1] << 21) | self.idx[2]
        u, inv = torch.unique(key, return_inverse=True)
        v = torch.zeros(u.numel(), dtype=torch.float64, device=DEV).index_add_(0, inv, self.val)
        return float((v * v).sum()), int(u.numel())


def _had(F, m):
    p, q = F[(m + 1) % 3], F[(m + 2) % 3]
    return (p.t() @ p) * (q.t() @ q)


def _stored(x, dtype):
    return x.float().double() if dtype == "f32" else x.float().to(torch.bfloat16).double()


def _als(S, F, dims, reg, iters, dtype, normsq):
    """CP-ALS in 64 bits from F (lists are updated), with the factors rounded
    to their storage type between modes where that is BF16."""
    bf = dtype == "bf16"
    for _ in range(iters):
        for m in range(3):
            M = S.mttkrp(m, F, dims[m])
            H = _had(F, m) + reg * torch.eye(M.shape[1], dtype=torch.float64, device=DEV)
            N = torch.linalg.solve(H.cpu(), M.t().cpu()).t().contiguous().to(DEV)
            lam = N.norm(dim=0)
            F[m] = N / torch.where(lam > 0, lam, torch.ones_like(lam))
            if bf:
                F[m] = _stored(F[m], dtype)
    G = [x.t() @ x for x in F]
    inner = (F[2] * lam * M).sum()
    xh = (lam[:, None] * lam[None, :] * G[0] * G[1] * G[2]).sum()
    res = torch.clamp(normsq + xh - 2 * inner, min=0.0)
    return lam, (1 - torch.sqrt(res) / math.sqrt(normsq)).reshape(1)


def _gd(S, F, dims, reg, normsq):
    G = [x.t() @ x for x in F]
    M = [S.mttkrp(m, F, dims[m]) for m in range(3)]
    eye = torch.eye(F[0].shape[1], dtype=torch.float64, device=DEV)
    grads = [-M[m] + F[m] @ (_had(F, m) + reg * eye) for m in range(3)]
    return grads, _objective(F, G, M[0], reg, normsq)


def _objective(F, G, M0, reg, normsq):
    return 0.5 * (normsq - 2 * (F[0] * M0).sum() + (G[0] * G[1] * G[2]).sum()) + \
        0.5 * reg * sum(x.diagonal().sum() for x in G)


def _gdsteps(S, F, dims, case, normsq):
    dt, alpha, steps = case["dtype"], 1.0, []
    for _ in range(case["iters"]):
        grads, f0 = _gd(S, F, dims, case["reg"], normsq)
        gn = sum((g * g).sum() for g in grads)
        took, f = 0.0, f0
        a = alpha
        for t in range(60):
            T = [_stored(x - a * g.float().double(), dt) for x, g in zip(F, grads)]
            ft = _objective(T, [x.t() @ x for x in T], S.mttkrp(0, T, dims[0]), case["reg"], normsq)
            if ft <= f0 - 1e-4 * a * gn:
                took, f = a, ft
                F[:] = T
                break
            a *= 0.5
        alpha = 2.0 * took if took else alpha
        steps.append([float(f0), float(f), float(gn), None])
    return dict(F=list(F), G=grads, steps=steps)


def _joint(S, F, dims, case, y):
    """One ALS iteration of the joint model: each user's and item's R x R
    system formed and solved in 64 bits."""
    mu, lam, R, dt = case["mu"], case["lam"], case["R"], case["dtype"]
    eye = torch.eye(R, dtype=torch.float64, device=DEV)
    ij, val = [y[0].long(), y[1].long()], y[3].double()
    for m in range(2):
        B = F[1 - m]
        base = mu * _had(F, m) + lam * eye
        rhs = mu * S.mttkrp(m, F, dims[m])
        o = torch.argsort(ij[m], stable=True)
        cnt = torch.bincount(ij[m], minlength=dims[m])
        end = torch.cumsum(cnt, 0)
        out = torch.empty_like(rhs)
        step = 1 << 14
        for a in range(0, dims[m], step):
            b = min(dims[m], a + step)
            lo = int(end[a - 1]) if a else 0
            row = torch.repeat_interleave(torch.arange(b - a, device=DEV), cnt[a:b])
            H = torch.zeros((b - a, R * R), dtype=torch.float64, device=DEV)
            for c in range(lo, int(end[b - 1]), 1 << 16):
                e = min(int(end[b - 1]), c + (1 << 16))
                v = B[ij[1 - m][o[c:e]]]
                rr, n = torch.unique_consecutive(row[c - lo:e - lo], return_counts=True)
                at = torch.cumsum(n, 0) - 1
                for X, z in ((H, (v[:, :, None] * v[:, None, :]).reshape(e - c, R * R)),
                             (rhs[a:b], v * val[o[c:e], None])):
                    s = torch.cumsum(z, 0)[at]
                    s[1:] = s[1:] - s[:-1].clone()
                    X[rr] += s
            L = torch.linalg.cholesky(H.reshape(b - a, R, R) + base)
            out[a:b] = torch.cholesky_solve(rhs[a:b, :, None], L)[:, :, 0]
        F[m] = _stored(out, dt) if dt == "bf16" else out
    H = mu * _had(F, 2) + lam * eye
    F[2] = mu * torch.linalg.solve(H.cpu(), S.mttkrp(2, F, dims[2]).t().cpu()).t().to(DEV)
    return F


def exact(case, seed):
    op = case["op"]
    if op == "group":
        mem, coos, start, sizes = _group_inputs(case, seed)
        flat, lams, fits = start.double(), [], []
        for (dims, _, _, R), coo, F in zip(mem, coos, _views(mem, flat, sizes)):
            S, X = _Sorted(coo), list(F)
            lam, fit = _als(S, X, dims, 0.0, case["iters"], case["dtype"], float((S.val ** 2).sum()))
            for f, x in zip(F, X):
                f.copy_(x)
            lams.append(lam)
            fits.append(fit)
        return dict(factors=flat, lam=torch.cat(lams), fit=torch.cat(fits))
    dims = _dims(case)
    F = [x.double() for x in _factors(dims, case["R"], case["dtype"], _gen(seed + 7))]
    coo = _coo(dims, case["nnz"], case["s"], seed, raw=op == "build")
    S = _Sorted(coo)
    if op == "mttkrp":
        return [S.mttkrp(m, F, dims[m]) for m in range(3)]
    if op == "build":
        return dict(M=[S.mttkrp(m, F, dims[m]) for m in range(3)], nnz=None, nfib=None, nroot=None, nentry=None,
                    normsq=S.normsq()[0])
    if op == "joint":
        y = _coo((dims[0], dims[1], 1), case["ratings"], case["s"], seed + 3)
        return _joint(S, F, dims, case, y)
    normsq = float((S.val ** 2).sum())
    if op == "als":
        lam, fit = _als(S, F, dims, case["reg"], case["iters"], case["dtype"], normsq)
        return dict(F=F, lam=lam, fit=fit)
    if op == "gd":
        G, f = _gd(S, F, dims, case["reg"], normsq)
        return dict(G=G, f=f.reshape(1))
    return _gdsteps(S, F, dims, case, normsq)
