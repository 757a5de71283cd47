"""The work this framework is measured by: one dict per case.

A case is a call, or the short sequence of calls, that a user's program makes
through the Python API (``paper_2103_16141_amd.api`` and ``soft_assign``) on a
seeded corpus of the shapes the repository's workloads use: Poisson row
lengths, Zipf term ids, lognormal values, unit rows.  Corpora are made on the
GPU from the seed alone.

Kinds of case (``"kind"``):

  serve    new objects against a trained file: ``assign_noalloc`` (small
           requests that must not allocate) or ``assign``, iter = 1
  first    the start of a run: ``init_centroids`` from k seeded objects and
           the first assignment step, every list walked
  step     one Lloyd iteration in the middle of a run: ``update`` from
           a^[r-1], assignment step r, and the new centroids copied out
  lloyd    a whole ``run_lloyd`` from the seeds and its centroids
  resume   a restart from a saved state: ``resume`` and the export of the
           structured file it builds
  soft     the differentiable form, loss and gradients through autograd
  softfwd  its forward alone (lse of every object and the loss)
"""
import math

import numpy as np
import torch

from paper_2103_16141_amd.api import Context, DeviceCsr, Lloyd
from paper_2103_16141_amd.soft_assign import soft_assign_loss

TAU = 0.05


def _case(kind, name=None, **kw):
    c = dict(kind=kind, n=1000, d=5000, lam=50, zipf=1.1, k=100, x="f32", post="fp32", mode="sivf", iters=2, train=0)
    c.update(kw)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest request a clustering service answers: 64 new documents
        # against 100 trained clusters; launches and synchronisations count
        _case("serve", "serve-64", n=64, d=5000, lam=50, zipf=1.0, k=100, train=10_000),
        # a batch of new documents against a larger, ragged model, BF16
        # postings; two tiles of centroids
        _case("serve", "serve-20k-bf16", n=20_011, d=30_011, lam=60, k=1_531, post="bf16", train=60_000),
        # the repository's smallest workload as a whole: 10,000 FP64 objects,
        # k = 100, 10 Lloyd iterations
        _case("lloyd", "lloyd-10k-f64", n=10_000, d=5_000, lam=50, zipf=1.0, k=100, x="f64", iters=10),
        # an iteration of the 1M-object workload (k = 1,000, one tile)
        _case("step", "step-1m-k1000", n=1_000_000, d=100_000, lam=100, k=1_000, iters=2),
        # an iteration at the headline k = 10,000 and D = 140,000, on a
        # quarter of its objects: the largest case
        _case("step", "step-2m-k10k", n=2_000_000, d=140_000, lam=90, k=10_000, iters=2),
        # the precision form's k = 20,000 at the start of a run
        _case("first", "first-400k-k20k-bf16", n=400_000, d=140_000, lam=90, k=20_000, post="bf16"),
        # late in a run: most clusters invariant, relaxed filter, odd sizes
        _case("step", "late-100k-relaxed", n=100_003, d=30_011, lam=60, k=1_003, mode="relaxed", iters=12),
        # long rows over a wide vocabulary (the NYT-shaped corpus), BF16
        _case("step", "step-nyt-60k-bf16", n=60_000, d=495_714, lam=226, k=1_000, post="bf16", iters=2),
        # a checkpoint read back and written out again
        _case("resume", "resume-200k", n=200_000, d=50_000, lam=80, k=2_000, iters=2),
        # a small differentiable step inside a larger model
        _case("soft", "soft-1k", n=1_000, d=5_000, lam=50, k=100),
        # an ordinary one at odd sizes (k no multiple of 4: unaligned rows)
        _case("soft", "soft-20k-odd", n=20_011, d=30_011, lam=90, k=1_021),
        # the differentiation form at its own size
        _case("soft", "soft-262k", n=262_144, d=100_000, lam=100, k=4_096),
    ]


def _logu(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ranges; sizes log-uniform, most of them odd,
    bounded so that none costs more than the largest listed one."""
    kind = rng.choice(["serve", "first", "step", "step", "lloyd", "resume", "soft", "softfwd"])
    d = _logu(rng, 5_000, 200_000)
    lam = _logu(rng, 30, 200)
    post = rng.choice(["fp32", "bf16"])
    zipf = rng.choice([1.0, 1.1])
    if kind in ("soft", "softfwd"):
        k = _logu(rng, 50, 4_096)
        # dC and C are dense: k * d bounded by the differentiation form's own
        return _case(kind, n=_logu(rng, 500, min(260_000, int(1e11 / (lam * k)))), d=min(d, int(4e8 // k)), lam=lam,
                     zipf=zipf, k=k)
    if kind == "serve":
        k = _logu(rng, 50, 4_000)
        return _case(kind, n=_logu(rng, 16, 100_000), d=d, lam=lam, zipf=zipf, k=k, post=post,
                     train=max(4 * k, 20_000))
    if kind == "lloyd":
        return _case(kind, n=_logu(rng, 4_000, 60_000), d=min(d, 60_000), lam=lam, zipf=zipf, k=_logu(rng, 16, 600),
                     x=rng.choice(["f32", "f64"]), post=post, iters=rng.randint(3, 10))
    k = _logu(rng, 200, 12_000)
    n = _logu(rng, max(20_000, 4 * k), max(8 * k, int(min(1e6, 5e11 / (lam * k)))))
    if kind == "step":
        return _case(kind, n=n, d=d, lam=lam, zipf=zipf, k=k, post=post, mode=rng.choice(["sivf", "sivf", "relaxed"]),
                     iters=rng.randint(1, 4))
    return _case(kind, n=n, d=d, lam=lam, zipf=zipf, k=k, post=post)


# ------------------------------------------------------------------ inputs
def _zipf_cdf(d, s):
    w = np.arange(1, d + 1, dtype=np.float64) ** (-float(s))
    c = np.cumsum(w)
    return torch.from_numpy(c / c[-1]).cuda()


def _distinct(gen, want, cdf, more=1):
    """want[i] distinct terms for each row i, as ascending keys row * d + term:
    the first distinct ones of an independent sequence of draws (rows whose
    sequence was too short take a longer one)."""
    d, m = cdf.numel(), want.numel()
    tries = more * (2 * want + 16)
    start = torch.cumsum(tries, 0) - tries
    row = torch.repeat_interleave(torch.arange(m, device="cuda"), tries)
    u = torch.rand(row.numel(), device="cuda", dtype=torch.float64, generator=gen)
    key = row * d + torch.searchsorted(cdf, u).clamp_(max=d - 1)
    key, at = torch.sort(key, stable=True)
    new = torch.ones_like(key, dtype=torch.bool)
    new[1:] = key[1:] != key[:-1]
    seen = torch.zeros_like(key)
    seen[at] = new.long()
    upto = torch.cumsum(seen, 0)
    rank = upto - (upto[start] - seen[start])[row]        # distinct terms of the row so far
    keep = (seen > 0) & (rank <= want[row])
    key = key[keep[at]]
    got = torch.bincount(key // d, minlength=m)
    short = (got < want).nonzero().flatten()
    if short.numel():
        longer = _distinct(gen, want[short], cdf, 4 * more)
        key = key[~torch.isin(key // d, short)]
        key = torch.sort(torch.cat([key, short[longer // d] * d + longer % d])).values
    return key


def _corpus(gen, n, d, lam, zipf, dtype):
    """n rows over d terms: Poisson(lam) distinct Zipf terms each, exp(N(0, 1))
    values divided by the row's L2 norm.  Row lengths depend on the sizes only,
    so every seed has the same number of nonzeros; row norms are summed as
    integers, so the same seed gives the same bits."""
    cdf = _zipf_cdf(d, zipf)
    lens = torch.poisson(torch.full((n,), float(lam), device="cuda"), generator=_gen(n))
    lens = lens.long().clamp_(1, d // 2)
    block = max(1, 40_000_000 // (2 * lam + 16))
    key = torch.cat([_distinct(gen, lens[b:b + block], cdf) + b * d for b in range(0, n, block)])
    row = key // d
    col = (key - row * d).int()
    row_ptr = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    row_ptr[1:] = torch.cumsum(lens, 0)
    v = torch.exp(torch.randn(key.numel(), device="cuda", dtype=torch.float64, generator=gen))
    ss = torch.zeros(n, dtype=torch.int64, device="cuda").index_add_(0, row, (v * v * 2.0 ** 24).round_().long())
    v /= torch.sqrt(ss.double() / 2.0 ** 24)[row]
    return DeviceCsr(row_ptr, col, v if dtype == "f64" else v.float(), d)


def _seeds(seed, n, k):
    """k distinct objects (a soft case may have more centroids than objects)."""
    ids = np.random.Generator(np.random.PCG64(seed)).permutation(n)
    return np.resize(ids, k).astype(np.int32)


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _inputs(case, seed):
    """(training corpus or None, objects, seed ids) of a case."""
    g = _gen(seed)
    args = (case["d"], case["lam"], case["zipf"], case["x"])
    train = _corpus(g, case["train"], *args) if case["train"] else None
    X = _corpus(g, case["n"], *args)
    return train, X, _seeds(seed, (train or X).n_rows, case["k"])


def _dense_centroids(case, seed, X, ids):
    """Unit rows around k objects: the row plus 1e-3 |N(0, 1)| everywhere."""
    C = torch.randn(case["k"], case["d"], device="cuda", generator=_gen(seed + 1)).abs_().mul_(1e-3)
    for j, i in enumerate(ids.tolist()):
        lo, hi = X.row_ptr[i], X.row_ptr[i + 1]
        C[j, X.col[lo:hi].long()] += X.val[lo:hi]
    for lo in range(0, case["k"], 256):
        C[lo:lo + 256] /= torch.linalg.vector_norm(C[lo:lo + 256].double(), dim=1, keepdim=True).float()
    return C


def _room(X, *names):
    """Buffers for a file's entries (at most one per object nonzero), of the
    same size for every seed; entries past the file's own stay zero."""
    types = dict(c_col=torch.int32, c_val=torch.float64, p_cid=torch.int32, p_val=torch.float64)
    return {m: torch.zeros(X.nnz, dtype=types[m], device="cuda") for m in names}


def _into(room, **entries):
    for m, t in entries.items():
        room[m][:t.numel()].copy_(t)
    return room


def _context(case):
    return Context(0, posting_dtype=case["post"], filter_mode=case["mode"])


def prepare(case, seed):
    kind = case["kind"]
    train, X, ids = _inputs(case, seed)
    s = dict(case=case, X=X)
    if kind in ("soft", "softfwd"):
        s["C"] = _dense_centroids(case, seed, X, ids)
        if kind == "soft":
            s["C"].requires_grad_(True)
            X.val.requires_grad_(True)
        else:
            s["ctx"] = Context(0)
        return s
    ctx = s["ctx"] = _context(case)
    n, k, dev = X.n_rows, case["k"], ctx.device
    if kind in ("lloyd", "first"):
        s["ids"] = ids
    if kind in ("lloyd", "step"):
        s["room"] = _room(X, "c_col", "c_val")
    if kind == "resume":
        s["room"] = _room(X, "c_col", "c_val", "p_cid", "p_val")
    if kind == "serve":
        _, _, s["ivf"], _ = ctx.run_lloyd(train, k, ids, 3)
    if kind in ("serve", "first"):
        s["a"] = torch.zeros(n, dtype=torch.int32, device=dev)
        s["own"] = torch.zeros(n, dtype=torch.float32, device=dev)
        s["lam"] = torch.zeros(k, dtype=torch.uint8, device=dev)
    if kind in ("step", "resume"):
        L = Lloyd(ctx, X, k, ids)
        prev = None
        for r in range(case["iters"]):
            if r:
                L.update()
                prev = L.a.clone()
            L.assign()
        if kind == "resume":
            L.update()
            s.update(C=L.ivf.centroids(), a=L.a, a_prev=prev)
            L.ivf.free()
        else:
            # the state between the two steps: assignments, own similarities
            # and flags of step r - 1, the file still holding mu^[r-2]
            s.update(ivf=L.ivf, a0=L.a, own0=L.own, own64_0=L.own64, lam0=L.lam, r=L.r + 1, a=L.a.clone(),
                     own=L.own.clone(), own64=None if L.own64 is None else L.own64.clone(), lam=L.lam.clone())
    return s


# ------------------------------------------------------------------ one pass
def _counts(st):
    return {n: st[n] for n in ("multadds", "moved", "icp_objects", "n_invariant", "relaxed_objects")}


def run(s):
    case, X = s["case"], s["X"]
    kind = case["kind"]
    if kind == "soft":
        loss = soft_assign_loss(X, s["C"], TAU)
        dC, dX = torch.autograd.grad(loss, (s["C"], X.val))
        return dict(loss=loss.detach(), dC=dC, dX=dX)
    ctx = s["ctx"]
    if kind == "softfwd":
        lse, loss = ctx.soft_assign_fwd(X, s["C"], TAU)
        return dict(lse=lse, loss=loss)
    if kind == "serve":
        # the no-allocation entry point takes small requests
        call = ctx.assign_noalloc if X.n_rows <= 100_000 and case["k"] <= 1024 else ctx.assign
        st = call(X, s["ivf"], 1, s["a"], s["own"], s["lam"])
        return dict(a=s["a"], own=s["own"], **_counts(st))
    if kind == "first":
        ivf = ctx.init_centroids(X, case["k"], s["ids"])
        st = ctx.assign(X, ivf, 1, s["a"], s["own"], s["lam"])
        ivf.free()
        return dict(a=s["a"], own=s["own"], lam=s["lam"], **_counts(st))
    if kind == "lloyd":
        a, own, ivf, stats = ctx.run_lloyd(X, case["k"], s["ids"], case["iters"])
        C = ivf.centroids()
        ivf.free()
        return dict(a=a, own=own, c_ptr=C.row_ptr, iters=len(stats), multadds=sum(st["multadds"] for st in stats),
                    **_into(s["room"], c_col=C.col, c_val=C.val))
    if kind == "resume":
        ivf, own, _ = ctx.resume(X, s["C"], s["a"], s["a_prev"])
        ex = ivf.export()
        ivf.free()
        _into(s["room"], **{m: ex[m] for m in s["room"]})
        return dict(own=own, **{**ex, **s["room"]})
    ctx.update(X, s["a0"], s["lam0"], s["ivf"])
    C = s["ivf"].centroids()
    s["a"].copy_(s["a0"])
    s["own"].copy_(s["own0"])
    if s["own64"] is not None:
        s["own64"].copy_(s["own64_0"])
    st = ctx.assign(X, s["ivf"], s["r"], s["a"], s["own"], s["lam"], own64=s["own64"])
    return dict(a=s["a"], own=s["own"], lam=s["lam"], c_ptr=C.row_ptr, **_into(s["room"], c_col=C.col, c_val=C.val),
                **_counts(st))


# ------------------------------------------------------------------ floors
def _term_probs(case):
    """P(term in a row) for rows of lam distinct terms."""
    w = np.arange(1, case["d"] + 1, dtype=np.float64) ** (-float(case["zipf"]))
    p = w / w.sum()
    lo, hi = 1.0, 1e6
    for _ in range(60):
        m = math.sqrt(lo * hi)
        lo, hi = (m, hi) if (1.0 - np.exp(m * np.log1p(-p))).sum() < case["lam"] else (lo, m)
    return 1.0 - np.exp(lo * np.log1p(-p))


def work(case):
    """Bytes: objects read once, outputs (and new centroids) written once.
    Operations: two per posting mult-add of the method, from the expected list
    lengths of clusters of equal size (without the filter's saving, which
    depends on the data)."""
    n, k, d, lam, kind = case["n"], case["k"], case["d"], case["lam"], case["kind"]
    nnz = float(n) * lam
    xb = nnz * (12 if case["x"] == "f64" else 8) + 8.0 * n
    if kind in ("soft", "softfwd"):
        both = kind == "soft"
        return dict(bytes=xb + 4.0 * k * d * (2 if both else 1) + 4.0 * (nnz if both else n),
                    flops=(6.0 if both else 2.0) * nnz * k)
    q = _term_probs(case)
    pb = 4 if case["post"] == "bf16" else 6

    def held(members):   # expected share of centroids holding each term
        return 1.0 - np.exp(members * np.log1p(-np.minimum(q, 1 - 1e-12)))

    seeded, grown = held(1.0), held(max(1.0, (case["train"] or n) / k))
    if kind in ("serve", "first"):
        h = grown if kind == "serve" else seeded
        return dict(bytes=xb + k * h.sum() * pb + 8.0 * n, flops=2.0 * n * k * float((q * h).sum()))
    madd = n * k * float((q * grown).sum())
    post = k * float(grown.sum())
    if kind == "resume":
        return dict(bytes=xb + post * (12 + 12 + 12) + 8.0 * n, flops=2.0 * nnz)
    if kind == "lloyd":
        first = n * k * float((q * seeded).sum())
        return dict(bytes=xb + post * 12 + 8.0 * n, flops=2.0 * (first + (case["iters"] - 1) * (madd + nnz)))
    return dict(bytes=xb + post * (12 + pb) + 16.0 * n, flops=2.0 * (madd + nnz))


# ------------------------------------------------------------------ 64 bits
def _rows(X):
    return torch.repeat_interleave(torch.arange(X.n_rows, device="cuda"), X.row_ptr[1:] - X.row_ptr[:-1])


def _sparse64(X, lo, hi):
    b, e = int(X.row_ptr[lo]), int(X.row_ptr[hi])
    return torch.sparse_csr_tensor(X.row_ptr[lo:hi + 1] - b, X.col[b:e].long(), X.val[b:e].detach().double(),
                                   size=(hi - lo, X.n_cols))


def _step_rows(k):
    return max(1, (1 << 28) // k)


def _best64(X, C):
    """Largest similarity of every object and its centroid, FP64 (C: k x d)."""
    CT = C.t().contiguous()
    own = torch.empty(X.n_rows, dtype=torch.float64, device="cuda")
    a = torch.empty(X.n_rows, dtype=torch.int64, device="cuda")
    for lo in range(0, X.n_rows, _step_rows(C.shape[0])):
        hi = min(X.n_rows, lo + _step_rows(C.shape[0]))
        own[lo:hi], a[lo:hi] = (_sparse64(X, lo, hi) @ CT).max(dim=1)
    return own, a


def _means64(X, rows, a, C):
    W = torch.zeros_like(C)
    W.view(-1).index_add_(0, a[rows] * C.shape[1] + X.col.long(), X.val.detach().double())
    norm = torch.linalg.vector_norm(W, dim=1)
    empty = norm == 0
    W /= torch.where(empty, torch.ones_like(norm), norm)[:, None]
    W[empty] = C[empty]
    return W


def _nonzeros(C, X):
    v = torch.cat([C[lo:lo + 256][C[lo:lo + 256] != 0] for lo in range(0, C.shape[0], 256)])
    return torch.cat([v, v.new_zeros(X.nnz - v.numel())])


def _seeded64(X, ids, k):
    C = torch.zeros(k, X.n_cols, dtype=torch.float64, device="cuda")
    for j, i in enumerate(ids.tolist()):
        lo, hi = X.row_ptr[i], X.row_ptr[i + 1]
        C[j, X.col[lo:hi].long()] = X.val[lo:hi].double()
    return C


def _lloyd64(X, ids, k, iters):
    """Centroids and assignment after `iters` assignment steps of plain Lloyd."""
    rows, C, a, own = _rows(X), _seeded64(X, ids, k), None, None
    for r in range(iters):
        if r:
            C = _means64(X, rows, a, C)
        before = a
        own, a = _best64(X, C)
        if r and torch.equal(a, before):
            break
    return rows, C, a, own


def _soft64(case, seed, X, ids):
    C = _dense_centroids(case, seed, X, ids)
    k, rows = case["k"], _rows(X)
    CT = C.double().t().contiguous()
    both = case["kind"] == "soft"
    lse = torch.empty(X.n_rows, dtype=torch.float64, device="cuda")
    dCT = torch.zeros_like(CT) if both else None
    dX = torch.empty(X.nnz, dtype=torch.float64, device="cuda") if both else None
    for lo in range(0, X.n_rows, _step_rows(k)):
        hi = min(X.n_rows, lo + _step_rows(k))
        b, e = int(X.row_ptr[lo]), int(X.row_ptr[hi])
        S = (_sparse64(X, lo, hi) @ CT) / TAU
        lse[lo:hi] = torch.logsumexp(S, dim=1)
        if not both:
            continue
        dS = torch.exp(S - lse[lo:hi, None]).mul_(-1.0 / TAU)
        del S
        col, row, val = X.col[b:e].long(), rows[b:e] - lo, X.val[b:e].detach().double()
        order = torch.argsort(col, stable=True)
        ptr = torch.zeros(X.n_cols + 1, dtype=torch.int64, device="cuda")
        ptr[1:] = torch.cumsum(torch.bincount(col, minlength=X.n_cols), 0)
        dCT += torch.sparse_csr_tensor(ptr, row[order], val[order], size=(X.n_cols, hi - lo)) @ dS
        for q in range(0, e - b, _step_rows(k)):
            z = slice(q, min(e - b, q + _step_rows(k)))
            dX[b + z.start:b + z.stop] = (CT[col[z]] * dS[row[z]]).sum(dim=1)
        del dS
    out = dict(loss=-lse.sum())
    return dict(out, dC=dCT.t().contiguous(), dX=dX) if both else dict(out, lse=lse)


def exact(case, seed):
    kind, k = case["kind"], case["k"]
    train, X, ids = _inputs(case, seed)
    if kind in ("soft", "softfwd"):
        return _soft64(case, seed, X, ids)
    counts = dict.fromkeys(("multadds", "moved", "icp_objects", "n_invariant", "relaxed_objects"))
    if kind == "serve":
        _, C, _, _ = _lloyd64(train, ids, k, 3)
        return dict(a=None, own=_best64(X, C)[0], **counts)
    if kind == "first":
        return dict(a=None, own=_best64(X, _seeded64(X, ids, k))[0], lam=None, **counts)
    rows, C, a, own = _lloyd64(X, ids, k, case["iters"])
    if kind == "lloyd":
        return dict(a=None, own=own, c_ptr=None, c_col=None, c_val=_nonzeros(C, X), iters=None, multadds=None)
    C = _means64(X, rows, a, C)
    if kind == "resume":
        # a_prev's similarity to its new centroid
        own = torch.empty(X.n_rows, dtype=torch.float64, device="cuda")
        own.zero_().index_add_(0, rows, X.val.double() * C.view(-1)[a[rows] * X.n_cols + X.col.long()])
        vals = _nonzeros(C, X)
        return dict(own=own, c_ptr=None, lam=None, term_ptr=None, split=None, c_col=None, c_val=vals, p_cid=None,
                    p_val=None)
    own = _best64(X, C)[0]
    return dict(a=None, own=own, lam=None, c_ptr=None, c_col=None, c_val=_nonzeros(C, X), **counts)
