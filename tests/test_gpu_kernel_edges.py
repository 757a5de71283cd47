"""Kernels at the sizes where their work splits change: window and tile edges,
remainders, smallest and largest cases, against the oracle or the general
statement of what they compute."""
import numpy as np
import pytest
import torch

import oracle
import synth
from tests.gpu_util import device, log

pytestmark = pytest.mark.gpu


def _ctx(**kw):
    from paper_2103_16141_amd.api import Context
    return Context(0, **kw)


def _status(fn):
    from paper_2103_16141_amd._native import SivfError
    try:
        fn()
    except SivfError as e:
        return e.name, str(e)
    return "SIVF_OK", ""


# ---------------------------------------------------------------- validation
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("shift", [0, 1])
def test_validation_of_long_and_short_rows_at_window_edges(dtype, shift):
    # nonzeros are read 4 per thread and 256 per wave whatever their rows; rows
    # of 1, 255 .. 257, 1,023 .. 1,025 and 5,000 nonzeros put faults on both
    # sides of those edges, and shift = 1 takes arrays off 16-byte alignment
    from paper_2103_16141_amd.api import DeviceCsr
    log("validation windows %s shift %d" % (np.dtype(dtype), shift))
    lens = [1, 255, 256, 257, 0, 1023, 1024, 1025, 0, 0, 5000, 3]
    d = 6000
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    col = np.concatenate([np.arange(m) for m in lens]).astype(np.int32)   # every row starts below its predecessor's end
    val = np.ones(rp[-1], dtype)
    ctx = _ctx()

    def check(c, v):
        cc = torch.from_numpy(np.concatenate([np.zeros(shift, np.int32), c])).to(device())[shift:]
        vv = torch.from_numpy(np.concatenate([np.zeros(shift, dtype), v])).to(device())[shift:]
        return _status(lambda: ctx.validate(DeviceCsr(torch.from_numpy(rp).to(device()), cc, vv, d)))

    assert check(col, val)[0] == "SIVF_OK"
    rows = np.repeat(np.arange(len(lens)), lens)
    edges = sorted({p for e in (256, 512, 768, 1024, 2048, 4096, len(col)) for p in (e - 1, e, e + 1) if 0 < p < len(col)})
    for p in edges:
        if rows[p] == rows[p - 1]:
            c = col.copy()
            c[p] = c[p - 1]
            name, msg = check(c, val)
            assert name == "SIVF_E_UNSORTED" and "row %d " % rows[p] in msg, p
        if p + 1 == len(col) or rows[p] != rows[p + 1]:
            c = col.copy()
            c[p] = d
            name, msg = check(c, val)
            assert name == "SIVF_E_RANGE" and "row %d " % rows[p] in msg, p
        v = val.copy()
        v[p] = -np.inf if p % 2 else np.nan
        name, msg = check(col, v)
        assert name == "SIVF_E_NONFINITE" and "row %d " % rows[p] in msg, p


# ---------------------------------------------------------------- member sums
def _rows_corpus(lens, d, dtype, seed, signed):
    """Rows of the given lengths, terms spread over [0, d), unit norm; signed:
    half the rows are the negated copy of the row before them."""
    rng = np.random.default_rng(seed)
    cols, vals = [], []
    for i, m in enumerate(lens):
        if signed and i % 2 and m == lens[i - 1]:
            cols.append(cols[-1])
            vals.append(-vals[-1])
            continue
        cols.append(np.sort(rng.choice(d, m, replace=False)).astype(np.int32))
        v = np.exp(rng.standard_normal(m))
        vals.append(v / np.sqrt((v * v).sum()) if m else v)
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    return synth.Corpus(len(lens), d, rp, np.concatenate(cols).astype(np.int32), np.concatenate(vals).astype(dtype))


# (row lengths, d): 4,096 nonzeros are summed at a time and 512 members enter a
# tile; 2^7 and 2^14 terms are where the sort takes another pass
_MEMBERS = {
    "one tile exactly": ([64] * 64, 700),
    "one nonzero over a tile": ([64] * 64 + [1], 700),
    "512 short members": ([3] * 512, 128),
    "513 short members": ([3] * 513, 129),
    "rows longer than a tile": ([4095, 4096, 4097, 9000, 1], 16384),
    "empty rows between and around": ([0, 0, 5, 0, 4100, 0, 0, 7, 0], 16385),
    "every term touched, many tiles": ([900] * 40, 1000),
    "a wide vocabulary": ([300] * 90, 150_001),
    "one term": ([1] * 5000, 1),
    # 8 tiles and more: term ranges side by side; the first has a term in every row
    "cut into ranges": ([64] * 512, 600),
    "just too small to cut": ([64] * 511 + [63], 600),
    "two tiles exactly, cut": ([64] * 128, 600),
    "two tiles less one, whole": ([64] * 127 + [63], 600),
    "more members than enter a tile, cut": ([40] * 1500 + [0, 700, 4099], 5000),
}


@pytest.mark.parametrize("name", list(_MEMBERS))
@pytest.mark.parametrize("dtype,signed", [(np.float32, False), (np.float64, False), (np.float32, True)])
def test_update_at_the_tile_edges_of_the_member_sums(name, dtype, signed):
    # three clusters: the listed rows, one row, none; then the listed rows and
    # the row swap a member so the accumulators are used again
    from paper_2103_16141_amd.api import DeviceCsr
    from tests.gpu_util import assert_centroids_equal, centroids_from_export
    log("member sums: %s %s signed %d" % (name, np.dtype(dtype).name, signed))
    lens, d = _MEMBERS[name]
    lens = list(lens) + [min(d, 11)]
    c = _rows_corpus(lens, d, dtype, len(name), signed)
    X = DeviceCsr.from_corpus(c, device())
    ids = [0, c.n - 1, min(1, c.n - 1)]
    ctx = _ctx()
    ivf = ctx.init_centroids(X, 3, ids)
    ref = oracle.init_centroids(c, np.array(ids, np.int32))
    lam = torch.zeros(3, dtype=torch.uint8, device=device())
    a = np.zeros(c.n, np.int32)
    a[-1] = 1
    for step in range(3):
        ctx.update(X, torch.from_numpy(a).to(device()), lam, ivf)
        ref, _ = oracle.update(c, a, ref)
        assert_centroids_equal(centroids_from_export(ivf.export(), 3, d), ref, "%s, step %d" % (name, step))
        a[step] = 1 - a[step]


# ---------------------------------------------------------------- soft form
@pytest.mark.parametrize("n,d,lam", [(1, 5, 3), (40, 512, 60), (64, 513, 64), (300, 4096, 90), (200, 262_145, 50)])
def test_soft_gradients_at_the_sort_edges_of_the_column_copy(n, d, lam):
    # one, two and three sort passes (2^9, 2^18 columns), tiles of 4,096
    # nonzeros with a remainder, and empty rows in a run; tolerances as in
    # test_gpu_soft
    from paper_2103_16141_amd.api import DeviceCsr
    log("column copy n=%d d=%d" % (n, d))
    c = synth.make_corpus(n, d, lam, 1.0, np.float32, seed=n + d)
    keep = np.ones(n, bool)
    keep[n // 3:n // 2] = False
    rows = np.repeat(keep, np.diff(c.row_ptr))
    rp = np.concatenate([[0], np.cumsum(np.where(keep, np.diff(c.row_ptr), 0))]).astype(np.int64)
    c = synth.Corpus(n, d, rp, np.ascontiguousarray(c.col[rows]), np.ascontiguousarray(c.val[rows]))
    k = 7
    C = np.abs(np.random.default_rng(d).standard_normal((k, d))).astype(np.float32)
    C /= np.linalg.norm(C, axis=1, keepdims=True)
    X, Cg = DeviceCsr.from_corpus(c, device()), torch.from_numpy(C).to(device())
    ctx = _ctx()
    lse, _ = ctx.soft_assign_fwd(X, Cg, 0.05)
    lse_ref = oracle.soft_forward(c, C.astype(np.float64), 0.05)
    np.testing.assert_allclose(lse.cpu().numpy(), lse_ref, rtol=0, atol=5e-4)
    dC, dX = ctx.soft_assign_bwd(X, Cg, 0.05, lse, 0.7)
    dC_ref, dX_ref = oracle.soft_backward(c, C.astype(np.float64), 0.05, 0.7, lse_ref)
    np.testing.assert_allclose(dC.cpu().numpy(), dC_ref, rtol=2e-3, atol=1e-7)
    np.testing.assert_allclose(dX.cpu().numpy(), dX_ref, rtol=2e-3, atol=1e-9)


@pytest.mark.parametrize("k", [1, 31, 32, 33, 63, 64, 65, 128, 511, 512, 513, 577, 1100])
def test_soft_blocks_of_columns_and_rows_of_every_length_class(k):
    # columns come in blocks of 64 (C^T) and 32 (dS, dC), eight blocks at a time
    # with XCDs sharing the last ones; rows of 0, 1, 15 .. 17, 63 .. 65, 112, 113,
    # 127 .. 129, 200 terms take every register class and the gathered-twice
    # path; terms of 1 .. 8, 9, 512, 513 and 1,400 entries every dC path
    from paper_2103_16141_amd.api import DeviceCsr
    log("soft blocks k=%d" % k)
    rng = np.random.default_rng(k)
    classes = [0, 1, 15, 16, 17, 63, 64, 65, 112, 113, 127, 128, 129, 200]
    d, n = 700, 1400
    lens = np.resize(classes, n)
    # term t < 12 in the first cut[t] rows that are long enough, the rest spread
    cut = [1400, 513, 512, 9, 8, 7, 6, 5, 4, 3, 2, 1]
    cols, used = [], np.zeros(12, int)
    for i in range(n):
        c = [t for t in range(12) if used[t] < cut[t]][:lens[i]]
        used[c] += 1
        rest = rng.choice(np.arange(12, d), lens[i] - len(c), replace=False)
        cols.append(np.sort(np.concatenate([c, rest])).astype(np.int32))
    assert list(used[1:]) == cut[1:]
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    v = np.exp(rng.standard_normal(rp[-1]))
    v /= np.sqrt(np.repeat(np.add.reduceat(np.append(v * v, 0), rp[:-1]), lens))
    c = synth.Corpus(n, d, rp, np.concatenate(cols), v.astype(np.float32))
    C = np.abs(rng.standard_normal((k, d))).astype(np.float32)
    C /= np.linalg.norm(C, axis=1, keepdims=True)
    X, Cg = DeviceCsr.from_corpus(c, device()), torch.from_numpy(C).to(device())
    ctx = _ctx()
    lse, loss = ctx.soft_assign_fwd(X, Cg, 0.05)
    lse_ref = oracle.soft_forward(c, C.astype(np.float64), 0.05)
    np.testing.assert_allclose(lse.cpu().numpy(), lse_ref, rtol=0, atol=5e-4)
    assert abs(loss + lse.double().sum().item()) <= 1e-9 * abs(loss)
    dC, dX = ctx.soft_assign_bwd(X, Cg, 0.05, lse, 1.1)
    dC_ref, dX_ref = oracle.soft_backward(c, C.astype(np.float64), 0.05, 1.1, lse_ref)
    np.testing.assert_allclose(dC.cpu().numpy(), dC_ref, rtol=2e-3, atol=1e-7)
    np.testing.assert_allclose(dX.cpu().numpy(), dX_ref, rtol=2e-3, atol=1e-9)
    again = ctx.soft_assign_bwd(X, Cg, 0.05, lse, 1.1)
    assert torch.equal(again[0], dC) and torch.equal(again[1], dX)
    alone = ctx.soft_assign_bwd(X, Cg, 0.05, lse, 1.1, want_dc=False)
    assert alone[0] is None and torch.equal(alone[1], dX)


def test_soft_forward_keeps_infinities_to_their_own_terms():
    # a -inf in one centroid's row of term 0 must not reach rows without that
    # term, and a whole block of -inf similarities still leaves a finite lse
    from paper_2103_16141_amd.api import DeviceCsr
    log("soft infinities")
    rp = torch.tensor([0, 2, 3, 5], device=device())
    col = torch.tensor([1, 2, 2, 0, 3], dtype=torch.int32, device=device())
    val = torch.tensor([0.6, 0.8, 1.0, 0.6, 0.8], device=device())
    C = torch.rand(130, 4, device=device())
    C[64:128, 0] = -float("inf")
    lse, _ = _ctx().soft_assign_fwd(DeviceCsr(rp, col, val, 4), C, 0.05)
    X = torch.zeros(3, 4, dtype=torch.float64, device=device())
    X[0, 1], X[0, 2], X[1, 2], X[2, 0], X[2, 3] = 0.6, 0.8, 1.0, 0.6, 0.8
    S = torch.zeros(3, 130, dtype=torch.float64, device=device())
    for t in range(4):   # term by term: 0 * inf must not appear
        hit = X[:, t] != 0
        S[hit] += X[hit, t:t + 1] * C[:, t].double()[None]
    want = torch.logsumexp(S / 0.05, 1)
    assert torch.isfinite(lse).all() and (lse.double() - want).abs().max() < 5e-4


# ---------------------------------------------------------------- walk
@pytest.mark.parametrize("posting", ["fp32", "bf16"])
@pytest.mark.parametrize("k", [60, 1500])
def test_assignment_of_batches_on_both_sides_of_the_work_shares(posting, k):
    # up to 8 objects a wave the objects are shared out, beyond that grabbed
    # (5,120 FP32 and 6,144 BF16 waves; half and less with wide tiles): every
    # batch must give what the first step gives for the same rows in one call
    from paper_2103_16141_amd.api import DeviceCsr
    log("batches %s k=%d" % (posting, k))
    c = synth.make_corpus(52_000, 900, 12, 1.1, np.float32, seed=k)
    X = DeviceCsr.from_corpus(c, device())
    ctx = _ctx(posting_dtype=posting)
    ivf = ctx.init_centroids(X, k, synth.init_ids(c.n, k, 3))

    def run(lo, hi):
        a = torch.full((hi - lo,), -1, dtype=torch.int32, device=device())
        own = torch.zeros(hi - lo, dtype=torch.float32, device=device())
        lam = torch.zeros(k, dtype=torch.uint8, device=device())
        b, e = int(c.row_ptr[lo]), int(c.row_ptr[hi])
        rows = DeviceCsr(X.row_ptr[lo:hi + 1] - b, X.col[b:e].clone(), X.val[b:e].clone(), c.d)
        return a, own, ctx.assign(rows, ivf, 1, a, own, lam)["multadds"]

    a, own, m = run(0, c.n)
    ref, _, _ = oracle.assign(c, oracle.init_centroids(c, synth.init_ids(c.n, k, 3)), rows=np.arange(0, c.n, 97))
    assert np.array_equal(a.cpu().numpy()[::97], ref)
    cuts = [0, 1, 4, 9, 5130, 5130 + 40_960, c.n]
    total = 0
    for lo, hi in zip(cuts[:-1], cuts[1:]):
        pa, po, pm = run(lo, hi)
        assert torch.equal(pa, a[lo:hi]) and torch.equal(po, own[lo:hi])
        total += pm
    assert total == m
    pa, po, _ = run(0, 40_961)
    assert torch.equal(pa, a[:40_961]) and torch.equal(po, own[:40_961])


# ---------------------------------------------------------------- structured file
@pytest.mark.parametrize("k,d", [(1, 3), (63, 400), (64, 8191), (65, 8192), (1023, 8193), (1024, 300), (1025, 300),
                                 (2049, 700), (17_000, 90)])
@pytest.mark.parametrize("posting", ["fp32", "bf16"])
def test_file_of_centroids_at_the_piece_and_scan_edges(k, d, posting):
    # entries are handled 256 at a time wherever the centroids begin, positions
    # 1,024 centroids at a time, scans of up to 16,384 elements in one
    # workgroup; centroids of 0, 1, 255 .. 257 and all entries, random flags
    log("file k=%d d=%d %s" % (k, d, posting))
    rng = np.random.default_rng(k + d)
    lens = np.minimum(np.resize([0, 1, 255, 256, 257, 7, 40, d], k), d)
    if k > 2000:
        lens = np.minimum(lens, 40)
    ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    col = np.concatenate([np.sort(rng.choice(d, m, replace=False)) for m in lens] + [np.zeros(0)]).astype(np.int32)
    val = rng.standard_normal(len(col))
    lam = (rng.random(k) < 0.4).astype(np.uint8)
    ctx = _ctx(posting_dtype=posting)
    ivf = ctx.build_centroid_ivf(*[torch.from_numpy(x).to(device()) for x in (ptr, col, val)], d,
                                 torch.from_numpy(lam).to(device()))
    ex = {m: t.cpu().numpy() for m, t in ivf.export().items()}
    ref = oracle.build_ivf(oracle.Centroids(k, d, ptr, col, val), lam)
    assert np.array_equal(ex["c_ptr"], ptr) and np.array_equal(ex["c_col"], col) and np.array_equal(ex["c_val"], val)
    assert np.array_equal(ex["term_ptr"], ref.term_ptr) and np.array_equal(ex["split"], ref.split)
    assert np.array_equal(ex["p_cid"], ref.cid) and np.array_equal(ex["p_val"], ref.val)


# ---------------------------------------------------------------- split walk
def _striped(n, d, lam, seed, dtype, signed=False, empty=False):
    """n unit rows of lam terms, one from each of lam stripes of the d terms
    (the first terms of a stripe more often); rows 0, 7, 14, .. empty if asked."""
    from paper_2103_16141_amd.api import DeviceCsr
    g = torch.Generator(device=device()).manual_seed(seed)
    w = d // lam
    u = torch.rand(n, lam, device=device(), generator=g)
    col = (u * u * w).int().clamp_(max=w - 1) + torch.arange(lam, device=device(), dtype=torch.int32) * w
    v = torch.rand(n, lam, device=device(), generator=g, dtype=dtype) + 0.05
    if signed:
        v *= torch.where(torch.rand(n, lam, device=device(), generator=g) < 0.3, -1.0, 1.0).to(dtype)
    v /= torch.linalg.vector_norm(v.double(), dim=1, keepdim=True).to(dtype)
    lens = torch.full((n,), lam, device=device(), dtype=torch.int64)
    if empty:
        lens[::7] = 0
        keep = lens > 0
        col, v = col[keep], v[keep]
    rp = torch.cat([torch.zeros(1, device=device(), dtype=torch.int64), lens.cumsum(0)])
    return DeviceCsr(rp, col.reshape(-1).contiguous(), v.reshape(-1).contiguous(), d)


@pytest.mark.parametrize("n,d,lam,k,kt,mode,dtype,signed,empty", [
    (500_003, 1_600, 100, 70, 64, "sivf", torch.float32, False, False),   # two tiles, the last of 6 centroids
    (300_001, 1_600, 80, 130, 0, "relaxed", torch.float64, False, True),  # three blocks, the last of 2; empty rows
    (150_002, 2_400, 150, 64, 0, "sivf", torch.float32, True, False),     # rows over two chunks, signed values
    (100_000, 2_400, 60, 600, 0, "ivf", torch.float32, False, False),     # ten blocks over eight parts; no filter
    (2_200_001, 1_120, 80, 12, 0, "sivf", torch.float32, False, False),   # two ranges of objects
])
def test_split_walk_equals_the_plain_walk(n, d, lam, k, kt, mode, dtype, signed, empty):
    # sliced terms x objects x centroids put the walk past the split's line; a
    # workspace cap (far above what is used) keeps it plain.  Assignments, own similarities and
    # counts are those of the plain walk, and the assignments the argmax in FP64
    log("split walk n %d d %d lam %d k %d" % (n, d, lam, k))
    X = _striped(n, d, lam, 5, dtype, signed, empty)
    ids = np.random.default_rng(7).choice(n, k, replace=False).astype(np.int32)
    opts = dict(k_tile=kt, filter_mode=mode, head_density=0.02)
    split, plain = _ctx(**opts), _ctx(workspace_cap_bytes=1 << 40, **opts)
    fs, fp = split.init_centroids(X, k, ids), plain.init_centroids(X, k, ids)
    state = [(split, fs), (plain, fp)]
    dev = device()
    a = torch.zeros(n, dtype=torch.int32, device=dev)
    own = torch.zeros(n, dtype=torch.float32, device=dev)
    own64 = torch.zeros(n, dtype=torch.float64, device=dev) if mode == "relaxed" else None
    lam_ = torch.zeros(k, dtype=torch.uint8, device=dev)
    was_split = False
    for r in (1, 2, 3, 4):
        out = []
        for ctx, f in state:
            a1, own1, l1 = a.clone(), own.clone(), lam_.clone()
            e1 = None if own64 is None else own64.clone()
            st = ctx.assign(X, f, r, a1, own1, l1, own64=e1)
            out.append((a1, own1, l1, e1, st))
        (a1, o1, l1, e1, s1), (a2, o2, l2, e2, s2) = out
        assert torch.equal(a1, a2) and torch.equal(l1, l2)
        if own64 is not None:
            assert torch.equal(e1, e2)
        for key in ("multadds", "moved", "icp_objects", "n_invariant", "relaxed_objects", "head_rows"):
            assert s1[key] == s2[key], key
        was_split |= s1["walk_bytes"] != s2["walk_bytes"]
        # own similarities: two FP32 sums of at most lam products of a unit row
        # and a unit column, each within lam * 2^-24 of the exact value, or the
        # FP64 value rounded
        assert float((o1.double() - o2.double()).abs().max()) <= 2 * (lam + 1) * 2.0 ** -24
        a, own, own64 = a1, o1, e1
        if r in (1, 4):
            c = fs.centroids()
            C = torch.zeros(k, d, dtype=torch.float64, device=dev)
            C[torch.repeat_interleave(torch.arange(k, device=dev), c.row_ptr.diff()), c.col.long()] = c.val.double()
            for lo in range(0, n, 50_000):
                hi = min(n, lo + 50_000)
                b, e = int(X.row_ptr[lo]), int(X.row_ptr[hi])
                D = torch.zeros(hi - lo, d, dtype=torch.float64, device=dev)
                rows = torch.repeat_interleave(torch.arange(hi - lo, device=dev), X.row_ptr[lo:hi + 1].diff())
                D[rows, X.col[b:e].long()] = X.val[b:e].double()
                S = D @ C.T
                mine = S.gather(1, a[lo:hi].long()[:, None])[:, 0]
                assert float((S.max(1).values - mine).max()) <= 1e-12
        lam_ = l1
        for ctx, f in state:
            ctx.update(X, a, lam_, f)
    assert was_split
    for ctx, f in state:
        f.free()
        ctx.close()


# ---------------------------------------------------------------- tile widths
@pytest.mark.parametrize("posting,k,d,widths", [
    ("fp32", 2_048, 2_000, (2_048, 2_048)),
    ("fp32", 2_049, 2_000, (1_088, 1_088)),
    ("bf16", 1_025, 400, (1_088, 1_088)),     # one tile however dense
    ("bf16", 2_048, 400, (2_048, 1_024)),     # two after the first update
    ("bf16", 3_100, 500, (1_600, 832)),       # 2 -> 4 tiles
    ("bf16", 3_100, 5_000, (1_600, 1_088)),   # 2 -> 3 tiles
])
def test_automatic_tiles_follow_the_file(posting, k, d, widths):
    # tile widths are chosen when a file is built: the trajectory is that of
    # fixed tiles of 512, whatever they are
    log("tiles %s k %d d %d" % (posting, k, d))
    n, lam = 2 * k + 3, 50
    X = _striped(n, d, lam, 3, torch.float32)
    ids = np.random.default_rng(1).choice(n, k, replace=False).astype(np.int32)
    state = []
    for kt in (0, 512):
        ctx = _ctx(posting_dtype=posting, k_tile=kt)
        f = ctx.init_centroids(X, k, ids)
        state.append([ctx, f, torch.zeros(n, dtype=torch.int32, device=device()),
                      torch.zeros(n, dtype=torch.float32, device=device()),
                      torch.zeros(k, dtype=torch.uint8, device=device())])
    for r in (1, 2, 3):
        assert state[0][1].sizes()["k_tile"] == widths[0 if r == 1 else 1]
        stats = [ctx.assign(X, f, r, a, own, lam_) for ctx, f, a, own, lam_ in state]
        (_, _, a1, _, l1), (_, _, a2, _, l2) = state
        assert torch.equal(a1, a2) and torch.equal(l1, l2)
        for key in ("multadds", "moved", "icp_objects", "n_invariant"):
            assert stats[0][key] == stats[1][key], key
        for ctx, f, a, own, lam_ in state:
            ctx.update(X, a, lam_, f)
    p1, p2 = state[0][1].export(), state[1][1].export()
    for m in p1:
        assert torch.equal(p1[m], p2[m]), m
    for ctx, f, *_ in state:
        f.free()
        ctx.close()


@pytest.mark.parametrize("n,d,k", [
    (91_003, 800, 641),    # more terms than LDS holds; 11 blocks over 8 XCDs
    (22_001, 600, 2_701),  # every term in LDS
    (235_001, 800, 250),   # four launches of rows; 4 blocks
])
def test_soft_forward_with_common_terms_in_lds(n, d, k):
    # rows of 0 .. 300 terms: no chunk, chunks filled up, several; four rows of
    # different lengths to a wave.  S is a sum of at most 300 products of unit
    # vectors' entries (302 * 2^-24), divided by tau, and exp and log add 1e-5
    from paper_2103_16141_amd.api import DeviceCsr
    log("soft forward in LDS n %d d %d k %d" % (n, d, k))
    rng = np.random.default_rng(k)
    lens = torch.from_numpy(rng.permutation(np.resize([0, 1, 15, 16, 17, 63, 64, 65, 200, 300], n))).to(device())
    g = torch.Generator(device=device()).manual_seed(k)
    cols = []
    for lo in range(0, n, 10_000):
        m = lens[lo:lo + 10_000]
        # m distinct terms of each row, early terms more often: the m smallest of weighted draws
        w = torch.rand(m.numel(), d, device=device(), generator=g) * torch.linspace(0.2, 1.0, d, device=device())
        take = torch.zeros(m.numel(), d, dtype=torch.bool, device=device())
        take.scatter_(1, w.argsort(1), torch.arange(d, device=device())[None, :] < m[:, None])
        cols.append(take.nonzero()[:, 1].int())
    col = torch.cat(cols)
    rp = torch.cat([torch.zeros(1, dtype=torch.int64, device=device()), lens.cumsum(0)])
    v = torch.rand(col.numel(), device=device(), generator=g) + 0.1
    row = torch.repeat_interleave(torch.arange(n, device=device()), lens)
    ss = torch.zeros(n, device=device(), dtype=torch.float64).index_add_(0, row, v.double() ** 2)
    v = (v / ss.sqrt()[row]).float()
    C = torch.randn(k, d, device=device(), generator=g).abs()
    C /= torch.linalg.vector_norm(C, dim=1, keepdim=True)
    X = DeviceCsr(rp, col, v, d)
    assert X.nnz * k >= 1 << 32
    ctx = _ctx()
    lse, loss = ctx.soft_assign_fwd(X, C, 0.05)
    tol = 302 * 2.0 ** -24 / 0.05 + 1e-5
    for lo in range(0, n, 10_000):
        hi = min(n, lo + 10_000)
        D = torch.zeros(hi - lo, d, dtype=torch.float64, device=device())
        b, e = int(rp[lo]), int(rp[hi])
        D[row[b:e] - lo, col[b:e].long()] = v[b:e].double()
        ref = torch.logsumexp(D @ C.double().T / 0.05, 1)
        assert float((lse[lo:hi].double() - ref).abs().max()) <= tol
    assert abs(loss + lse.double().sum().item()) <= 1e-9 * abs(loss)
    again, _ = ctx.soft_assign_fwd(X, C, 0.05)
    assert torch.equal(again, lse)
    plain, _ = _ctx(workspace_cap_bytes=1 << 40).soft_assign_fwd(X, C, 0.05)   # capped: no LDS form
    assert float((plain - lse).abs().max()) <= 2 * tol


@pytest.mark.parametrize("n,d,k,common,broken", [
    (5_101, 700, 2_201, 700, False),     # 256 of 700 dense terms; 35 column groups, the last of 25 columns
    (70_001, 50_000, 1_500, 40, False),   # 40 dense terms, three chunks of rows, the last with splits of its own
    (9_500, 3_000, 5_300, 130, True),    # 130: one past half the terms of a workgroup; a column of C is infinite
])
def test_soft_gradient_of_the_densest_terms(n, d, k, common, broken):
    # dC of the densest terms is a matrix product, the others' a sum over entries;
    # against FP64 with the tolerance of the other gradients, and against the
    # entry-by-entry form (which a workspace cap selects)
    from paper_2103_16141_amd.api import DeviceCsr
    log("densest terms n %d d %d k %d" % (n, d, k))
    dev = device()
    g = torch.Generator(device=dev).manual_seed(k)
    rows, cols = [], []
    for lo in range(0, n, 5_000):
        m = min(5_000, n - lo)
        # the common terms in 12 to 100% of the rows, the others rarely
        p = torch.full((d,), min(0.02, 20.0 / d), device=dev)
        p[:common] = torch.linspace(1.0, 0.12, common, device=dev)
        hit = (torch.rand(m, d, device=dev, generator=g) < p).nonzero()
        rows.append(hit[:, 0] + lo)
        cols.append(hit[:, 1])
    row, col = torch.cat(rows), torch.cat(cols)
    rp = torch.zeros(n + 1, dtype=torch.int64, device=dev)
    rp[1:] = torch.bincount(row, minlength=n).cumsum(0)
    v = torch.rand(col.numel(), device=dev, generator=g) + 0.1
    ss = torch.zeros(n, device=dev, dtype=torch.float64).index_add_(0, row, v.double() ** 2)
    v = (v / ss.sqrt()[row]).float()
    C = torch.rand(k, d, device=dev, generator=g)
    C /= torch.linalg.vector_norm(C, dim=1, keepdim=True)
    if broken:
        C[7, common + 5] = float("inf")
    X = DeviceCsr(rp, col.int(), v, d)
    assert X.nnz * k >= 1 << 32
    ctx = _ctx()
    lse, _ = ctx.soft_assign_fwd(X, C, 0.05)
    dC, dX = ctx.soft_assign_bwd(X, C, 0.05, lse, 0.9)
    dP, dXp = _ctx(workspace_cap_bytes=1 << 40).soft_assign_bwd(X, C, 0.05, lse, 0.9)
    assert torch.equal(torch.isnan(dC), torch.isnan(dP)) and torch.equal(torch.isnan(dX), torch.isnan(dXp))
    assert torch.equal(torch.nan_to_num(dX, nan=0.0), torch.nan_to_num(dXp, nan=0.0))
    if broken:
        assert bool(torch.isnan(dC).any()) and not bool(torch.isnan(dC).all())
        assert torch.equal(torch.nan_to_num(dC, nan=0.0), torch.nan_to_num(dP, nan=0.0))
        return
    ref = torch.zeros(k, d, dtype=torch.float64, device=dev)
    for lo in range(0, n, 2_000):
        hi = min(n, lo + 2_000)
        b, e = int(rp[lo]), int(rp[hi])
        D = torch.zeros(hi - lo, d, dtype=torch.float64, device=dev)
        D[row[b:e] - lo, col[b:e]] = v[b:e].double()
        P = torch.softmax(D @ C.double().T / 0.05, 1)
        ref += (-0.9 / 0.05) * (P.T.contiguous() @ D)
    assert bool(((dC.double() - ref).abs() <= 2e-3 * ref.abs() + 1e-7).all())
    assert torch.equal(ctx.soft_assign_bwd(X, C, 0.05, lse, 0.9)[0], dC)
