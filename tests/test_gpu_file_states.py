"""A file of centroids through other contexts than the one it was made in, and
after calls on it that failed."""
import numpy as np
import pytest
import torch

import synth
from tests.gpu_util import device, log

pytestmark = pytest.mark.gpu


def _ctx(**kw):
    from paper_2103_16141_amd.api import Context
    return Context(0, **kw)


def _X(c):
    from paper_2103_16141_amd.api import DeviceCsr
    return DeviceCsr.from_corpus(c, device())


def _state(n, k):
    return (torch.zeros(n, dtype=torch.int32, device=device()), torch.zeros(n, dtype=torch.float32, device=device()),
            torch.zeros(k, dtype=torch.uint8, device=device()))


def _same_export(f, g):
    p, q = f.export(), g.export()
    for m in p:
        assert torch.equal(p[m], q[m]), m


@pytest.mark.parametrize("made,other", [
    (dict(), dict(k_tile=64)),
    (dict(), dict(posting_dtype="bf16")),
    (dict(posting_dtype="bf16"), dict(posting_dtype="bf16", k_tile=64)),
    (dict(posting_dtype="bf16"), dict()),
    (dict(k_tile=512), dict(k_tile=64, head_density=0.9)),
])
def test_a_file_keeps_its_tiling_when_another_context_updates_it(made, other):
    # tiles follow from the options the file was made with, whoever updates it:
    # every step is that of a file that stays in its own context
    log("file of %s updated by %s" % (made, other))
    k, d = 3_100, 400
    c = synth.make_corpus(2 * k + 3, d, 40, 1.0, np.float32, seed=11)
    X, ids = _X(c), synth.init_ids(c.n, k, 12)
    home, guest = _ctx(**made), _ctx(**other)
    f, g = home.init_centroids(X, k, ids), home.init_centroids(X, k, ids)
    (a, own, lam), (a2, own2, lam2) = _state(c.n, k), _state(c.n, k)
    for r in (1, 2, 3):
        home.assign(X, f, r, a, own, lam)
        home.assign(X, g, r, a2, own2, lam2)
        assert torch.equal(a, a2) and torch.equal(own, own2) and torch.equal(lam, lam2)
        home.update(X, a, lam, f)
        guest.update(X, a2, lam2, g)
        assert f.sizes() == g.sizes()
        _same_export(f, g)
    f.free()
    g.free()


@pytest.mark.parametrize("posting", ["fp32", "bf16"])
def test_a_file_whose_update_ran_out_of_memory_is_refused_until_updated(posting):
    # caps from too small for the first buffer to enough for the whole update:
    # whatever request fails, the file is either as it was or refused, and the
    # same update with enough memory gives what it would have given
    from paper_2103_16141_amd._native import SivfError
    log("failed updates, %s" % posting)
    k, d = 2_000, 900
    c = synth.make_corpus(9_001, d, 60, 1.0, np.float32, seed=21)
    X, ids = _X(c), synth.init_ids(c.n, k, 22)
    home = _ctx(posting_dtype=posting)
    (a, own, lam), (a2, own2, lam2) = _state(c.n, k), _state(c.n, k)
    want = home.init_centroids(X, k, ids)
    home.assign(X, want, 1, a, own, lam)
    home.update(X, a, lam, want)
    refused = kept = 0
    done = False
    for cap in (int(2.0 ** (e / 16)) for e in range(368, 500)):
        f = home.init_centroids(X, k, ids)
        guest = _ctx(posting_dtype=posting, workspace_cap_bytes=cap)
        try:
            guest.update(X, a, lam, f)
            done = True
        except SivfError as e:
            assert e.name == "SIVF_E_NOMEM"
            try:
                home.assign(X, f, 1, a2, own2, lam2)
                kept += 1
                assert torch.equal(a2, a) and torch.equal(own2, own)
            except SivfError as e:
                refused += 1
                assert e.name == "SIVF_E_INVALID"
                with pytest.raises(SivfError):
                    f.export()
            home.update(X, a, lam, f)
        _same_export(f, want)
        home.assign(X, f, 1, a2, own2, lam2)
        f.free()
        guest.close()
        if done:
            break
    assert done and refused and kept


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("rows", [1, 64, 200])
def test_no_nonzero_past_the_last_row_bound_is_read(dtype, rows):
    # a matrix whose stated number of nonzeros is far more than its row bounds
    # (and its arrays) hold is refused without a look past them
    import ctypes
    from paper_2103_16141_amd import _native as N
    log("stated nonzeros, %d rows" % rows)
    c = synth.make_corpus(rows, 50, 5, 1.0, dtype, seed=rows)
    X = _X(c)
    ctx = _ctx()
    for stated in (c.nnz + 1, 1 << 33, 1 << 40):
        s = X.struct()
        s.nnz = stated
        assert N.load().sivf_validate_csr(ctx.handle, ctypes.byref(s)) == -3
        assert b"row_ptr[n] != nnz" in N.load().sivf_last_error(ctx.handle)
    s = X.struct()
    s.nnz = c.nnz - 1
    assert N.load().sivf_validate_csr(ctx.handle, ctypes.byref(s)) == -3
    ctx.validate(X)


def test_buffers_of_faster_forms_leave_room_for_what_calls_need():
    # 2,100,000 of 2,200,001 objects at a time, 512 slots each: the split walk
    # asks for about 7 GB.  With 10 GB free that is more than half: the walk is
    # not split, and nothing is said.  Held from an earlier call, they are given
    # back when a call that needs 3.4 GB finds 2.5 GB free
    from paper_2103_16141_amd import _native as N
    from paper_2103_16141_amd.api import DeviceCsr
    from tests.test_gpu_kernel_edges import _striped
    log("optional buffers on a full device")
    n, d, lam, k = 2_200_001, 1_120, 80, 12
    X = _striped(n, d, lam, 5, torch.float32)
    ids = np.arange(k, dtype=np.int32) * 1_000
    wide = 12_000_000   # columns of a matrix of two rows: 64 of them are 3.1 GB
    rp = torch.tensor([0, 2, 3], device=device())
    col = torch.tensor([5, wide - 1, 7], dtype=torch.int32, device=device())
    Y = DeviceCsr(rp, col, torch.tensor([0.6, 0.8, 1.0], device=device()), wide)
    C = torch.zeros(1, wide, device=device())
    C[0, 5], C[0, 7], C[0, wide - 1] = 1.0, 0.25, 0.5

    def step(ctx):
        f = ctx.init_centroids(X, k, ids)
        a, own, l = _state(n, k)
        ctx.assign(X, f, 1, a, own, l)
        ctx.update(X, a, l, f)
        st = ctx.assign(X, f, 1, a, own, l)   # (iter 1: no state needed)
        return f, a, st

    def fill(left):
        torch.cuda.empty_cache()
        free, _ = torch.cuda.mem_get_info()
        return torch.empty(free - left, dtype=torch.uint8, device=device())

    holder, plain, late = _ctx(head_density=0.02), _ctx(head_density=0.02, workspace_cap_bytes=1 << 40), \
        _ctx(head_density=0.02)
    f0, a0, s0 = step(holder)
    f1, a1, s1 = step(plain)
    assert torch.equal(a0, a1) and s0["walk_bytes"] != s1["walk_bytes"]
    plain.soft_assign_fwd(Y, C, 0.05)   # its kernels are loaded
    plain.close()
    hog = fill(10 << 30)
    f2, a2, s2 = step(late)
    assert torch.equal(a2, a0) and s2["walk_bytes"] == s1["walk_bytes"]
    assert N.load().sivf_last_error(late.handle) == b""
    late.close()
    del hog
    hog = fill(5 << 29)
    lse, _ = holder.soft_assign_fwd(Y, C, 0.05)
    # one centroid: the log of the sum is its similarity / tau (two products and one sum in FP32)
    assert float((lse.double() * 0.05 - torch.tensor([1.0, 0.25], device=device())).abs().max()) < 4 * 2.0 ** -24
    del hog
    torch.cuda.empty_cache()
    a, own, l = _state(n, k)
    assert holder.assign(X, f0, 1, a, own, l)["walk_bytes"] == s0["walk_bytes"] and torch.equal(a, a0)


@pytest.mark.parametrize("posting", ["fp32", "bf16"])
def test_more_dense_rows_than_a_launch_has_workgroups(posting):
    # one centroid with 2^24 + 1,000 terms: each has a dense row of 512 slots
    # (17 or 34 GB), more workgroups of 256 threads than 32 bits count threads
    from paper_2103_16141_amd.api import DeviceCsr
    log("dense rows of a wide centroid, %s" % posting)
    d = (1 << 24) + 1_000
    dev = device()
    ctx = _ctx(posting_dtype=posting)
    col = torch.arange(d, dtype=torch.int32, device=dev)
    val = ((col % 251).double() + 1.0) / 256.0     # exact in BF16
    f = ctx.build_centroid_ivf(torch.tensor([0, d], device=dev), col, val, d)
    # rows of one term on both sides of 2^24 and at the ends, of value 1
    terms = torch.tensor([0, 1, (1 << 24) - 2, (1 << 24) - 1, 1 << 24, (1 << 24) + 1, d - 1], device=dev)
    X = DeviceCsr(torch.arange(8, device=dev), terms.int(), torch.ones(7, device=dev), d)
    a, own, lam = _state(7, 1)
    st = ctx.assign(X, f, 1, a, own, lam)
    assert st["head_rows"] == d and bool((a == 0).all())
    assert torch.equal(own.double(), val[terms])
    f.free()
    ctx.close()
    torch.cuda.empty_cache()


@pytest.mark.parametrize("lens", [[1], [0, 0, 1], [2, 0, 3, 1], [15, 17, 0, 16, 18], [0] * 40 + [700] + [1] * 30],
                         ids=["ones", "mostly empty", "short", "about sixteen a piece", "a long one among short"])
def test_files_of_many_short_centroids(lens):
    # a piece of entries with 16 centroids and more is taken an entry per lane
    import oracle
    log("short centroids %s" % lens[:6])
    k, d = 3_001, 800
    rng = np.random.default_rng(len(lens))
    m = np.resize(lens, k)
    ptr = np.concatenate([[0], np.cumsum(m)]).astype(np.int64)
    col = np.concatenate([np.sort(rng.choice(d, q, replace=False)) for q in m] + [np.zeros(0)]).astype(np.int32)
    val = rng.standard_normal(len(col))
    lam = (rng.random(k) < 0.5).astype(np.uint8)
    f = _ctx().build_centroid_ivf(*[torch.from_numpy(x).to(device()) for x in (ptr, col, val)], d,
                                  torch.from_numpy(lam).to(device()))
    ex = {q: t.cpu().numpy() for q, t in f.export().items()}
    ref = oracle.build_ivf(oracle.Centroids(k, d, ptr, col, val), lam)
    assert np.array_equal(ex["c_ptr"], ptr) and np.array_equal(ex["c_col"], col) and np.array_equal(ex["c_val"], val)
    assert np.array_equal(ex["term_ptr"], ref.term_ptr) and np.array_equal(ex["split"], ref.split)
    assert np.array_equal(ex["p_cid"], ref.cid) and np.array_equal(ex["p_val"], ref.val)


@pytest.mark.parametrize("n,per", [
    (16_384, 1), (16_385, 1),       # rows: the last size of small workgroups, the first of large ones
    (64, 1_024), (5, 13_108),       # nonzeros: 65,536 and 65,540
    (1, 4), (700_000, 1),           # a thread; more rows than the groups have threads
])
def test_validation_errors_at_the_ends_of_its_workgroups(n, per):
    from paper_2103_16141_amd._native import SivfError
    from paper_2103_16141_amd.api import DeviceCsr
    log("validation n %d per %d" % (n, per))
    ctx, dev, nnz = _ctx(), device(), n * per
    rp = torch.arange(n + 1, device=dev) * per
    col = torch.arange(per, dtype=torch.int32, device=dev).repeat(n)
    val = torch.full((nnz,), per ** -0.5, device=dev)
    ctx.validate(DeviceCsr(rp, col, val, per))
    for at in sorted({0, min(1_023, nnz - 1), min(1_024, nnz - 1), min(4_096, nnz - 1), nnz - 1}):
        for kind, arr, v in (("RANGE", col, per), ("NONFINITE", val, float("inf"))):
            bad = arr.clone()
            bad[at] = v
            X = DeviceCsr(rp, bad if arr is col else col, bad if arr is val else val, per)
            with pytest.raises(SivfError) as err:
                ctx.validate(X)
            if kind == "RANGE" and at % per < per - 1:
                kind = "UNSORTED"   # above its right neighbour too, which is what is reported
            assert err.value.name == "SIVF_E_" + kind and "row %d " % (at // per) in str(err.value)
    if per > 1:   # equal columns in the last row
        bad = col.clone()
        bad[-1] = bad[-2]
        with pytest.raises(SivfError) as err:
            ctx.validate(DeviceCsr(rp, bad, val, per))
        assert err.value.name == "SIVF_E_UNSORTED" and "row %d " % (n - 1) in str(err.value)


@pytest.mark.parametrize("d,long,dtype,signed", [
    (8_192, 900, np.float32, False),     # the widest vocabulary summed member by member
    (8_193, 900, np.float32, False),     # the next is not
    (700, 700, np.float64, True),
    (250, 250, np.float32, True),
])
def test_update_of_clusters_summed_member_by_member(d, long, dtype, signed):
    # clusters of more than a tile (4,096 nonzeros) and of at most twice the mean of
    # members: one of exactly as many and one of one more; rows of no, few, 256, 257
    # and many terms; twice, so that the sums are used again
    import oracle
    from tests.gpu_util import assert_centroids_equal, centroids_from_export
    from tests.test_gpu_kernel_edges import _rows_corpus
    log("member by member d %d" % d)
    rng = np.random.default_rng(d)
    row = min(d, 250)
    n, k = 5_500_000 // row, 900
    lens = np.full(n, row)
    for m in (0, 3, 256, 257, long):
        lens[rng.integers(0, n, 100)] = min(d, m)
    c = _rows_corpus([int(x) for x in lens], d, dtype, 3, signed)
    most = 2 * n // k
    assert c.nnz // 100_000 >= most and c.nnz > 4_096 * k and most * row < 4 * 4_096
    tile = 4_096 // row
    sizes = [most, most + 1, most - 1, tile, tile + 1, tile + 2, 1, 0, 2 * most]
    sizes += [(n - sum(sizes) - 40 * most) // (k - 50)] * (k - 50) + [most] * 40
    a = np.repeat(np.arange(k), sizes + [n - sum(sizes)]).astype(np.int32)
    rng.shuffle(a)
    X, ids = _X(c), [int(i) for i in rng.choice(n, k, replace=False)]
    ctx = _ctx()
    ivf = ctx.init_centroids(X, k, ids)
    ref = oracle.init_centroids(c, np.array(ids, np.int32))
    lam = torch.zeros(k, dtype=torch.uint8, device=device())
    for step in range(2):
        ctx.update(X, torch.from_numpy(a).to(device()), lam, ivf)
        ref, _ = oracle.update(c, a, ref)
        assert_centroids_equal(centroids_from_export(ivf.export(), k, d), ref, "d %d, step %d" % (d, step))
        a = np.roll(a, 1)
    ivf.free()
    ctx.close()


@pytest.mark.parametrize("terms", [1, 3, 4, 8_191, 8_192, 8_193, 16_385, 20_000])
def test_exact_similarity_to_centroids_of_many_terms(terms):
    # the search for an object's terms among a centroid's: by quarters, from 8,192
    # terms on by halves; objects of the centroid's first and last terms, of terms
    # between and beside them, and of all kinds; the FP64 fold in ascending order
    from paper_2103_16141_amd.api import DeviceCsr
    log("exact similarity, %d terms" % terms)
    d = 20_000
    rng = np.random.default_rng(terms)
    have = np.sort(rng.choice(d, terms, replace=False)).astype(np.int32)
    lack = np.setdiff1d(np.arange(d, dtype=np.int32), have)
    u = rng.random(terms) + 0.1
    u /= np.sqrt((u * u).sum())
    rows = [have[:40], have[-40:], np.concatenate([have[:1], have[-1:]]), lack[:50], lack[-50:]]
    rows += [np.unique(rng.choice(d, 150)) for _ in range(200)]
    rows += [np.unique(np.concatenate([rng.choice(have, min(terms, 60)), rng.choice(d, 20)])) for _ in range(200)]
    rows = [np.unique(r).astype(np.int32) for r in rows if len(r)]
    vals = [(rng.random(len(r)) + 0.1).astype(np.float32) for r in rows]
    vals = [(v / np.sqrt((v.astype(np.float64) ** 2).sum())).astype(np.float32) for v in vals]
    rp = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int64)
    X = DeviceCsr.from_numpy(rp, np.concatenate(rows), np.concatenate(vals), d)
    C = DeviceCsr.from_numpy(np.array([0, terms, 2 * terms], np.int64), np.concatenate([have, have]),
                             np.concatenate([u, u]), d)
    dense = np.zeros(d)
    dense[have] = u
    in_c = np.zeros(d, bool)
    in_c[have] = True
    want = []
    for r, v in zip(rows, vals):
        acc = 0.0
        for t, x in zip(r, v):
            if in_c[t]:
                acc = acc + float(x) * dense[t]
        want.append(acc)
    ctx = _ctx()
    a = torch.zeros(len(rows), dtype=torch.int32, device=device())
    f, own, _ = ctx.resume(X, C, a, a)
    assert np.array_equal(own.cpu().numpy(), np.array(want).astype(np.float32))
    f.free()
    ctx.close()
