"""The split walk where its own filter and list code runs: objects with dense
and listed terms, flags chosen so that moving centroids end inside a tile and
inside a block of 64 slots, several tiles and ranges."""
import numpy as np
import pytest
import torch

from tests.gpu_util import device, log

pytestmark = pytest.mark.gpu

DENSE, RARE, WIDTH = 100, 200, 1_000   # stripes of 4 common terms, of 1,000 rare ones
D = 4 * DENSE + RARE * WIDTH


def _objects(n, dtype, signed, seed):
    """Unit rows: one term of each of 100 stripes of 4, and of the first m of 200
    stripes of 1,000, m from 0 to 200; every 501st row empty.  The common terms'
    ids lie in the middle."""
    from paper_2103_16141_amd.api import DeviceCsr
    g = torch.Generator(device=device()).manual_seed(seed)
    half = RARE // 2
    rare = torch.randint(WIDTH, (n, RARE), device=device(), generator=g, dtype=torch.int32)
    rare += torch.arange(RARE, device=device(), dtype=torch.int32) * WIDTH
    rare[:, half:] += 4 * DENSE
    dense = torch.randint(4, (n, DENSE), device=device(), generator=g, dtype=torch.int32)
    dense += torch.arange(DENSE, device=device(), dtype=torch.int32) * 4 + half * WIDTH
    m = torch.tensor([0, 1, 27, 28, 29, 64, 92, 127, 128, 129, 160, 200], device=device())
    m = m[torch.randint(m.numel(), (n,), device=device(), generator=g)]
    keep = torch.arange(RARE, device=device())[None, :] < m[:, None]
    col = torch.cat([rare[:, :half], dense, rare[:, half:]], 1)
    keep = torch.cat([keep[:, :half], torch.ones_like(dense, dtype=torch.bool), keep[:, half:]], 1)
    keep[::501] = False
    lens = keep.sum(1)
    v = torch.rand(n, DENSE + RARE, device=device(), generator=g, dtype=torch.float64) + 0.05
    if signed:
        v *= torch.where(torch.rand(n, DENSE + RARE, device=device(), generator=g) < 0.3, -1.0, 1.0)
    v *= keep
    v /= torch.linalg.vector_norm(v, dim=1, keepdim=True).clamp_(min=1e-30)
    rp = torch.cat([torch.zeros(1, dtype=torch.int64, device=device()), lens.cumsum(0)])
    return DeviceCsr(rp, col[keep].contiguous(), v[keep].to(dtype).contiguous(), D)


@pytest.mark.parametrize("n,k,kt,mode,dtype,signed,moving,ranges", [
    (60_003, 1_100, 640, "sivf", torch.float32, False, (700, 333, 1_037), 1),   # into tile 1, short of it, nearly all
    (60_003, 1_100, 640, "relaxed", torch.float64, False, (450, 641), 1),
    (40_001, 1_500, 0, "sivf", torch.float32, True, (1_001, 70), 1),            # one tile, signed values
    (300_007, 4_200, 4_096, "sivf", torch.float32, False, (2_000, 4_130), 2),   # two tiles of two ranges of objects
    (270_001, 4_200, 4_096, "relaxed", torch.float32, True, (3_333,), 2),
])
def test_split_walk_of_objects_with_listed_terms_under_the_filter(n, k, kt, mode, dtype, signed, moving, ranges):
    from paper_2103_16141_amd.api import Context
    log("split walk with lists n %d k %d %s" % (n, k, mode))
    dev = device()
    X = _objects(n, dtype, signed, n)
    rng = np.random.default_rng(k)
    ids = (rng.choice(n - 1, k, replace=False) + 1).astype(np.int32)
    ids[ids % 501 == 0] = 1    # no empty seed (ids may repeat)
    opts = dict(k_tile=kt, filter_mode=mode)
    split, plain = Context(0, **opts), Context(0, workspace_cap_bytes=1 << 40, **opts)
    state = [(split, split.init_centroids(X, k, ids)), (plain, plain.init_centroids(X, k, ids))]
    a = torch.zeros(n, dtype=torch.int32, device=dev)
    own = torch.zeros(n, dtype=torch.float32, device=dev)
    own64 = torch.zeros(n, dtype=torch.float64, device=dev) if mode == "relaxed" else None
    lam = torch.zeros(k, dtype=torch.uint8, device=dev)
    plain.assign(X, state[1][1], 1, a, own, lam, own64=own64)
    for r, mv in enumerate(moving, 2):
        # any clusters may be kept: flagged ones keep their centroids bitwise, so
        # the filter's premise holds and the argmax stays the exact one
        flags = np.ones(k, np.uint8)
        flags[rng.choice(k, mv, replace=False)] = 0
        flags = torch.from_numpy(flags).to(dev)
        out = []
        for ctx, f in state:
            ctx.update(X, a, flags, f)
            a1, own1, l1 = a.clone(), own.clone(), lam.clone()
            e1 = None if own64 is None else own64.clone()
            out.append((a1, own1, l1, e1, ctx.assign(X, f, r, a1, own1, l1, own64=e1)))
        (a1, o1, l1, e1, s1), (a2, o2, l2, e2, s2) = out
        tiles = state[0][1].sizes()["n_tiles"]
        assert s1["walk_bytes"] != s2["walk_bytes"] and s1["walk_launches"] == tiles * ranges   # split
        assert s2["walk_launches"] == tiles
        assert torch.equal(a1, a2) and torch.equal(l1, l2)
        for key in ("multadds", "moved", "icp_objects", "n_invariant", "relaxed_objects", "head_rows"):
            assert s1[key] == s2[key], key
        assert 0 < s1["icp_objects"] < n and (mode != "relaxed" or s1["relaxed_objects"] > 0)
        if own64 is not None:
            assert torch.equal(e1, e2)
        # two FP32 sums of at most 300 products of a unit row and a unit column,
        # each within 302 * 2^-24 of the exact value, or the FP64 value rounded
        assert float((o1.double() - o2.double()).abs().max()) <= 2 * 302 * 2.0 ** -24
        # the assignment is the argmax in FP64, on rows at the ends of the ranges and between
        c = state[0][1].centroids()
        C = torch.zeros(k, D, dtype=torch.float64, device=dev)
        C[torch.repeat_interleave(torch.arange(k, device=dev), c.row_ptr.diff()), c.col.long()] = c.val
        step = (n + ranges - 1) // ranges
        pick = {0, 1, 500, 501, 502, n - 1, n // 2, (1 << 30) // 4_096, (1 << 30) // 4_096 - 1, step, step - 1}
        pick |= set(rng.choice(n, 1_500).tolist())
        pick = torch.tensor(sorted(p for p in pick if p < n), device=dev)
        rows = torch.zeros(pick.numel(), D, dtype=torch.float64, device=dev)
        for q, i in enumerate(pick.tolist()):
            b, e = int(X.row_ptr[i]), int(X.row_ptr[i + 1])
            rows[q, X.col[b:e].long()] = X.val[b:e].double()
        S = rows @ C.T
        mine = S.gather(1, a1[pick].long()[:, None])[:, 0]
        assert float((S.max(1).values - mine).max()) <= 1e-12
        del C, S, rows
        a, own, own64, lam = a1, o1, e1, l1
    for ctx, f in state:
        f.free()
        ctx.close()
    torch.cuda.empty_cache()


@pytest.mark.parametrize("mode", ["sivf", "relaxed"])
def test_noalloc_assign_where_assign_splits_the_walk(mode):
    # the call that allocates nothing never splits: the same assignments, flags,
    # exact similarities and mult-adds, own similarities within the bound of both
    from paper_2103_16141_amd.api import Context
    log("no-alloc assign against a split walk, %s" % mode)
    n, k, dev = 60_003, 1_100, device()
    X = _objects(n, torch.float32, False, 9)
    rng = np.random.default_rng(9)
    ids = (rng.choice(n - 1, k, replace=False) + 1).astype(np.int32)
    ids[ids % 501 == 0] = 1
    ctx = Context(0, filter_mode=mode)
    na = Context(0, filter_mode=mode, workspace_cap_bytes=1)
    f = ctx.init_centroids(X, k, ids)
    a = torch.zeros(n, dtype=torch.int32, device=dev)
    own = torch.zeros(n, dtype=torch.float32, device=dev)
    own64 = torch.zeros(n, dtype=torch.float64, device=dev) if mode == "relaxed" else None
    lam = torch.zeros(k, dtype=torch.uint8, device=dev)
    ctx.assign(X, f, 1, a, own, lam, own64=own64)
    flags = torch.from_numpy((rng.random(k) < 0.4).astype(np.uint8)).to(dev)
    ctx.update(X, a, flags, f)
    out = []
    for call in (ctx.assign, na.assign_noalloc):
        a1, o1, l1, e1 = a.clone(), own.clone(), lam.clone(), None if own64 is None else own64.clone()
        out.append((a1, o1, l1, e1, call(X, f, 2, a1, o1, l1, own64=e1)))
    (a1, o1, l1, e1, s1), (a2, o2, l2, e2, s2) = out
    assert s1["walk_bytes"] != s2["walk_bytes"]   # split there, plain here
    assert torch.equal(a1, a2) and torch.equal(l1, l2) and (e1 is None or torch.equal(e1, e2))
    for key in ("multadds", "moved", "icp_objects", "n_invariant", "relaxed_objects"):
        assert s1[key] == s2[key], key
    assert float((o1.double() - o2.double()).abs().max()) <= 2 * 302 * 2.0 ** -24


@pytest.mark.parametrize("posting", ["fp32", "bf16"])
@pytest.mark.parametrize("mode", ["sivf", "cbicp"])
def test_assignment_in_several_pieces_of_objects_a_wave(posting, mode):
    # up to 16 or 24 objects a wave (5,120 or 6,144 waves) are taken in two or
    # three pieces of at most 8: every batch gives what its objects give in batches of at
    # most 8 a wave, with and without the filter
    from paper_2103_16141_amd.api import Context, DeviceCsr
    import oracle
    import synth
    log("pieces %s %s" % (posting, mode))
    n, d, dev = 150_000, 700, device()
    c = synth.make_corpus(n, d, 8, 1.1, np.float32, seed=77)
    X = DeviceCsr.from_corpus(c, dev)
    for k in (9, 300):
        ctx = Context(0, posting_dtype=posting, filter_mode=mode)
        ids = synth.init_ids(n, k, 3)
        f = ctx.init_centroids(X, k, ids)
        a = torch.zeros(n, dtype=torch.int32, device=dev)
        own = torch.zeros(n, dtype=torch.float32, device=dev)
        lam = torch.zeros(k, dtype=torch.uint8, device=dev)
        ctx.assign(X, f, 1, a, own, lam)
        ref, _, _ = oracle.assign(c, oracle.init_centroids(c, ids), rows=np.arange(0, n, 191))
        assert np.array_equal(a.cpu().numpy()[::191], ref)
        flags = torch.zeros(k, dtype=torch.uint8, device=dev)
        flags[k // 2:] = 1
        ctx.update(X, a, flags, f)

        def run(lo, hi, it):
            b, e = int(c.row_ptr[lo]), int(c.row_ptr[hi])
            rows = DeviceCsr(X.row_ptr[lo:hi + 1] - b, X.col[b:e].clone(), X.val[b:e].clone(), d)
            pa, po = a[lo:hi].clone(), own[lo:hi].clone()
            st = ctx.assign(rows, f, it, pa, po, lam.clone())
            return pa, po, st["multadds"], st["icp_objects"]

        for it in (1, 2):
            small = [run(lo, min(n, lo + 37_000), it) for lo in range(0, n, 37_000)]
            want_a, want_o = torch.cat([s[0] for s in small]), torch.cat([s[1] for s in small])
            for hi in (40_961, 49_153, 81_920, 81_921, 98_304, 98_305, 122_880, 122_881, 147_456, 147_457, n):
                pa, po, m, icp = run(0, hi, it)
                assert torch.equal(pa, want_a[:hi]) and torch.equal(po, want_o[:hi]), hi
                if hi == n:
                    assert m == sum(s[2] for s in small) and icp == sum(s[3] for s in small) and (icp > 0) == (it == 2)
        f.free()
        ctx.close()


@pytest.mark.parametrize("n", [40_960, 40_961, 81_920, 81_921, 122_880, 122_881])
def test_split_lists_in_several_pieces_of_objects_a_wave(n):
    # one tile of 512: equal shares up to 24 objects a wave, then grabs
    from paper_2103_16141_amd.api import Context
    log("pieces of a split walk, n %d" % n)
    k, dev = 512, device()
    X = _objects(n, torch.float32, False, 3)
    split, plain = Context(0), Context(0, workspace_cap_bytes=1 << 40)
    ids = np.arange(1, k + 1, dtype=np.int32)
    ids[500] = 600   # row 501 is empty
    out = []
    a = torch.zeros(n, dtype=torch.int32, device=dev)
    own = torch.zeros(n, dtype=torch.float32, device=dev)
    lam = torch.zeros(k, dtype=torch.uint8, device=dev)
    for ctx in (split, plain):
        f = ctx.init_centroids(X, k, ids)
        ctx.assign(X, f, 1, a, own, lam)
        flags = torch.zeros(k, dtype=torch.uint8, device=dev)
        flags[::3] = 1
        ctx.update(X, a, flags, f)
        for it in (1, 2):
            a1, o1, l1 = a.clone(), own.clone(), lam.clone()
            out.append((a1, o1, l1, ctx.assign(X, f, it, a1, o1, l1)))
        f.free()
    for (a1, o1, l1, s1), (a2, o2, l2, s2) in zip(out[:2], out[2:]):
        assert s1["walk_bytes"] != s2["walk_bytes"]
        assert torch.equal(a1, a2) and torch.equal(l1, l2) and s1["multadds"] == s2["multadds"]
        assert s1["icp_objects"] == s2["icp_objects"]
        assert float((o1.double() - o2.double()).abs().max()) <= 2 * 302 * 2.0 ** -24


def test_tiles_of_a_capped_file_narrow_once_it_has_many_dense_rows():
    # a workspace cap keeps the walk plain; 650 dense rows and more are then read in tiles
    # of 1,024 from the second update on, and every step is that of fixed tiles
    from tests.test_gpu_kernel_edges import _striped
    from paper_2103_16141_amd.api import Context
    log("capped tiles")
    n, d, lam, k, dev = 8_195, 2_800, 700, 2_048, device()
    X = _striped(n, d, lam, 4, torch.float32)
    ids = np.random.default_rng(2).choice(n, k, replace=False).astype(np.int32)
    state = []
    for kt, cap in ((0, 1 << 40), (512, 1 << 40), (0, 0)):
        ctx = Context(0, k_tile=kt, workspace_cap_bytes=cap, head_density=0.5)
        state.append([ctx, ctx.init_centroids(X, k, ids), torch.zeros(n, dtype=torch.int32, device=dev),
                      torch.zeros(n, dtype=torch.float32, device=dev), torch.zeros(k, dtype=torch.uint8, device=dev)])
    widths = []
    for r in (1, 2, 3, 4):
        widths.append([f.sizes()["k_tile"] for _, f, *_ in state])
        st = [ctx.assign(X, f, r, a, own, l) for ctx, f, a, own, l in state]
        for (_, _, a, _, l), s in zip(state[1:], st[1:]):
            assert torch.equal(a, state[0][2]) and torch.equal(l, state[0][4])
            assert all(s[q] == st[0][q] for q in ("multadds", "moved", "icp_objects", "n_invariant", "head_rows"))
        for ctx, f, a, own, l in state:
            ctx.update(X, a, l, f)
    assert st[0]["head_rows"] >= 650
    assert widths == [[2048, 512, 2048], [2048, 512, 2048], [1024, 512, 2048], [1024, 512, 2048]]
    # the file made without a cap narrows when a capped ctx updates it
    ctx, f, a, own, l = state[2]
    state[0][0].update(X, a, l, f)
    assert f.sizes()["k_tile"] == 1024
    for ctx, f, *_ in state:
        f.free()


@pytest.mark.parametrize("k,lam,wide,narrow,rows_from,options", [
    (2_100, 1_500, 1_088, 704, 2_600, dict(posting_dtype="bf16")),
    (2_048, 30, 2_048, 1_024, 650, dict(head_density=0.02)),   # rows too short for the split walk
    (4_000, 30, 2_048, 1_024, 480, dict(head_density=0.01, filter_mode="cbicp")),
])
def test_tiles_narrow_once_many_dense_rows_are_walked_as_they_are(k, lam, wide, narrow, rows_from, options):
    # every step is that of fixed tiles
    from tests.test_gpu_kernel_edges import _striped
    from paper_2103_16141_amd.api import Context
    log("tiles k %d %s" % (k, options))
    n, d, dev = 4 * k + 3, 4_000, device()
    X = _striped(n, d, lam, 5, torch.float32)
    ids = np.random.default_rng(3).choice(n, k, replace=False).astype(np.int32)
    state = []
    for kt in (0, 512):
        ctx = Context(0, k_tile=kt, **options)
        state.append([ctx, ctx.init_centroids(X, k, ids), torch.zeros(n, dtype=torch.int32, device=dev),
                      torch.zeros(n, dtype=torch.float32, device=dev), torch.zeros(k, dtype=torch.uint8, device=dev)])
    widths, rows = [], []
    for r in (1, 2, 3, 4):
        widths.append(state[0][1].sizes()["k_tile"])
        st = [ctx.assign(X, f, r, a, own, l) for ctx, f, a, own, l in state]
        rows.append(st[0]["head_rows"])
        assert torch.equal(state[0][2], state[1][2]) and torch.equal(state[0][4], state[1][4])
        assert all(st[0][q] == st[1][q] for q in ("multadds", "moved", "icp_objects", "n_invariant", "head_rows"))
        for ctx, f, a, own, l in state:
            ctx.update(X, a, l, f)
    # a file narrows at the update after the one that made the rows
    assert widths == [narrow if r and rows[r - 1] >= rows_from else wide for r in range(4)]
    assert wide in widths and narrow in widths
    for ctx, f, *_ in state:
        f.free()
        ctx.close()
