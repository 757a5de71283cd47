"""The soft form under workspace caps: long and skewed rows, column groups and
chunk copies against the form that has all the memory it asks for."""
import numpy as np
import pytest
import torch

from tests.gpu_util import device, log
from tests.test_gpu_kernel_edges import test_soft_gradient_of_the_densest_terms as _dense_terms

pytestmark = pytest.mark.gpu


def _ctx(**kw):
    from paper_2103_16141_amd.api import Context
    return Context(0, **kw)


def _corpus(n, d, short, long, every, seed):
    """n unit rows of `short` distinct terms, every `every`-th one of `long`."""
    from paper_2103_16141_amd.api import DeviceCsr
    g = torch.Generator(device=device()).manual_seed(seed)
    cols, lens = [], []
    for lo in range(0, n, 5_000):
        m = torch.full((min(5_000, n - lo),), short, device=device())
        m[(torch.arange(lo, lo + m.numel(), device=device()) % every) == 0] = long
        w = torch.rand(m.numel(), d, device=device(), generator=g) * torch.linspace(0.3, 1.0, d, device=device())
        take = torch.zeros(m.numel(), d, dtype=torch.bool, device=device())
        take.scatter_(1, w.argsort(1), torch.arange(d, device=device())[None, :] < m[:, None])
        cols.append(take.nonzero()[:, 1].int())
        lens.append(m)
    lens, col = torch.cat(lens), torch.cat(cols)
    rp = torch.cat([torch.zeros(1, dtype=torch.int64, device=device()), lens.cumsum(0)])
    v = torch.rand(col.numel(), device=device(), generator=g) + 0.1
    row = torch.repeat_interleave(torch.arange(n, device=device()), lens)
    ss = torch.zeros(n, device=device(), dtype=torch.float64).index_add_(0, row, v.double() ** 2)
    return DeviceCsr(rp, col, (v / ss.sqrt()[row]).float(), d), row


def _needed(X, k):
    """Bytes that are always enough for k >= 64, by the array: C^T and dC^T, dS of
    2^26 / k rows, 32 B per nonzero of such a chunk, row and value per nonzero,
    counts per 1,024 rows, 88 B per term; each an eighth more."""
    n, d, nnz = X.n_rows, X.n_cols, X.nnz
    rc = min(n, (64 << 20) // k)
    rp = X.row_ptr.cpu().numpy()
    most = max(int(rp[min(n, c + rc)] - rp[c]) for c in range(0, n, rc))
    return 9 * (8 * k * d + 4 * rc * k + 32 * most + 8 * nnz + 4 * ((n + 1023) // 1024) * d + 88 * d) // 8 + (1 << 16)


@pytest.mark.parametrize("n,d,short,long,every,k", [
    (30_000, 2_000, 20, 1_500, 100, 1_000),    # two chunks of rows, a few rows hold most nonzeros
    (6_000, 4_000, 700, 3_999, 1_000, 4_096),  # long rows throughout
    (1_000, 60_000, 30, 2_000, 50, 64),        # one block of columns
    (67, 900, 40, 300, 5, 10_000),             # few rows, 157 blocks: phases of blocks side by side
    (25_000, 8_000, 4_000, 8_000, 5_000, 64),  # 1e8 nonzeros: two chunks for their number
    (50_000, 300, 3, 300, 49_000, 130),        # a chunk of short rows after one long row; three blocks, the last of 2
])
def test_soft_backward_within_the_memory_of_eight_shares(n, d, short, long, every, k):
    from paper_2103_16141_amd._native import SivfError
    log("soft backward under caps n %d d %d k %d" % (n, d, k))
    X, row = _corpus(n, d, short, long, every, k)
    g = torch.Generator(device=device()).manual_seed(k)
    C = torch.rand(k, d, device=device(), generator=g)
    C /= torch.linalg.vector_norm(C, dim=1, keepdim=True)
    lse, _ = _ctx().soft_assign_fwd(X, C, 0.05)
    dC, dX = _ctx().soft_assign_bwd(X, C, 0.05, lse, 0.9)
    ref = torch.zeros(k, d, dtype=torch.float64, device=device())
    for lo in range(0, n, 2_000):
        hi = min(n, lo + 2_000)
        b, e = int(X.row_ptr[lo]), int(X.row_ptr[hi])
        D = torch.zeros(hi - lo, d, dtype=torch.float64, device=device())
        D[row[b:e] - lo, X.col[b:e].long()] = X.val[b:e].double()
        P = torch.softmax(D @ C.double().T / 0.05, 1)
        ref += (-0.9 / 0.05) * (P.T.contiguous() @ D)
    need, fits = _needed(X, k), []
    for cap in [need] + [int(need * 0.8 ** e) for e in range(1, 24)] + [1 << 12]:
        ctx = _ctx(workspace_cap_bytes=cap)
        try:
            c, x = ctx.soft_assign_bwd(X, C, 0.05, lse, 0.9)
        except SivfError as e:
            assert e.name == "SIVF_E_NOMEM"
            c = None
        fits.append(c is not None)
        if c is not None:
            # dX adds its blocks in order whatever is in memory at once; dC's sums
            # are cut where the chunks are
            assert torch.equal(x, dX)
            assert bool(((c.double() - ref).abs() <= 2e-3 * ref.abs() + 1e-7).all())
        ctx.close()
    assert fits[0] and fits == sorted(fits, reverse=True) and not fits[-1]
    assert bool(((dC.double() - ref).abs() <= 2e-3 * ref.abs() + 1e-7).all())


@pytest.mark.parametrize("n,d,short,long,every,k", [
    (300_000, 600, 5, 60, 10, 1_000),       # sixteen blocks: partials of 128 B a row
    (5_000, 20_000, 30, 300, 50, 777),      # C^T is most of it; the last block of 9 columns
    (7, 500, 20, 500, 3, 5_000),            # more blocks than eight per row
])
def test_soft_forward_within_the_memory_of_eight_partials(n, d, short, long, every, k):
    from paper_2103_16141_amd._native import SivfError
    log("soft forward under caps n %d d %d k %d" % (n, d, k))
    X, row = _corpus(n, d, short, long, every, k)
    C = torch.rand(k, d, device=device(), generator=torch.Generator(device=device()).manual_seed(k))
    C /= torch.linalg.vector_norm(C, dim=1, keepdim=True)
    want, loss = _ctx(workspace_cap_bytes=1 << 40).soft_assign_fwd(X, C, 0.05)
    ref = torch.empty(n, dtype=torch.float64, device=device())
    for lo in range(0, n, 10_000):
        hi = min(n, lo + 10_000)
        b, e = int(X.row_ptr[lo]), int(X.row_ptr[hi])
        D = torch.zeros(hi - lo, d, dtype=torch.float64, device=device())
        D[row[b:e] - lo, X.col[b:e].long()] = X.val[b:e].double()
        ref[lo:hi] = torch.logsumexp(D @ C.double().T / 0.05, 1)
    # a sum of at most d products of unit vectors' entries over tau; exp and log add 1e-5
    assert float((want.double() - ref).abs().max()) <= (long + 2) * 2.0 ** -24 / 0.05 + 1e-5
    need, fits = 9 * (4 * k * d + 64 * n) // 8 + (1 << 16), []
    for cap in [need] + [int(need * 0.8 ** e) for e in range(1, 12)] + [1 << 12]:
        ctx = _ctx(workspace_cap_bytes=cap)
        try:
            lse, lo = ctx.soft_assign_fwd(X, C, 0.05)
        except SivfError as e:
            assert e.name == "SIVF_E_NOMEM"
            lse = None
        fits.append(lse is not None)
        if lse is not None:
            assert torch.equal(lse, want) and abs(lo - loss) <= 1e-12 * abs(loss)
        ctx.close()
    assert fits[0] and fits == sorted(fits, reverse=True) and not fits[-1]


def test_soft_gradient_of_a_large_call_without_dense_terms():
    # nonzeros x k past the line of the products, every term in fewer than 1/32 of
    # the rows: the matrix of dense terms is not written and dC is the capped
    # call's (entries only) bit for bit
    log("no dense terms")
    n, d, k = 70_001, 40_000, 2_100
    dev = device()
    g = torch.Generator(device=dev).manual_seed(3)
    from paper_2103_16141_amd.api import DeviceCsr
    width = 40   # a term from each of 30 stripes of the first 1,200 terms
    col = torch.randint(width, (n, 30), device=dev, generator=g) + torch.arange(30, device=dev) * width
    v = torch.rand(n, 30, device=dev, generator=g) + 0.1
    v /= torch.linalg.vector_norm(v, dim=1, keepdim=True)
    X = DeviceCsr(torch.arange(n + 1, device=dev) * 30, col.int().reshape(-1).contiguous(), v.reshape(-1).contiguous(), d)
    assert X.nnz * k >= 1 << 32 and int(torch.bincount(col.reshape(-1)).max()) * 32 < n
    C = torch.rand(k, d, device=dev, generator=g)
    C /= torch.linalg.vector_norm(C, dim=1, keepdim=True)
    ctx = _ctx()
    lse, _ = ctx.soft_assign_fwd(X, C, 0.05)
    dC, dX = ctx.soft_assign_bwd(X, C, 0.05, lse, 0.9)
    pC, pX = _ctx(workspace_cap_bytes=1 << 40).soft_assign_bwd(X, C, 0.05, lse, 0.9)
    assert torch.equal(dC, pC) and torch.equal(dX, pX) and bool((dC != 0).any())


@pytest.mark.parametrize("d,k", [
    (16_777_215, 3),    # the last width whose slices a 4 GiB descriptor holds
    (16_777_216, 70),   # the first read by 64-bit offsets; two blocks of columns
    (20_000_000, 3),
])
def test_soft_form_of_very_wide_rows(d, k):
    from paper_2103_16141_amd.api import DeviceCsr
    log("wide rows d %d k %d" % (d, k))
    dev, tau, grad = device(), 0.05, 0.9
    g = torch.Generator(device=dev).manual_seed(d % 1000 + k)
    pool = torch.cat([torch.arange(100), d // 2 + torch.arange(100), d - 200 + torch.arange(200)]).to(dev)
    lens = 1 + (3 * torch.arange(134, device=dev)) % 200   # each number of 16-term groups, and more than 8
    n = lens.numel()
    order = torch.rand(n, 400, device=dev, generator=g).argsort(1)
    order[0] = torch.arange(399, -1, -1, device=dev)       # the last term alone
    take = torch.zeros(n, 400, dtype=torch.bool, device=dev)
    take.scatter_(1, order, torch.arange(400, device=dev)[None, :] < lens[:, None])
    D = torch.where(take, torch.rand(n, 400, device=dev, generator=g) + 0.1, 0.0)
    D /= torch.linalg.vector_norm(D, dim=1, keepdim=True)
    rp = torch.cat([torch.zeros(1, dtype=torch.int64, device=dev), take.sum(1).cumsum(0)])
    X = DeviceCsr(rp, pool[take.nonzero()[:, 1]].int().contiguous(), D[take].contiguous(), d)
    c = torch.rand(k, 400, device=dev, generator=g)
    c /= torch.linalg.vector_norm(c, dim=1, keepdim=True)
    C = torch.zeros(k, d, device=dev)
    C[:, pool] = c
    S = D.double() @ c.double().T / tau
    P = torch.softmax(S, 1)
    ctx = _ctx()
    lse, loss = ctx.soft_assign_fwd(X, C, tau)
    dC, dX = ctx.soft_assign_bwd(X, C, tau, lse, grad)
    ctx.close()
    # a sum of at most 200 products of unit vectors' entries over tau; exp and log add 1e-5
    assert float((lse.double() - torch.logsumexp(S, 1)).abs().max()) <= 202 * 2.0 ** -24 / tau + 1e-5
    # the terms of every sum have one sign, and P is off by the error of S and lse
    ref = -grad / tau * (P.T.contiguous() @ D.double())
    assert bool(((dC[:, pool].double() - ref).abs() <= 2e-3 * ref.abs() + 1e-7).all())
    ref = (-grad / tau * (P @ c.double()))[take]
    assert bool(((dX.double() - ref).abs() <= 2e-3 * ref.abs() + 1e-7).all())
    dC[:, pool] = 0.0
    assert not bool(dC.any())


@pytest.mark.parametrize("k", [64, 128, 129])
def test_soft_forward_of_many_rows_and_few_blocks(k):
    # 2^32 nonzeros x k and more: up to two blocks of columns by gathers alone (bit
    # for bit the capped call's), from three with the commonest terms in LDS
    from paper_2103_16141_amd.api import DeviceCsr
    log("many rows, k %d" % k)
    dev, d, per = device(), 2_000, 40
    n = (1 << 32) // (per * k) + 11
    g = torch.Generator(device=dev).manual_seed(k)
    # a term from each of 40 stripes, the first of a stripe most often
    off = (torch.rand(n, per, device=dev, generator=g) ** 3 * (d // per)).int()
    col = (off + torch.arange(per, device=dev, dtype=torch.int32) * (d // per)).reshape(-1).contiguous()
    v = torch.rand(n, per, device=dev, generator=g) + 0.1
    v /= torch.linalg.vector_norm(v, dim=1, keepdim=True)
    X = DeviceCsr(torch.arange(n + 1, device=dev) * per, col, v.reshape(-1).contiguous(), d)
    assert X.nnz * k >= 1 << 32
    C = torch.rand(k, d, device=dev, generator=g)
    C /= torch.linalg.vector_norm(C, dim=1, keepdim=True)
    lse, loss = _ctx().soft_assign_fwd(X, C, 0.05)
    plain, _ = _ctx(workspace_cap_bytes=1 << 40).soft_assign_fwd(X, C, 0.05)
    tol = (per + 2) * 2.0 ** -24 / 0.05 + 1e-5   # products of unit vectors' entries over tau; exp and log
    assert torch.equal(plain, lse) if k <= 128 else float((plain - lse).abs().max()) <= 2 * tol
    for rows in (slice(0, 3_000), slice(n - 3_000, n)):
        D = torch.zeros(3_000, d, dtype=torch.float64, device=dev)
        D.scatter_(1, col.view(n, per)[rows].long(), v[rows].double())
        ref = torch.logsumexp(D @ C.double().T / 0.05, 1)
        assert float((lse[rows].double() - ref).abs().max()) <= tol
    assert abs(loss + lse.double().sum().item()) <= 1e-9 * abs(loss)


@pytest.mark.parametrize("n,d,k,common,broken", [
    (70_001, 20_000, 2_500, 70, False),   # three chunks of rows, the last with splits of its own
    (70_001, 20_000, 2_500, 12, False),   # 7 dense terms a row are too few: entry by entry
])
def test_soft_gradient_of_dense_terms_over_several_chunks(n, d, k, common, broken):
    _dense_terms(n, d, k, common, broken)
