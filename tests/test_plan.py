"""Sizes the host decides without a device (csrc/plan.h), compiled for the CPU
and checked over their ranges."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

HARNESS = r"""
#include "plan.h"
extern "C" {
void tiles(int32_t k_tile, int bf16, int32_t k, double postings, int64_t d, int64_t heads, double terms, int32_t* kt,
           int32_t* T) {
    sivf::choose_tiles(k_tile, bf16 != 0, k, postings, d, heads, terms, kt, T);
}
int bwd_plan(int attempt, int64_t n, int64_t nnz, int64_t d, int64_t nblk, int64_t* rows, int64_t* blocks, int* whole) {
    sivf::SoftPlan p;
    if (!sivf::soft_bwd_plan(attempt, n, nnz, d, nblk, &p)) return 0;
    *rows = p.rows;
    *blocks = p.blocks;
    *whole = p.whole;
    return 1;
}
int lds_pays(int64_t nnz, int64_t k) { return sivf::soft_lds_pays(nnz, k); }
int prod_may(int64_t n, int64_t nnz, int64_t k) { return sivf::soft_prod_may(n, nnz, k); }
int prod_pays(int64_t entries, int64_t n, int64_t k) { return sivf::soft_prod_pays(entries, n, k); }
int64_t members(int64_t n, int64_t nnz, int64_t d, int64_t k) { return sivf::upd_members(n, nnz, d, k); }
int64_t bwd_blocks(int64_t blocks, int64_t nnz_max) { return sivf::soft_bwd_blocks(blocks, nnz_max); }
int shared(int64_t n, int64_t waves, double terms, int32_t kt, int split, int tiles) {
    return sivf::walk_shared(n, waves, terms, kt, tiles, split != 0);
}
typedef int64_t (*fn)(int64_t);
int64_t split(int64_t most, fn pays, fn longest, int64_t* pairs) {
    return sivf::split_range(most, [=](int64_t r) { return pays(r) != 0; }, longest, pairs);
}
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    src, lib = d / "plan.cpp", d / "plan.so"
    src.write_text(HARNESS)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I",
                           os.path.join(ROOT, "paper_2103_16141_amd", "csrc"), str(src), "-o", str(lib)])
    return ctypes.CDLL(str(lib))


def test_no_number_of_postings_gives_more_tiles_than_a_file_is_made_for(plan):
    # a file's arrays are allocated for infinitely many postings; an update
    # chooses the tiles again for the postings it expects
    def tiles(k_tile, bf16, k, postings, d, heads, terms=60.0):
        kt, T = ctypes.c_int32(), ctypes.c_int32()
        plan.tiles(k_tile, bf16, k, ctypes.c_double(postings), ctypes.c_int64(d), ctypes.c_int64(heads), ctypes.c_double(terms), ctypes.byref(kt),
                   ctypes.byref(T))
        return kt.value, T.value

    rng = np.random.default_rng(0)
    ks = [1, 63, 64, 65, 1023, 1024, 1025, 1536, 1537, 2047, 2048, 2049, 3071, 3072, 3073, 4096, 2 ** 31 - 1]
    ks += [int(k) for k in np.exp(rng.uniform(0, np.log(1e7), 2000))]
    for k in ks:
        for bf16 in (0, 1):
            for k_tile in (0, 64, 128, 4096):
                for heads in (0, 200, 300, 500, 700, 1000, 1200, 2600, 2 ** 63 - 1):
                    _, most = tiles(k_tile, bf16, k, float("inf"), 1000, 2 ** 63 - 1 if heads else 0, float("inf"))
                    for density in (0.0, 0.002, 0.004, 0.03, 0.04, 1.0):
                        kt, T = tiles(k_tile, bf16, k, density * k * 1000, 1000, heads)
                        assert T <= most and kt % 64 == 0 and 64 <= kt <= 4096 and (T - 1) * kt < k <= T * kt
    width = lambda k, heads: tiles(0, 0, k, 0.0, 1000, heads, 30.0)[0]
    assert [width(2048, h) for h in (0, 649, 650)] == [2048, 2048, 1024]
    assert [width(1600, h) for h in (1199, 1200)] == [1600, 832] and [width(1500, h) for h in (1299, 1300)] == [1536, 768]
    assert [width(4000, h) for h in (479, 480)] == [2048, 1024] and [width(2500, h) for h in (1099, 1100)] == [1280, 896]
    assert [width(10_000, h) for h in (259, 260)] == [2048, 1024] and width(1280, 10 ** 6) == 1280
    bf16 = lambda k, heads: tiles(0, 1, k, 0.02 * k * 1000, 1000, heads)[0]
    assert [bf16(3072, h) for h in (2599, 2600)] == [1536, 1024] and bf16(2100, 2600) == 704
    assert [bf16(4000, h) for h in (799, 800)] == [1344, 1024]     # 4,608 and 4,096 slots
    assert [bf16(12_288, h) for h in (999, 1000)] == [1536, 1024]   # 12,288 both
    assert [bf16(7319, h) for h in (2599, 2600)] == [1472, 960]     # 7,680 and 8,192
    # shorter rows, later
    assert [tiles(0, 0, 2048, 0.0, 1000, h, 15.0)[0] for h in (1299, 1300)] == [2048, 1024]
    assert [tiles(0, 1, 4000, 80_000.0, 1000, h, 15.0)[0] for h in (3199, 3200)] == [1344, 1024]
    assert bf16(1536, 10 ** 6) == 1536 and bf16(2048, 10 ** 6) == 1024


@pytest.mark.parametrize("objects,row,floor,want", [
    (1, 1 << 30, 0, 0),                        # one row alone has too many pairs: not split
    (1_000_000, 1 << 30, 0, 0),
    (1_000_000, 100, 0, 1_000_000),            # everything fits
    (1_000_000, 2_000, 0, 250_000),            # 2,032 pairs an object: at most 264,208 objects
    (1_000_000, 2_000, 300_000, 0),            # no longer pays so small
    (3, (1 << 29) - 65, 0, 1),                 # one row just fits (64 pairs of fill)
    (3, (1 << 29) - 64, 0, 0),                 # one more does not
])
def test_ranges_of_the_split_walk_end(plan, objects, row, floor, want):
    fn = ctypes.CFUNCTYPE(ctypes.c_int64, ctypes.c_int64)
    calls = []

    def longest(r):
        calls.append(r)
        assert len(calls) < 64, "does not end"
        return r * row

    plan.split.restype = ctypes.c_int64
    pairs = ctypes.c_int64()
    got = plan.split(ctypes.c_int64(objects), fn(lambda r: r >= floor), fn(longest), ctypes.byref(pairs))
    assert got == want
    if want:
        assert pairs.value == 32 + want * (row + 32)


def test_soft_backward_plans_shrink_to_less_than_eight_shares_took(plan):
    # bytes per array, as the library asks for them, against 32 B per nonzero of a
    # chunk of 2^26 / k rows, 8 B per nonzero, counts per 1,024 rows and 88 B a term
    plan.bwd_plan.restype = ctypes.c_int
    plan.bwd_blocks.restype = ctypes.c_int64
    rng = np.random.default_rng(1)
    for _ in range(3000):
        k = int(np.exp(rng.uniform(np.log(64), np.log(1e5))))
        n = int(np.exp(rng.uniform(0, np.log(1e7))))
        d = int(np.exp(rng.uniform(np.log(100), np.log(1e6))))
        lam = int(np.exp(rng.uniform(0, np.log(d))))
        nnz, nblk, least = n * lam, (k + 63) // 64, None
        old_rows = max(1, min(n, (64 << 20) // k))
        old = 8 * k * d + 4 * old_rows * k + 40 * old_rows * lam + 88 * d
        attempt = 0
        while True:
            rows, blocks, whole = ctypes.c_int64(), ctypes.c_int64(), ctypes.c_int()
            if not plan.bwd_plan(attempt, ctypes.c_int64(n), ctypes.c_int64(nnz), ctypes.c_int64(d),
                                 ctypes.c_int64(nblk), ctypes.byref(rows), ctypes.byref(blocks), ctypes.byref(whole)):
                break
            rows, copy = rows.value, nnz if whole.value else min(n, rows.value) * lam
            blocks = plan.bwd_blocks(ctypes.c_int64(blocks.value), ctypes.c_int64(rows * lam))
            assert 1 <= rows <= max(n, 1) and 1 <= blocks <= nblk
            if attempt == 0 and 5 * rows * lam * nblk <= 2 << 30:
                assert blocks == nblk   # everything at once where it is not much
            size = 512 * blocks * d + 256 * rows * blocks + 5 * rows * lam * blocks + 26 * copy + 44 * d + 16384
            if least is not None:
                assert size <= least + 16384
            least, last, attempt = size, (rows, blocks), attempt + 1
        assert last == (1, 1) and attempt < 40
        # the last plan fits wherever those bytes were there
        assert least <= old + 16384


def test_equal_shares_reach_further_for_lighter_walks(plan):
    def shared(n, terms, kt, split=0, waves=5_120, tiles=1):
        return plan.shared(ctypes.c_int64(n), ctypes.c_int64(waves), ctypes.c_double(terms), kt, split, tiles)

    assert shared(1, 1e6, 4096) and shared(40_960, 1e6, 4096)            # up to 8 objects a wave whatever they cost
    assert not shared(122_881, 0, 64) and not shared(122_881, 0, 64, 1)  # never beyond 24
    assert [shared(60_000, 60, kt) for kt in (64, 128, 320, 1024)] == [1, 1, 1, 0]
    assert shared(60_000, 60, 128, tiles=1) and not shared(60_000, 60, 128, tiles=2)
    assert [shared(100_000, 60, kt) for kt in (64, 128)] == [1, 0]
    assert not shared(55_000, 100, 512) and not shared(42_569, 131, 256) and not shared(88_424, 273, 64, waves=6_144)
    assert [shared(55_000, 45, kt, 1) for kt in (512, 1024)] == [1, 1] and not shared(55_000, 45, 2048, 1, waves=4_096)
    for n in (41_000, 60_000, 80_000, 100_000, 122_880):   # fewer terms or narrower tiles never take it away
        for kt in (64, 512, 2048):
            got = [shared(n, t, kt) for t in (0, 5, 20, 60, 200, 1000)]
            assert got == sorted(got, reverse=True) and all(shared(n, t, 64) >= g for t, g in zip((0, 5, 20), got))


def test_soft_forward_uses_lds_in_larger_calls_of_three_blocks_and_more(plan):
    pays = lambda nnz, k: plan.lds_pays(ctypes.c_int64(nnz), ctypes.c_int64(k)) != 0
    assert [pays(1 << 26, k) for k in (1, 63, 64, 65, 128, 129, 4_096)] == [False] * 5 + [True] * 2
    assert not pays((1 << 20) - 1, 4_096) and pays(1 << 20, 4_096) and not pays(0, 4_096)


def test_dense_terms_are_products_where_rows_hold_enough_of_them(plan):
    pays = lambda entries, n, k: plan.prod_pays(*(ctypes.c_int64(i) for i in (entries, n, k))) != 0
    assert pays(18_000, 1_000, 1_000) and not pays(17_999, 1_000, 1_000)
    assert pays(13 * 10 ** 9, 10 ** 9, 4_096) and not pays(256 * 10, 10, 32)   # all 256 terms in every row
    assert not pays(0, 1, 4_096) and not pays(0, 10 ** 9, 10 ** 9)
    may = lambda n, nnz, k: plan.prod_may(*(ctypes.c_int64(i) for i in (n, nnz, k))) != 0
    assert may(10_000, 1 << 22, 1_024) and not may(10_000, (1 << 22) - 1, 1_024)   # in all
    assert may(10 ** 6, 18 * 10 ** 6, 1_000) and not may(10 ** 6, 18 * 10 ** 6 - 1, 1_000)   # too few terms a row, dense or not


def test_member_by_member_only_where_chains_are_short_and_sums_fit(plan):
    plan.members.restype = ctypes.c_int64
    members = lambda *a: plan.members(*(ctypes.c_int64(i) for i in a))
    assert members(400_000, 80_000_000, 4_000, 1_000) == 800 and members(400_000, 80_000_000, 4_000, 3_000) == 266
    assert members(400_000, 80_000_000, 8_192, 3_000) == 266 and members(400_000, 80_000_000, 8_193, 3_000) == 0
    assert members(100_000, 15_000_000, 4_000, 1_000) == 150 and members(100_000, 15_000_000, 4_000, 999) == 0
    assert members(150_000, 11_250_000, 4_000, 2_747) == 0 and members(150_000, 11_250_000, 4_000, 2_746) > 0   # a tile
    assert members(1, 0, 1, 1) == 0 and members(0, 0, 5, 3) == 0
