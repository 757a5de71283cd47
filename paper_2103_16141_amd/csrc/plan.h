// Sizes the host decides before it touches the device.  No HIP here: these are
// checked on the CPU over their whole ranges.
#pragma once

#include <algorithm>
#include <cstdint>

namespace sivf {

constexpr int kTileWide = 2048, kTileMid = 1536, kTileNarrow = 1024;   // automatic tile widths

// workgroups of 256 threads a launch may have: its threads are counted in 32 bits
constexpr int64_t kMaxGroups = (1 << 24) - 1;

// Tiles of k centroids holding an estimated `postings` over d terms; k_tile and
// bf16: the options the file was made with (k_tile 0: automatic).  Every
// tile repeats an object's work per term and its scan, so the widest is the best
// as long as its rows stay in cache; wider than 2048 costs occupancy (LDS).
// FP32, walk in ms with 1024 and 2048: 60,000 objects, k = 1,531 1.14 and 0.71
// (one tile for two); 400,000, k = 20,000 84.4 and 68.9; 5,000,000, k = 10,000
// 536 and 500 (2560: 10 - 15% more).  BF16 files, half the bytes, pay the
// scattered access to a wider tile sooner: sparse (the seed objects: 62.5 and
// 51.7) 2048; up to 3% dense, or in at most two tiles, 1536 (k = 10,000, 2%
// dense: 86.2 with 1024, 86.0 with 1536, 88.8 with 2048; k = 1,500, 12% dense
// 19.7 and 15.4); denser 1024 (5,000,000 objects, 6% dense: 439, 460, 490).
// FP32 files with many dense rows that no split walk will read: `heads` dense rows
// (0: few, unknown, or read by a split walk) are read through L2 by the plain walk, and
// a wide tile's no longer fit.  ms with 1024 and as wide as it gets, (rows, width):
// one tile (357, 1856) 1.26 and 1.10, (589, 2048) 1.53 and 1.51, (632, 2048) 5.80 and
// 5.94, (724, 1856) 5.75 and 5.85, (1,089, 2048) 14.7 and 16.6, (1,301, 2048) 12.2 and
// 16.5; (1,036, 1600) 5.9 and 5.5, (1,304, 1600) 11.9 and 13.0; (1,250, 1344) 5.1 and
// 4.6, (1,337, 1536) 10.1 and 10.0, (1,625, 1536) 2.7 and 3.6; (1,369, 1216) 10.1 and
// 8.3, (2,701, 1216) 13.1 and 11.3.  Two tiles (380, 2048) 10.9 both, (652, 2048) 27.2
// and 29.9, (1,201, 2048) 24.5 and 34.7; (819, 1664) 26.9 and 25.4, (1,233, 1664) 24.1
// and 26.2; (882, 1536) 21.4 and 21.8, (1,243, 1536) 18.7 and 20.2; (755, 1088) 7.5 both,
// (1,296, 1088) 15.4 and 16.8, (2,026, 1088) 5.0 and 7.7.  5 tiles: (278, 2048)
// 58.5 and 69.3, (214, 2048) 34.4 and 36.4, (250, 2048) 42.5 and 41.3; 9: (775, 1856)
// 25.5 and 38.1; 3 tiles: (382, 1728) 25.5 and 26.0, (151, 1728) 9.1 and 8.7.
// The lines hold for 30 terms a row and more (`terms`); shorter rows read fewer of the
// rows for the same work per tile: 17 terms (608, 2048) 2.03 and 1.96, (1,276, 2048) 5.1
// and 5.9, (1,827, 1472) 4.6 and 4.3, (2,881, 1472) 4.9 and 6.1, 3 tiles (316, 1600) 12.5
// and 10.7; 11 terms (880, 2048) 5.8 and 5.2, (1,321, 1472) 5.2 and 3.8.
// BF16 files narrow for the same reason, later: in two tiles from 2,600 rows on
// ((rows, width, D): 1,999, 1344, 30,000 9.44 with 1024 and 9.30 so; 2,725, 1536, 5,000
// 12.5 and 12.7; 2,878, 1344, 150,000 14.5 and 14.2; 3,465, 1344, 30,000 5.15 and 5.61;
// 4,285, 1536, 30,000 10.3 and 11.8), in more from 1,000 (967, 1536 39.2 and 39.2; 518,
// 1536 56.4 and 53.1; 1,221, 2048 19.2 and 20.0), from 800 if the narrow tiles' rows,
// which come in 512s, are shorter in all (431, 1344 4.81 and 4.84; 583, 1344 37.7 and
// 39.5; 831, 1344 37.7 and 40.3; 1,815, 1344 19.5 and 20.9), from 2,600 if longer (1,275,
// 1472 19.7 and 18.3); for 60 terms a row and more: 17 terms (1,244, 1216) 10.7 and 10.4,
// 25 (1,460, 1216) 9.0 and 9.2, 40 (2,620, 1216) 12.5 and 13.9.
// More postings or dense rows never give fewer tiles: a file's arrays are made for
// infinitely many.
inline void choose_tiles(int32_t k_tile, bool bf16, int32_t k, double postings, int64_t d, int64_t heads, double terms,
                         int32_t* kt, int32_t* T) {
    int32_t want = k_tile;
    if (want <= 0) {
        const double density = postings / ((double)k * (double)d);
        int32_t kmax = kTileWide;
        if (bf16 && density > 0.003) kmax = density < 0.033 || k <= 2 * kTileMid ? kTileMid : kTileNarrow;
        auto width = [k](int32_t most) {
            const int32_t t = (int32_t)(((int64_t)k + most - 1) / most);
            const int32_t w = (int32_t)(((int64_t)k + t - 1) / t);
            return ((w + 63) / 64) * 64;
        };
        want = width(kmax);
        const int32_t narrow = width(kTileNarrow);
        auto slots = [k](int32_t w) { return ((int64_t)k + w - 1) / w * ((w + 511) / 512 * 512); };
        const bool two = k <= 2 * (int64_t)want;
        if (want < k ? want > kTileNarrow : !bf16 && want > 1280) {
            const int64_t less = slots(want) - slots(narrow);
            const int64_t many = bf16       ? (two || less < 0 ? 2600 : less > 0 ? 800 : 1000)
                                 : !two     ? 260
                                 : want < k ? (want > 1792 ? 480 : 1100)
                                            : (want > 1728 ? 650 : want > 1536 ? 1200 : 1300);
            if ((double)heads * std::min(1.0, terms / (bf16 ? 60.0 : 30.0)) >= (double)many) want = narrow;
        }
    }
    *kt = want;
    *T = (int32_t)(((int64_t)k + want - 1) / want);
}

// Objects a wave grabs from a walk's counter at a time: 8, or at least four times.
inline int64_t walk_grab(int64_t n, int64_t waves) {
    return std::max<int64_t>(1, std::min<int64_t>(8, n / (waves * 4)));
}

// Members up to which a cluster of more than a tile of nonzeros is summed member by
// member (k_upd_members), 0: none is.  The sums of the whole vocabulary have to fit
// 64 KB of LDS.  A member waits for the one before it, 0.4 us in all, and the tiles of
// all clusters take 24 ps a nonzero, so only chains of at most nonzeros / 100,000
// members (a sixth of that) are worth it, and only where most clusters have more than
// a tile and are no longer: 1.5 times the mean is, the limit is twice the mean.  Update in us, tiles and
// members, D = 4,000, flat vocabulary: 150,000 rows of 200 terms, k = 3,000 2,016 and
// 994; 400,000 rows, k = 1,000 2,372 and 969; 1,000,000 rows of 75, k = 10,000 6,278
// and 3,138; skewed: 400,000 rows of 200, k = 1,000 2,296 and 2,042.  Where the mean is
// longer: 1,000,000 rows of 75, k = 1,000 2,160 and 2,587.
inline int64_t upd_members(int64_t n, int64_t nnz, int64_t d, int64_t k) {
    const int64_t chain = nnz / 100000;
    return d <= 8192 && nnz > 4096 * k && 2 * chain * k >= 3 * n ? std::min(2 * n / k, chain) : 0;
}

// Whether the waves of a walk of `tiles` tiles take equal shares of n objects instead,
// of `terms` terms on average (split: of the listed ones).  A grab costs 15 ns, one
// after the other for all waves: 22,000 of them (44,000 objects by twos) hold a walk
// that could be done in 80 us to 340.  But the heavier an object, the more uneven the
// shares, and the less the counter shows: the line is where the objects of a grab take
// about as long as the grab itself, by an estimate that fits these.  Walk in us by grabs
// and in equal shares, FP32, 60 terms an object: 60,000 objects (12 a wave, by twos) k =
// 1 435 and 97, 100 479 and 390, 300 515 and 465, 2,048 654 and 724; 100,000 (by fours)
// k = 16 430 and 390, 100 630 and 655; 100 terms, 55,000 objects, k = 500 564 and 620;
// 131 terms over a wide vocabulary, 42,569 objects, k = 242 757 and 854; 273 terms,
// 88,424 objects, k = 1 1,960 and 2,210.  Lists of a split walk, 100 terms, about 45 listed: 55,000
// objects, k = 500 721 and 508, k = 2,000 1,200 and 1,216; 70,000, k = 1,000 993 and 958;
// 100,000, k = 500 914 and 770, k = 1,000 1,281 and 1,324.  Over 1,940 walks of four
// vocabularies, 30,000 to 115,000 objects of 5 to 130 terms, k = 16 to 4,000, it loses
// 1.7% on average to the better way of each (worst: two light tiles a launch, 14%).
inline bool walk_shared(int64_t n, int64_t waves, double terms, int32_t kt, int tiles, bool split) {
    if (n <= 8 * waves) return true;
    if (n > 24 * waves) return false;
    const double object = terms * (0.065 + (split ? 0.000045 : 0.00009) * kt) * tiles;   // ns of the whole chip
    return object * (double)walk_grab(n, waves) <= 17.0;
}

// pairs of a range of the split walk's objects: two chunks of fill, then every
// object's, filled up twice
inline int64_t split_pairs(int64_t nnz, int64_t objects) { return 32 + nnz + 32 * objects; }
constexpr int64_t kSplitMaxPairs = (1 << 29) - 1;   // of a range: less than 4 GiB

// Objects per range: at most `most` (at least 1), halved while the longest range
// has too many pairs; 0 if that is so for one object, pays(range) ends, or
// longest(range), the nonzeros of the longest range, is negative (not known).
template <typename Pays, typename Longest>
int64_t split_range(int64_t most, Pays pays, Longest longest, int64_t* pairs) {
    for (int64_t range = most;; range = (range + 1) / 2) {
        if (!pays(range)) return 0;
        const int64_t nnz = longest(range);
        if (nnz < 0) return 0;
        *pairs = split_pairs(nnz, range);
        if (*pairs <= kSplitMaxPairs) return range;
        if (range == 1) return 0;
    }
}

// ---------------------------------------------------------------- soft forward
// As for the backward below: rows per launch and blocks of 64 columns in C^T at
// once.  The per-block partials of one launch take at most 512 MiB, in the later
// plans 64 B per row of the matrix.
struct SoftFwdPlan {
    int64_t rows, blocks;
};

inline bool soft_fwd_plan(int attempt, int64_t n, int64_t nblk, SoftFwdPlan* p) {
    const int64_t partials = attempt == 0 ? (int64_t)64 << 20 : 8 * n;
    p->rows = std::max<int64_t>(1, std::min<int64_t>(n, partials / nblk));
    p->blocks = attempt < 2 ? nblk : 1;
    return attempt < 3;
}

// Whether the forward keeps its commonest terms' slices in LDS: from 2^32 nonzeros
// x k, and from three blocks of columns.  Fewer leave most XCDs to one block, whose
// slices their L2 holds, and the pairs and LDS panels are made for little.  Forward
// in ms without and with, 6.5e9 nonzeros x k, 30 terms a row (D = 20,000) and 100
// (50,000): k = 64 1.88 and 3.50, 1.68 and 2.24; 128 1.67 and 2.23, 1.47 and 1.60;
// 160 2.31 and 2.25, 2.01 and 1.65; 256 1.52 and 1.56, 1.30 and 1.29; 320 2.23 and
// 1.49, 1.91 and 1.24; 512 1.45 and 1.30, 1.31 and 1.13.  Smaller calls, k of 1,021
// to 4,096: 1.8e9 0.44 and 0.48, 2.2e9 0.63 and 0.65, 3.7e9 0.77 and 0.69.
inline bool soft_lds_pays(int64_t nnz, int64_t k) { return nnz * k >= (int64_t)1 << 32 && k > 128; }

// ---------------------------------------------------------------- soft backward
// What of the backward is in memory at once: chunks of `rows` rows, `blocks`
// blocks of 64 columns, the column copy of the whole matrix or of a chunk.
struct SoftPlan {
    int64_t rows, blocks;
    bool whole;
};

// The attempt-th plan, until one fits the memory; false: there is none left.
// Each needs less than the one before: all columns at once; eight blocks (one
// per XCD); one block and the copy of a chunk, 31 B per nonzero of a chunk and
// 556 B per term; the same with ever fewer rows.  The results are the same, but
// for the rounding where dC's chunks are cut elsewhere.
// Rows: 24,576 rows of a 32-column dS block take 3 MB of an XCD's
// 4 MB L2; smaller chunks read and write dC more often, larger ones miss L2.
// Where a term has few entries in a chunk (below 32 on average), dC costs more
// than the misses: backward with 16,384 / 24,576 / 32,768 / 40,960 rows, N =
// 262,144, D = 100,000, 100 terms, k = 4,096 (25 entries) 78.6 / 73.2 / 71.0 /
// 71.6 ms; N = 97,062, D = 38,883, 177 terms, k = 3,837 (112) - / 46.2 / 47.5 /
// 48.9.  The line is a rough one (it also matters how full the last chunk is): against
// 24,576 rows, 32,768 take, at 8 / 14 / 18 / 21 / 24 / 28 / 31 entries, 7 / 5 / 4 / 4 /
// 1 / 2 / 1% less (N = 131,072, D = 50,000, k = 512), 4 / 4 / 3 / 4 / 3 / 2 / 1% less
// (200,000, 100,000, 512), 5 / 3 / 3 / 1 / 1 / 0 / 0% less (131,072, 50,000, 1,500), but
// 5 / 1 / 1% less and 1 / 0 / 2 / 1% more (131,072, 50,000, 4,000) and 2% less, then 1 /
// 4 / 1 / 3 / 6 / 7% more (200,000, 100,000, 4,000).  dS of a chunk is at most 512 MiB.
inline bool soft_bwd_plan(int attempt, int64_t n, int64_t nnz, int64_t d, int64_t nblk, SoftPlan* p) {
    const int64_t most = (double)nnz * 24576.0 < 32.0 * (double)n * (double)d ? 32768 : 24576;
    int64_t rows = std::max<int64_t>(1, std::min<int64_t>({std::max<int64_t>(n, 1), most, (int64_t)(128ll << 20) / (64 * nblk)}));
    for (int a = 3; a <= attempt; ++a) {
        if (rows == 1) return false;
        rows = (rows + 1) / 2;
    }
    *p = SoftPlan{rows, attempt == 0 ? nblk : attempt == 1 ? std::min<int64_t>(nblk, 8) : 1, attempt < 2};
    return true;
}

// Whether dC of the densest terms may be made by matrix products: in calls of 2^32
// nonzeros x k.  Whether it is depends on their entries (at most all; the device knows
// them): an entry costs 0.5 ps a column, a row of the matrix of dense terms 4 ns and its
// products 5 ps a column.  Backward in ms without and with, 8.6e9 nonzeros x k, by dense terms a row:
// 9 (40 terms, D = 20,000) k = 256 8.25 and 10.41, 1,024 6.27 and 6.99, 3,000 7.32 and
// 7.55; 14 (100, 100,000) 256 6.61 and 7.41, 1,536 5.93 and 5.93, 3,000 7.13 and 6.81;
// 41 (200, 30,000) 256 7.04 and 7.26, 512 6.18 and 6.13, 2,048 6.53 and 6.13; 52
// (109, 2,281, 2.5e10) 922 14.6 and 11.9; 30 terms, k = 64, 3,000,000 rows 14.4 and 28.5.
constexpr bool soft_prod_pays(double entries, double n, double k) { return entries * k >= n * (8000.0 + 10.0 * k); }
inline bool soft_prod_may(int64_t n, int64_t nnz, int64_t k) {
    return nnz * k >= (int64_t)1 << 32 && soft_prod_pays((double)nnz, (double)n, (double)k);
}

// A chunk of rows takes 5 B per nonzero and block for dX's shares (4) and dC's
// partial rows (1): blocks are taken in groups of at least eight where those of
// the longest chunk would pass 2 GiB, and chunks of more than kSoftChunkNnz
// nonzeros are halved.
constexpr int64_t kSoftChunkNnz = 1ll << 26;
inline int64_t soft_bwd_blocks(int64_t blocks, int64_t nnz_max) {
    const int64_t fit = (int64_t)(2ll << 30) / (5 * std::max<int64_t>(nnz_max, 1));
    return fit >= blocks ? blocks : std::min(blocks, std::max<int64_t>(8, fit / 8 * 8));
}

}  // namespace sivf
