// Sizes the host decides before it touches the device.  No HIP here: these are
// checked on the CPU over their whole ranges.
#pragma once

#include <cstdint>

namespace sivf {

constexpr int kTileWide = 2048, kTileMid = 1536, kTileNarrow = 1024;   // automatic tile widths

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
// More postings never give fewer tiles: a file's arrays are made for infinitely
// many.
inline void choose_tiles(int32_t k_tile, bool bf16, int32_t k, double postings, int64_t d, int32_t* kt, int32_t* T) {
    int32_t want = k_tile;
    if (want <= 0) {
        const double density = postings / ((double)k * (double)d);
        int32_t kmax = kTileWide;
        if (bf16 && density > 0.003) kmax = density < 0.033 || k <= 2 * kTileMid ? kTileMid : kTileNarrow;
        const int32_t t = (int32_t)(((int64_t)k + kmax - 1) / kmax);
        const int32_t w = (int32_t)(((int64_t)k + t - 1) / t);
        want = ((w + 63) / 64) * 64;
    }
    *kt = want;
    *T = (int32_t)(((int64_t)k + want - 1) / want);
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

}  // namespace sivf
