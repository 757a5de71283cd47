// Stable radix sort of (key, row, value) entries by a small integer key
// (k_sort.hip): the column copy of X (soft form) and the objects by cluster.
#pragma once

#include "internal.h"

namespace sivf {

// Where the entries of the first pass come from.  Entry p in [0, n):
//   kSortCsr:    rows of a CSR matrix: key[p], value val[p], row row0 + r with rp[r] <= p0 + p < rp[r + 1]
//   kSortIota:   key[p], row p, no value
enum SortSource { kSortCsr, kSortIota };

template <typename V>
struct SortIn {
    SortSource kind;
    int64_t n;              // entries
    const int32_t* key;
    const V* val;           // kSortIota: nullptr
    int64_t rows;           // kSortCsr
    const int64_t* rp;      // row bounds, p0 the first of them
    int64_t p0, row0;
};

// two buffers of entries (val: nullptr without values), the digit counts of
// every tile and their scan
template <typename V>
struct SortWs {
    int32_t* key[2];
    int32_t* row[2];
    V* val[2];
    int64_t* count;   // [sort_table_elems(n)]
    int64_t* start;   // [sort_table_elems(n)]
    int64_t* scan_ws; // scan_ws_elems(sort_table_elems(n))
};

int64_t sort_table_elems(int64_t n);

// Sorts by key in [0, nkeys), equal keys in entry order.  *key, *row and *val
// point to the sorted entries in w.
template <typename V>
hipError_t sort_entries(const SortIn<V>& in, int64_t nkeys, const SortWs<V>& w, const int32_t** key,
                        const int32_t** row, const V** val, hipStream_t s);

// ptr[t] = first of the n sorted entries with key >= t, t in [0, nkeys]
hipError_t sort_starts(const int32_t* key, int64_t n, int64_t nkeys, int64_t* ptr, hipStream_t s);

}  // namespace sivf
