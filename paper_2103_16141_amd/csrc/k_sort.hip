// Stable radix sort, 9 bits per pass (sort.h).  A pass counts the digits of
// every tile of 4,096 entries, scans the counts digit by digit, and moves each
// tile's entries, sorted by the digit in LDS first, so that every digit's share
// of a tile is written in one run.  No ordering atomics: the result is the same
// on every run.
// Bound: the bytes moved, about 44 per entry for two passes with FP32 values.
// Column copy of X: one workgroup walking 1,024 rows in order took 650 us for
// 1,000 rows of 50 and 3.5 ms for 262,144 rows of 100; this takes 60 us and
// 1.2 ms.
#include "sort.h"
#include "tile_sort.h"
#include "wave.h"

namespace sivf {

constexpr int kMoved = -1;   // later passes: entries of the previous one

// last row starting at or before entry p, among rows [lo, hi]
__device__ inline int64_t row_of(const int64_t* __restrict__ rp, int64_t lo, int64_t hi, int64_t p) {
    while (lo < hi) {
        const int64_t mid = (lo + hi + 1) >> 1;
        if (rp[mid] <= p) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

template <typename V>
struct SortArgs {
    SortIn<V> in;
    const int32_t* key;   // kMoved
    const int32_t* row;
    const V* val;
    int shift, nbits;
    int64_t ntiles;
};

template <int KIND, typename V>
__global__ __launch_bounds__(kFoldThreads) void k_sort_hist(SortArgs<V> A, int64_t* __restrict__ table) {
    __shared__ uint32_t h[kFoldBins];
    const uint32_t dm = (1u << A.nbits) - 1u;
    h[threadIdx.x] = 0;
    __syncthreads();
    const int64_t n = A.in.n, lo = (int64_t)blockIdx.x * kFoldTile;
#pragma unroll
    for (int i = 0; i < kFoldPer; ++i) {
        const int64_t p = lo + i * kFoldThreads + threadIdx.x;
        if (p < n) atomicAdd(&h[((uint32_t)(KIND == kMoved ? A.key : A.in.key)[p] >> A.shift) & dm], 1u);
    }
    __syncthreads();
    table[(int64_t)threadIdx.x * A.ntiles + blockIdx.x] = h[threadIdx.x];
}

// (values go through LDS as floats)
struct SortLds {
    uint32_t key[kFoldTile];
    int32_t row[kFoldTile];
    float val[kFoldTile];
    uint16_t order[kFoldTile];
    int64_t at[kFoldBins];
    TileSortLds s;
};

template <int KIND, typename V>
__global__ __launch_bounds__(kFoldThreads) void k_sort_move(SortArgs<V> A, const int64_t* __restrict__ table,
                                                            int32_t* __restrict__ okey, int32_t* __restrict__ orow,
                                                            V* __restrict__ oval) {
    static_assert(sizeof(V) == sizeof(float), "a wider value would be rounded in LDS");
    __shared__ SortLds L;
    const int tid = threadIdx.x;
    const int64_t n = A.in.n, lo = (int64_t)blockIdx.x * kFoldTile;
    if (lo >= n) return;   // workgroup-uniform
    const int ne = (int)min((int64_t)kFoldTile, n - lo);
    int64_t ra = 0, rb = 0;
    if (KIND == kSortCsr) {
        ra = row_of(A.in.rp, 0, A.in.rows - 1, A.in.p0 + lo);
        rb = row_of(A.in.rp, ra, A.in.rows - 1, A.in.p0 + lo + ne - 1);
    }
#pragma unroll
    for (int i = 0; i < kFoldPer; ++i) {
        const int e = i * kFoldThreads + tid;
        if (e >= ne) continue;
        const int64_t p = lo + e;
        if (KIND == kMoved) {
            L.key[e] = (uint32_t)A.key[p];
            L.row[e] = A.row[p];
            if (A.val) L.val[e] = A.val[p];
        } else if (KIND == kSortIota) {
            L.key[e] = (uint32_t)A.in.key[p];
            L.row[e] = (int32_t)p;
        } else {
            const int64_t r = row_of(A.in.rp, ra, rb, A.in.p0 + p);
            L.key[e] = (uint32_t)A.in.key[p];
            L.row[e] = (int32_t)(A.in.row0 + r);
            L.val[e] = A.in.val[p];
        }
    }
    const int64_t first = table[(int64_t)tid * A.ntiles + blockIdx.x];
    __syncthreads();
    tile_radix(L.s, L.key, nullptr, L.order, ne, A.shift, A.nbits);
    L.at[tid] = first - L.s.base[tid];
    __syncthreads();
    const uint32_t dm = (1u << A.nbits) - 1u;
#pragma unroll
    for (int i = 0; i < kFoldPer; ++i) {
        const int s = i * kFoldThreads + tid;
        if (s >= ne) continue;
        const int e = L.order[s];
        const int64_t to = L.at[(L.key[e] >> A.shift) & dm] + s;
        okey[to] = (int32_t)L.key[e];
        orow[to] = L.row[e];
        if (oval) oval[to] = L.val[e];
    }
}

int64_t sort_table_elems(int64_t n) { return ((n + kFoldTile - 1) / kFoldTile) * kFoldBins + 1; }

template <int KIND, typename V>
static hipError_t sort_pass(const SortArgs<V>& A, const SortWs<V>& w, int b, hipStream_t s) {
    const dim3 grid((unsigned)A.ntiles), wg(kFoldThreads);
    hipLaunchKernelGGL((k_sort_hist<KIND, V>), grid, wg, 0, s, A, w.count);
    const hipError_t e = exclusive_scan_i64(w.count, w.start, A.ntiles * kFoldBins, w.scan_ws, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_sort_move<KIND, V>), grid, wg, 0, s, A, w.start, w.key[b], w.row[b], w.val[b]);
    return hipGetLastError();
}

template <typename V>
hipError_t sort_entries(const SortIn<V>& in, int64_t nkeys, const SortWs<V>& w, const int32_t** key,
                        const int32_t** row, const V** val, hipStream_t s) {
    int passes, nbits;
    tile_sort_plan(nkeys, &passes, &nbits);
    SortArgs<V> A{in, nullptr, nullptr, nullptr, 0, nbits, (in.n + kFoldTile - 1) / kFoldTile};
    for (int p = 0; p < passes && A.ntiles > 0; ++p) {
        const int b = p & 1;
        A.shift = p * nbits;
        const hipError_t e = p > 0                  ? sort_pass<kMoved, V>(A, w, b, s)
                             : in.kind == kSortCsr ? sort_pass<kSortCsr, V>(A, w, b, s)
                                                   : sort_pass<kSortIota, V>(A, w, b, s);
        if (e != hipSuccess) return e;
        A.key = w.key[b];
        A.row = w.row[b];
        A.val = w.val[b];
    }
    *key = A.key;
    *row = A.row;
    *val = A.val;
    return hipSuccess;
}
template hipError_t sort_entries<float>(const SortIn<float>&, int64_t, const SortWs<float>&, const int32_t**,
                                        const int32_t**, const float**, hipStream_t);
__global__ void k_sort_starts(int64_t nkeys, int64_t n, const int32_t* __restrict__ key, int64_t* __restrict__ ptr) {
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (t > nkeys) return;
    int64_t lo = 0, hi = n;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (key[mid] < t) lo = mid + 1;
        else hi = mid;
    }
    ptr[t] = lo;
}

hipError_t sort_starts(const int32_t* key, int64_t n, int64_t nkeys, int64_t* ptr, hipStream_t s) {
    hipLaunchKernelGGL(k_sort_starts, dim3((unsigned)((nkeys + 256) / 256)), dim3(256), 0, s, nkeys, n, key, ptr);
    return hipGetLastError();
}

}  // namespace sivf
