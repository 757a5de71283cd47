// Column copy (CSC) of an FP32 CSR matrix with ascending rows per column: a
// stable radix sort of the nonzeros by column, 9 bits per pass.  A pass counts
// the digits of every tile of 4,096 nonzeros, scans the counts digit by digit,
// and moves each tile's nonzeros, sorted by the digit in LDS first, so that
// every digit's share of a tile is written in one run.
// Bound: about 44 bytes moved per nonzero for two passes.  One workgroup
// walking 1,024 rows in order (a count per row block and column, then one
// wave's cursors) took 650 us for 1,000 rows of 50 and 3.5 ms for 262,144 rows
// of 100; this takes 60 us and 1.2 ms.
#include "internal.h"
#include "soft.h"
#include "tile_sort.h"
#include "wave.h"

namespace sivf {

struct CscLds {
    uint32_t key[kFoldTile];
    int32_t row[kFoldTile];
    float val[kFoldTile];
    uint16_t order[kFoldTile];
    int64_t at[kFoldBins];
    TileSortLds s;
};

__global__ __launch_bounds__(kFoldThreads) void k_csc_hist(int64_t nnz, const int32_t* __restrict__ key, int shift,
                                                           int nbits, int64_t ntiles, int64_t* __restrict__ table) {
    __shared__ uint32_t h[kFoldBins];
    const uint32_t dm = (1u << nbits) - 1u;
    h[threadIdx.x] = 0;
    __syncthreads();
    const int64_t lo = (int64_t)blockIdx.x * kFoldTile;
#pragma unroll
    for (int i = 0; i < kFoldPer; ++i) {
        const int64_t p = lo + i * kFoldThreads + threadIdx.x;
        if (p < nnz) atomicAdd(&h[((uint32_t)key[p] >> shift) & dm], 1u);
    }
    __syncthreads();
    table[(int64_t)threadIdx.x * ntiles + blockIdx.x] = h[threadIdx.x];
}

// last row starting at or before nonzero p, among rows [lo, hi]
__device__ inline int64_t row_of(const int64_t* __restrict__ rp, int64_t lo, int64_t hi, int64_t p) {
    while (lo < hi) {
        const int64_t mid = (lo + hi + 1) >> 1;
        if (rp[mid] <= p) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// rows: nullptr on the first pass (they come from rp), else the moved rows
__global__ __launch_bounds__(kFoldThreads) void k_csc_move(int64_t N, int64_t nnz, const int64_t* __restrict__ rp,
                                                           const int32_t* __restrict__ key,
                                                           const int32_t* __restrict__ row,
                                                           const float* __restrict__ val, int shift, int nbits,
                                                           int64_t ntiles, const int64_t* __restrict__ table,
                                                           int32_t* __restrict__ okey, int32_t* __restrict__ orow,
                                                           float* __restrict__ oval) {
    __shared__ CscLds L;
    const int tid = threadIdx.x;
    const int64_t lo = (int64_t)blockIdx.x * kFoldTile;
    const int ne = (int)min((int64_t)kFoldTile, nnz - lo);
    int64_t ra = 0, rb = 0;
    if (!row) {
        ra = row_of(rp, 0, N - 1, lo);
        rb = row_of(rp, ra, N - 1, lo + ne - 1);
    }
#pragma unroll
    for (int i = 0; i < kFoldPer; ++i) {
        const int e = i * kFoldThreads + tid;
        if (e < ne) {
            L.key[e] = (uint32_t)key[lo + e];
            L.val[e] = val[lo + e];
            L.row[e] = row ? row[lo + e] : (int32_t)row_of(rp, ra, rb, lo + e);
        }
    }
    const int64_t first = table[(int64_t)tid * ntiles + blockIdx.x];
    __syncthreads();
    tile_radix(L.s, L.key, nullptr, L.order, ne, shift, nbits);
    L.at[tid] = first - L.s.base[tid];
    __syncthreads();
    const uint32_t dm = (1u << nbits) - 1u;
#pragma unroll
    for (int i = 0; i < kFoldPer; ++i) {
        const int s = i * kFoldThreads + tid;
        if (s < ne) {
            const int e = L.order[s];
            const int64_t to = L.at[(L.key[e] >> shift) & dm] + s;
            okey[to] = (int32_t)L.key[e];
            orow[to] = L.row[e];
            oval[to] = L.val[e];
        }
    }
}

// colptr[t] = first entry of column t (the columns are sorted)
__global__ void k_csc_ptr(int64_t d, int64_t nnz, const int32_t* __restrict__ key, int64_t* __restrict__ colptr) {
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (t > d) return;
    int64_t lo = 0, hi = nnz;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (key[mid] < t) lo = mid + 1;
        else hi = mid;
    }
    colptr[t] = lo;
}

int64_t csc_table_elems(int64_t nnz) { return ((nnz + kFoldTile - 1) / kFoldTile) * kFoldBins + 1; }

hipError_t build_csc(int64_t N, int64_t d, int64_t nnz, const int64_t* rp, const int32_t* col, const float* xv,
                     CscWs w, int64_t* colptr, const int32_t** rows, const float** vals, hipStream_t s) {
    int passes, nbits;
    tile_sort_plan(d, &passes, &nbits);
    const int64_t ntiles = (nnz + kFoldTile - 1) / kFoldTile;
    const int32_t *key = col, *row = nullptr;
    const float* val = xv;
    for (int p = 0; p < passes && ntiles > 0; ++p) {
        const int b = p & 1, shift = p * nbits;
        hipLaunchKernelGGL(k_csc_hist, dim3((unsigned)ntiles), dim3(kFoldThreads), 0, s, nnz, key, shift, nbits, ntiles,
                           w.count);
        const hipError_t e = exclusive_scan_i64(w.count, w.start, ntiles * kFoldBins, w.scan_ws, s);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_csc_move, dim3((unsigned)ntiles), dim3(kFoldThreads), 0, s, N, nnz, rp, key, row, val,
                           shift, nbits, ntiles, w.start, w.key[b], w.row[b], w.val[b]);
        key = w.key[b];
        row = w.row[b];
        val = w.val[b];
    }
    hipLaunchKernelGGL(k_csc_ptr, dim3((unsigned)((d + 256) / 256)), dim3(256), 0, s, d, nnz, key, colptr);
    *rows = row;
    *vals = val;
    return hipGetLastError();
}

}  // namespace sivf
