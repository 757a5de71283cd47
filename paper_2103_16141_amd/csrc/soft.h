// Declarations of the soft-assignment kernels (k_soft.hip) used by the C ABI.
#pragma once

#include <algorithm>

#include "internal.h"

namespace sivf {

constexpr int kSoftBlk = 64;     // columns of a C^T block
constexpr int kSoftSub = 32;     // columns of a dS / dC^T block
constexpr int kSoftPiece = 512;  // CSC entries a wave sums at most

// C (k x d) -> blocks [ceil(k / 64)][d][64] of C^T, zero past column k
hipError_t soft_pack(const float* C, float* out, int64_t k, int64_t d, hipStream_t s);
// blocks [2 ceil(k / 64)][d][32] of dC^T -> dC (k x d)
hipError_t soft_unpack(const float* dCT, float* dC, int64_t k, int64_t d, hipStream_t s);
struct SoftFwdWs {
    int64_t rows;    // rows per launch
    int64_t blocks;  // blocks of 64 columns in C^T at once
    float* CT;       // [64 * blocks * d]
    float* pmax;     // [ceil(k / 64) * rows] max of S / tau per (block, row)
    float* psum;     // [ceil(k / 64) * rows] sum of exp(S / tau - max)
    double* part;    // partial sums of lse: one per 256 rows of every launch
    // with the commonest terms in LDS (ent == nullptr: not)
    int64_t nnz;
    uint2* ent;      // [split_pairs(nnz, rows)] pairs of a launch's rows
    uint2* hdr;      // [rows]
    uint32_t* count; // [d] sampled nonzeros of each term
    int32_t *slot, *term, *nhot;   // [d], [kSplitHot], [1]
};
// rows per launch with the commonest terms in LDS, or 0: not so
int64_t soft_lds_rows(int64_t N, int64_t nnz, int64_t d, int32_t k);
hipError_t soft_forward(int64_t N, int64_t nnz, const int64_t* rp, const int32_t* col, const float* xv, const float* C, int64_t d,
                        int32_t k, float tau, float* lse, double* loss_dev, SoftFwdWs w, int n_cu, hipStream_t s);
// rows [c0, c1) whose nonzeros are [p0, p1), k columns of C^T.  dS: blocks
// [2 ceil(k / 64)][c1 - c0][32] or nullptr; dxv: dX or nullptr; dxp:
// [ceil(k / 64) * (p1 - p0)], or nullptr when k <= 64 are all columns; add: dX has
// the columns before these
hipError_t soft_bwd_rows(int64_t c0, int64_t c1, int64_t p0, int64_t p1, const int64_t* rp, const int32_t* col,
                         const float* xv, const float* CT, int64_t d, int32_t k, float tau, float grad,
                         const float* lse, float* dS, float* dxp, float* dxv, bool add, int n_cu, hipStream_t s);
// out[j] = rp[min(j * rc, n)] for j in [0, nch]: the nonzero offsets of the row chunks
hipError_t soft_chunk_offsets(const int64_t* rp, int64_t n, int64_t rc, int64_t nch, int64_t* out, hipStream_t s);
// workspace of the dC pass of one chunk of rows
struct DctWs {
    int64_t* next;        // [d] CSC entry the next chunk's range starts at (set by each)
    int64_t* lo;          // [d] first CSC entry of the chunk's rows
    int32_t* len;         // [d] entries
    int32_t* mid;         // [d] terms summed by a wave each
    int32_t* longt;       // [d] terms summed in pieces
    int64_t* longp;       // [d] their first piece
    int64_t* piece;       // [max_pieces] first CSC entry
    int32_t* piece_len;   // [max_pieces] entries
    float* part;          // [2 ceil(k / 64) * max_pieces * 32] partial rows
    int64_t max_pieces;   // at least the pieces of any chunk (nonzeros / (kSoftPiece / 2) suffice)
    unsigned long long* count;   // [4] mid terms, pieces, long terms, dS not finite; zero before every chunk
    // the densest terms by matrix products (xd == nullptr: not)
    int64_t nnz;          // of all rows
    float* xd;            // [rows * kDctDense] their values in the chunk's rows
    float* prod;          // [dct_prod_elems(rows, k)] partial products
    int32_t* slot;        // [d] of the densest terms, else -1 (set by dct_pick)
    int32_t* term;        // [kDctDense] its inverse
    int32_t* cand;        // [dct_cands(nonzeros, rows)] workspace of dct_pick
    uint32_t* cand_df;
    unsigned long long* ndense;   // [2] candidates, densest terms; zero before dct_pick
};
constexpr int kDctDense = 256;
// values of the partial products of a chunk of `rows` rows; terms dct_pick considers at most
int64_t dct_prod_elems(int64_t rows, int32_t k);
inline int64_t dct_cands(int64_t nnz, int64_t rows) { return 32 * (nnz / std::max<int64_t>(rows, 1) + 1); }
// the terms in at least 1/32 of N rows, at most kDctDense of them
hipError_t dct_pick(int64_t N, int64_t d, int32_t k, const int64_t* colptr, DctWs w, hipStream_t s);
// rows [c0, c1) of the densest terms into w.xd
hipError_t dct_dense_rows(int64_t c0, int64_t c1, const int64_t* rp, const int32_t* col, const float* xv, DctWs w,
                          int n_cu, hipStream_t s);
// first: dCT is overwritten; fresh: the chunk's ranges start at colptr (else at w.next)
hipError_t soft_dct(int64_t d, int32_t k, int64_t c0, int64_t c1, int first, int fresh, const int64_t* colptr,
                    const int32_t* xt_row, const float* xt_val, const float* dS, float* dCT, DctWs w, int n_cu,
                    hipStream_t s);

}  // namespace sivf
