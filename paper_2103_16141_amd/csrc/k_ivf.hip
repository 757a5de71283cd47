// Structured inverted file of the centroids (Section 4; Alg. 5, "determine an
// inverted-file structure" and "make structured inverted-file").
//
// Device layout (one list per term, split by centroid tile for the LDS-tiled
// walk): postings are ordered by (term, tile, part, position) where part 0
// holds the moving centroids (flag 0) and part 1 the invariant ones.  With a
// single tile this is exactly the paper's per-term [moving | invariant] list.
// Positions renumber the centroids with the moving ones first, each group in
// ascending id (perm[q] = centroid at position q, iperm its inverse), and the
// tiles cover positions: a tile's moving centroids are a prefix of it, so an
// object that compares moving centroids only reads that prefix and skips the
// tiles past the last moving centroid.  Inside each part positions ascend
// with the ids, so per part the order is the paper's.
//   seg[t*T + tile]  start of segment (t, tile); its end is seg[t*T + tile + 1]
//   mid[t*T + tile]  length of the moving part of that segment
//   cid[p]           position minus tile*kt (16 bits)
//   v32/v16[p]       posting value, RN to f32 (or RNE of that to bf16)
//   v64[p]           the FP64 value (exact re-score over whole lists)
//
// Placement is deterministic without ordering atomics: a bitmap bm[w][t] marks
// which centroids hold term t; the rank of centroid j inside its (t, tile,
// part) segment is a popcount of lower bits, so every part comes out in
// ascending centroid id regardless of thread timing (Alg. 5 fills in ascending
// j the same way).
#include <algorithm>

#include "internal.h"
#include "slices.h"
#include "wave.h"

namespace sivf {

int64_t ivf_w64(int32_t k) { return ((int64_t)k + 63) / 64; }

// ---------------------------------------------------------------- positions
// One workgroup: position of every centroid (moving ones first, each group in
// ascending id), cscan = exclusive scan of the centroids' entry counts, and
// meta[0] = moving centroids, meta[1] = entries, meta[2] = 0 (head rows so far).
__global__ __launch_bounds__(1024) void k_ivf_perm(const uint8_t* __restrict__ lam, int32_t k,
                                                   const int64_t* __restrict__ nnz, int32_t* __restrict__ perm,
                                                   int32_t* __restrict__ iperm, int64_t* __restrict__ cscan,
                                                   int64_t* __restrict__ meta) {
    __shared__ int32_t sm[2][16];
    __shared__ int64_t sn[2][16];
    __shared__ int32_t stot[16];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    int32_t moving = 0;
    for (int64_t j = threadIdx.x; j < k; j += 1024) moving += lam[j] ? 0 : 1;
    moving = (int32_t)wave_sum_i64(moving);
    if (lane == 0) stot[wid] = moving;
    __syncthreads();
    int32_t nm = 0;
    for (int w = 0; w < 16; ++w) nm += stot[w];
    int32_t mcarry = 0;
    int64_t ncarry = 0;
    int buf = 0;
    for (int64_t b = 0; b < k; b += 1024, buf ^= 1) {
        const int64_t j = b + threadIdx.x;
        const bool mv = j < k && !lam[j];
        const int64_t n = j < k ? nnz[j] : 0;
        const unsigned long long mm = ballot(mv);
        const int64_t inc = wave_incl_scan_i64(n);
        if (lane == 63) {
            sm[buf][wid] = __popcll(mm);
            sn[buf][wid] = inc;
        }
        __syncthreads();
        int32_t before = mcarry + lanes_below(mm);
        int64_t nb = ncarry + inc - n;
        for (int w = 0; w < 16; ++w) {
            if (w < wid) {
                before += sm[buf][w];
                nb += sn[buf][w];
            }
            mcarry += sm[buf][w];
            ncarry += sn[buf][w];
        }
        if (j < k) {
            const int32_t q = mv ? before : nm + (int32_t)(j - before);
            iperm[j] = q;
            perm[q] = (int32_t)j;
            cscan[j] = nb;
        }
    }
    if (threadIdx.x == 0) {
        cscan[k] = ncarry;
        meta[0] = nm;
        meta[1] = ncarry;
        meta[2] = 0;
        meta[4] = 0;
        meta[5] = 0;
        meta[6] = 0;
    }
}

hipError_t ivf_perm(const uint8_t* lam, int32_t k, const int64_t* nnz, int32_t* perm, int32_t* iperm, int64_t* cscan,
                    int64_t* meta, hipStream_t s) {
    hipLaunchKernelGGL(k_ivf_perm, dim3(1), dim3(1024), 0, s, lam, k, nnz, perm, iperm, cscan, meta);
    return hipGetLastError();
}

// Calls f(centroid j, first entry's address, past the last, lane, lanes) for the
// entries of all centroids in pieces of kPiece consecutive ones per wave, wherever
// the centroids begin.  (A wave per centroid left 1,000 waves with 30,000 entries
// each: presence bits 0.57, file fill 2.07 ms at k = 1,000, D = 100,000; 0.25 and
// 1.14 in pieces.)
constexpr int kPiece = 256;

template <typename F>
__device__ inline void each_entry(const Store& st, int32_t k, const int64_t* __restrict__ cscan, F f) {
    const int64_t n = cscan[k], nw = ((int64_t)gridDim.x * blockDim.x) >> 6;
    const int64_t wave = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6;
    for (int64_t p0 = wave * kPiece; p0 < n; p0 += nw * kPiece)
        piece_entries(cscan, k, p0, min(n, p0 + kPiece), [&](int64_t j, int64_t a, int64_t e, int first, int step) {
            const int64_t b = st.start[j] - cscan[j];
            f(j, b + a, b + e, first, step);
        });
}

__global__ __launch_bounds__(256) void k_ivf_bits(Store st, int32_t k, int64_t d, const int64_t* __restrict__ cscan,
                                                  const int32_t* __restrict__ iperm,
                                                  unsigned long long* __restrict__ bm) {
    each_entry(st, k, cscan, [&](int64_t j, int64_t a, int64_t e, int first, int step) {
        const int64_t q = iperm[j];
        unsigned long long* row = bm + (q >> 6) * d;
        const unsigned long long bit = 1ull << (q & 63);
        for (int64_t p = a + first; p < e; p += step) {
            const int32_t t = st.term[p];
            if (t >= 0 && t < d) atomicOr(&row[t], bit);
        }
    });
}

// the moving positions (below n_moving) among word w's 64
__device__ inline unsigned long long moving_bits(int64_t w, int64_t n_moving) {
    const int64_t left = n_moving - w * 64;
    return left >= 64 ? ~0ull : left <= 0 ? 0ull : (1ull << left) - 1ull;
}

// One thread per (tile, term): per-word prefix counts inside the tile and the
// segment's part sizes.
__global__ void k_ivf_counts(const unsigned long long* __restrict__ bm, const int64_t* __restrict__ meta,
                             int64_t d, int32_t kt, int32_t T, int64_t W64, uint16_t* __restrict__ pre0,
                             uint16_t* __restrict__ pre1, int64_t* __restrict__ cnt) {
    int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (idx >= d * T) return;
    const int64_t tile = idx / d, t = idx - tile * d, nm = meta[0];
    const int64_t w0 = tile * (kt / 64);
    int64_t w1 = w0 + kt / 64;
    if (w1 > W64) w1 = W64;
    uint32_t c0 = 0, c1 = 0;
    for (int64_t w = w0; w < w1; ++w) {
        const unsigned long long m = bm[w * d + t], mv = moving_bits(w, nm);
        pre0[w * d + t] = (uint16_t)c0;
        pre1[w * d + t] = (uint16_t)c1;
        c0 += __popcll(m & mv);
        c1 += __popcll(m & ~mv);
    }
    cnt[(t * T + tile) * 2 + 0] = c0;
    cnt[(t * T + tile) * 2 + 1] = c1;
}

static unsigned entry_grid(int64_t bound) {
    return (unsigned)std::min<int64_t>(16384, std::max<int64_t>(1, (bound + 4 * kPiece - 1) / (4 * kPiece)));
}

hipError_t ivf_count(const Store st, int32_t k, int64_t d, int32_t kt, int32_t T, const int32_t* iperm,
                     const int64_t* cscan, const int64_t* meta, IvfBuildWs w, hipStream_t s) {
    const int64_t W64 = ivf_w64(k);
    hipError_t e = fill_u64(w.bm, 0ull, W64 * d, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_ivf_bits, dim3(entry_grid(st.cap)), dim3(256), 0, s, st, k, d, cscan, iperm, w.bm);
    int64_t nt = d * T;
    hipLaunchKernelGGL(k_ivf_counts, dim3((unsigned)((nt + 255) / 256)), dim3(256), 0, s, w.bm, meta, d, kt, T, W64,
                       w.pre0, w.pre1, w.cnt);
    return hipGetLastError();
}

// Segment bounds, and the dense head rows: a term whose lists hold at least
// min_len postings gets the next row (head[t], hterm[row]; the rows' order is
// that of the atomics and changes no result).  head == nullptr: no rows.
__global__ __launch_bounds__(256) void k_ivf_seg(const int64_t* __restrict__ off, const int64_t* __restrict__ cnt,
                                                 int64_t d, int32_t T, int64_t min_len, int64_t* __restrict__ seg,
                                                 int32_t* __restrict__ mid, int32_t* __restrict__ head,
                                                 int32_t* __restrict__ hterm, int64_t split_len,
                                                 int2* __restrict__ tlen, int32_t* __restrict__ srow,
                                                 int32_t* __restrict__ sterm, int64_t* __restrict__ meta) {
    const int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    const int64_t nt = d * T;
    if (idx < nt) {
        seg[idx] = off[idx * 2];
        mid[idx] = (int32_t)cnt[idx * 2];
    } else if (idx == nt) {
        seg[nt] = off[nt * 2];
    }
    if (!head) return;
    const bool term = idx < d;
    const int64_t len = term ? off[(idx + 1) * T * 2] - off[idx * T * 2] : 0;
    // the next row of a list for each lane whose term gets one
    auto take = [&](bool has, int64_t* count) -> int64_t {
        const unsigned long long m = ballot(has);
        int64_t row = 0;
        if (m) {
            if (lanes_below(m) == 0 && has) row = (int64_t)atomicAdd((unsigned long long*)count, (unsigned long long)__popcll(m));
            row = bcast_i64(row, __builtin_ctzll(m)) + lanes_below(m);
        }
        return row;
    };
    const bool hd = term && len >= min_len;
    const int64_t row = take(hd, &meta[2]);
    if (term) head[idx] = hd ? (int32_t)row : -1;
    if (hd) hterm[row] = (int32_t)idx;
    if (!srow) return;
    const bool sl = term && len >= split_len;
    const int64_t q = take(sl, &meta[4]);
    if (term) {
        int64_t mv = 0;
        for (int32_t tile = 0; tile < T; ++tile) mv += cnt[(idx * T + tile) * 2];
        tlen[idx] = make_int2((int)len, (int)mv);
        srow[idx] = sl ? (int32_t)q : -1;
    }
    if (sl) sterm[q] = (int32_t)idx;
}

hipError_t ivf_offsets(int64_t d, int32_t T, IvfBuildWs w, int64_t min_len, int64_t* seg, int32_t* mid, int32_t* head,
                       int32_t* hterm, int64_t split_len, int2* tlen, int32_t* srow, int32_t* sterm, int64_t* meta,
                       hipStream_t s) {
    const int64_t n = d * T * 2;
    hipError_t e = exclusive_scan_i64(w.cnt, w.off, n, w.scan_ws, s);
    if (e != hipSuccess) return e;
    int64_t nt = d * T + 1;
    hipLaunchKernelGGL(k_ivf_seg, dim3((unsigned)((nt + 255) / 256)), dim3(256), 0, s, w.off, w.cnt, d, T, min_len, seg,
                       mid, head, hterm, split_len, tlen, srow, sterm, meta);
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void k_ivf_fill(Store st, int32_t k, int64_t d, int32_t kt, int32_t T,
                                                  const int64_t* __restrict__ cscan,
                                                  const int32_t* __restrict__ iperm, int32_t n_moving,
                                                  const unsigned long long* __restrict__ bm,
                                                  const uint16_t* __restrict__ pre0, const uint16_t* __restrict__ pre1,
                                                  const int64_t* __restrict__ off, uint16_t* __restrict__ cid,
                                                  float* __restrict__ v32, uint16_t* __restrict__ v16,
                                                  double* __restrict__ v64) {
    each_entry(st, k, cscan, [&](int64_t j, int64_t a, int64_t e, int first, int step) {
        const int64_t q = iperm[j];
        const int part = q >= n_moving ? 1 : 0;
        const int64_t tile = q / kt, w = q >> 6;
        const unsigned long long mv = moving_bits(w, n_moving);
        const unsigned long long pm = (part ? ~mv : mv) & ((1ull << (q & 63)) - 1ull);
        const uint16_t* pre = part ? pre1 : pre0;
        const uint16_t local = (uint16_t)(q - tile * kt);
        for (int64_t p = a + first; p < e; p += step) {
            const int64_t t = st.term[p];
            const double u = st.val[p];
            const int64_t rank = pre[w * d + t] + __popcll(bm[w * d + t] & pm);
            const int64_t pos = off[(t * T + tile) * 2 + part] + rank;
            cid[pos] = local;
            const float f = (float)u;  // round to nearest even
            if (v32) v32[pos] = f;
            if (v16) v16[pos] = f32_to_bf16_rne(f);
            v64[pos] = u;
        }
    });
}

hipError_t ivf_fill(const Store st, int32_t k, int64_t d, int32_t kt, int32_t T, const int32_t* iperm,
                    const int64_t* cscan, int32_t n_moving, int64_t P, IvfBuildWs w, uint16_t* cid, float* v32,
                    uint16_t* v16, double* v64, hipStream_t s) {
    hipLaunchKernelGGL(k_ivf_fill, dim3(entry_grid(P)), dim3(256), 0, s, st, k, d, kt, T, cscan, iperm, n_moving, w.bm,
                       w.pre0, w.pre1, w.off, cid, v32, v16, v64);
    return hipGetLastError();
}

// ---------------------------------------------------------------- dense head rows
// A memory layout of this implementation (not the paper's): a term whose
// lists hold at least min_len postings gets a row of kpad = T * ktp values,
// one per position (zero where the centroid lacks the term), rounded to
// the posting dtype exactly as its postings are.  Rows are numbered by atomics (no
// result depends on it).  Each tile's kt centroids take ktp = kt rounded up to 512 slots.
// FP32 rows hold the tile's centroids in order.  BF16 rows interleave each
// 512-centroid block so that one 16-byte load gives a lane both of its
// 4-centroid groups: slots 8l..8l+3 hold centroids 4l..4l+3 of the block,
// slots 8l+4..8l+7 centroids 256+4l..256+4l+3.
// Slot of position c (0 <= c < ktp) inside a tile's part of a row.
__device__ inline int32_t tile_slot(int32_t c, bool bf16) {
    if (!bf16) return c;
    const int32_t i = c & 511;
    return (c & ~511) + 8 * ((i & 255) >> 2) + 4 * (i >> 8) + (i & 3);
}

// One workgroup per (row, tile): the tile's postings of the row's term are
// placed in LDS over zeros and the whole slice is written once, in order.
// (Zeroing all rows and scattering the centroids' entries into them, one write
// each: 0.74 ms at k = 1,000, D = 100,000; 0.015 now.)
__global__ __launch_bounds__(256) void k_head_rows(const int32_t* __restrict__ hterm, const int64_t* __restrict__ seg,
                                                   const uint16_t* __restrict__ cid, const float* __restrict__ v32,
                                                   const uint16_t* __restrict__ v16, int32_t T, int32_t ktp,
                                                   void* __restrict__ hval) {
    __shared__ float slot[kMaxTile];
    const int64_t r = blockIdx.x / T;
    const int tile = (int)(blockIdx.x - r * T);
    const int64_t t = hterm[r];
    const int64_t lo = seg[t * T + tile], hi = seg[t * T + tile + 1];
    for (int c = threadIdx.x; c < ktp; c += 256) slot[c] = 0.0f;
    __syncthreads();
    // slots hold the posting's bits: binary32, or bf16 in the low half
    for (int64_t p = lo + threadIdx.x; p < hi; p += 256)
        slot[tile_slot(cid[p], v16 != nullptr)] = v16 ? __uint_as_float(v16[p]) : v32[p];
    __syncthreads();
    const int64_t base = (r * T + tile) * ktp;
    if (v16) {
        uint32_t* out = (uint32_t*)hval + base / 2;
        for (int c = threadIdx.x; c < ktp / 2; c += 256)
            out[c] = __float_as_uint(slot[2 * c]) | (__float_as_uint(slot[2 * c + 1]) << 16);
    } else {
        float* out = (float*)hval + base;
        for (int c = threadIdx.x; c < ktp; c += 256) out[c] = slot[c];
    }
}

// Tile-major copy of the segment bounds for the walk: one 16-byte record per
// (tile, term) holding the segment start, its length and moving length (each
// at most kt <= 4096, so 16 bits apiece) and the term's dense head row (-1:
// none, or head == nullptr).  A launch over one tile then reads a 16*d-byte
// slice with one load per term instead of three scattered over the whole
// term-major table.
__global__ void k_seg_records(const int64_t* __restrict__ seg, const int32_t* __restrict__ mid,
                              const int32_t* __restrict__ head, int64_t d, int32_t T, uint4* __restrict__ rec) {
    const int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (idx >= d * T) return;
    const int64_t tile = idx / d, t = idx - tile * d;
    const int64_t s0 = seg[t * T + tile], len = seg[t * T + tile + 1] - s0;
    const uint32_t mv = (uint32_t)mid[t * T + tile];
    uint4 r;
    r.x = (uint32_t)(uint64_t)s0;
    r.y = (uint32_t)((uint64_t)s0 >> 32);
    r.z = (uint32_t)len | (mv << 16);
    r.w = (uint32_t)(head ? head[t] : -1);
    rec[idx] = r;
}

hipError_t seg_records(const int64_t* seg, const int32_t* mid, const int32_t* head, int64_t d, int32_t T, uint4* rec,
                       hipStream_t s) {
    const int64_t n = d * T;
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_seg_records, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, seg, mid, head, d, T, rec);
    return hipGetLastError();
}

hipError_t head_fill(const int32_t* hterm, const int64_t* seg, const uint16_t* cid, const float* v32,
                     const uint16_t* v16, int32_t T, int32_t ktp, int64_t H, void* hval, hipStream_t s) {
    const int64_t most = std::max<int64_t>(1, kMaxGroups / T);
    for (int64_t r = 0; r < H; r += most) {
        const int64_t n = std::min(most, H - r);
        void* to = v16 ? (void*)((uint16_t*)hval + r * T * ktp) : (void*)((float*)hval + r * T * ktp);
        hipLaunchKernelGGL(k_head_rows, dim3((unsigned)(n * T)), dim3(256), 0, s, hterm + r, seg, cid, v32, v16, T, ktp, to);
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------- sliced rows
// The split walk's rows: like dense head rows (FP32), but stored by blocks of
// 64 slots, [tile][block][row], 256-byte slices, so that a pass over one block
// reads one contiguous array of slices, whatever rows it needs.

// 1024 runs of 64 nonzeros
__global__ __launch_bounds__(256) void k_split_sample(const int32_t* __restrict__ col, int64_t nnz,
                                                      const int32_t* __restrict__ srow, int64_t* __restrict__ meta) {
    __shared__ int sh[4][2];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    int has = 0, all = 0;
    for (int q = 0; q < 4; ++q) {
        const int64_t run = (blockIdx.x * 4 + wid) * 4 + q, p = run * (nnz / 1024) + lane;
        const bool in = p < nnz;
        all += __popcll(ballot(in));
        has += __popcll(ballot(in && srow[col[in ? p : 0]] >= 0));
    }
    if (lane == 0) {
        sh[wid][0] = has;
        sh[wid][1] = all;
    }
    __syncthreads();
    if (threadIdx.x < 2)
        atomicAdd((unsigned long long*)&meta[5 + threadIdx.x],
                  (unsigned long long)(sh[0][threadIdx.x] + sh[1][threadIdx.x] + sh[2][threadIdx.x] + sh[3][threadIdx.x]));
}

hipError_t split_sample(const int32_t* col, int64_t nnz, const int32_t* srow, int64_t* meta, hipStream_t s) {
    hipLaunchKernelGGL(k_split_sample, dim3(64), dim3(256), 0, s, col, nnz, srow, meta);
    return hipGetLastError();
}

// sum of |values| of each row's postings (a fixed order), as ordered bits
__global__ __launch_bounds__(256) void k_split_weight(const int32_t* __restrict__ sterm, const int64_t* __restrict__ seg,
                                                     int32_t T, const float* __restrict__ v32, int64_t H,
                                                     uint32_t* __restrict__ wt) {
    const int lane = threadIdx.x & 63;
    const int64_t r = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6;
    if (r >= H) return;
    const int64_t t = sterm[r], lo = seg[t * T], hi = seg[(t + 1) * T];
    float acc = 0.0f;
    for (int64_t p = lo + lane; p < hi; p += 64) acc = acc + fabsf(v32[p]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) acc = acc + __shfl_xor(acc, o, 64);
    if (lane == 0) wt[r] = __float_as_uint(acc);
}

// One workgroup: the heaviest rows that fit LDS, numbered first.  The numbers
// inside the two groups come from atomics; they change no result.
__global__ __launch_bounds__(1024) void k_split_order(const uint32_t* __restrict__ wt, const int32_t* __restrict__ sterm,
                                                      int64_t H, int32_t* __restrict__ sterm2, int32_t* __restrict__ srow,
                                                      int64_t* __restrict__ meta) {
    __shared__ uint32_t sh[258];
    __shared__ uint32_t count, nh, nc;
    if (threadIdx.x == 0) count = nh = nc = 0;
    const uint32_t x = top_weights(wt, H, kSplitHot, sh);
    uint32_t hot = 0;
    each_weight(wt, H, [&](uint32_t v, int64_t) { hot += v >= x ? 1u : 0u; });
    hot = (uint32_t)wave_sum_i64(hot);
    if ((threadIdx.x & 63) == 0) atomicAdd(&count, hot);
    __syncthreads();
    hot = count;
    // a wave takes its lanes' numbers at once
    auto take = [&](bool has, uint32_t* c) -> uint32_t {
        const unsigned long long m = ballot(has);
        uint32_t at = 0;
        if (m && (threadIdx.x & 63) == 0) at = atomicAdd(c, (uint32_t)__popcll(m));
        return (uint32_t)__builtin_amdgcn_readfirstlane((int)at) + lanes_below(m);
    };
    each_weight(wt, H, [&](uint32_t v, int64_t r) {
        const bool h = r < H && v >= x, c = r < H && v < x;
        const uint32_t qh = take(h, &nh), qc = hot + take(c, &nc);
        if (!h && !c) return;
        const int32_t t = sterm[r];
        sterm2[h ? qh : qc] = t;
        srow[t] = (int32_t)(h ? qh : qc);
    });
    if (threadIdx.x == 0) meta[3] = hot;
}

hipError_t split_order(const int32_t* sterm, const int64_t* seg, int32_t T, const float* v32, int64_t H, uint32_t* wt, int32_t* sterm2, int32_t* srow, int64_t* meta,
                      hipStream_t s) {
    hipLaunchKernelGGL(k_split_weight, dim3((unsigned)((H + 3) / 4)), dim3(256), 0, s, sterm, seg, T, v32, H, wt);
    hipLaunchKernelGGL(k_split_order, dim3(1), dim3(1024), 0, s, wt, sterm, H, sterm2, srow, meta);
    return hipGetLastError();
}

// As k_head_rows: one workgroup per (row, tile).
__global__ __launch_bounds__(256) void k_split_rows(const int32_t* __restrict__ sterm, const int64_t* __restrict__ seg,
                                                    const uint16_t* __restrict__ cid, const float* __restrict__ v32,
                                                    int32_t T, int32_t ktp, int64_t H, float* __restrict__ sval) {
    __shared__ float slot[kMaxTile];
    const int64_t r = blockIdx.x / T;
    const int tile = (int)(blockIdx.x - r * T);
    const int64_t t = sterm[r];
    const int64_t lo = seg[t * T + tile], hi = seg[t * T + tile + 1];
    for (int c = threadIdx.x; c < ktp; c += 256) slot[c] = 0.0f;
    __syncthreads();
    for (int64_t p = lo + threadIdx.x; p < hi; p += 256) slot[cid[p]] = v32[p];
    __syncthreads();
    const int64_t b0 = (int64_t)tile * (ktp / kSliceCols);
    for (int c = threadIdx.x; c < ktp; c += 256)
        sval[((b0 + c / kSliceCols) * H + r) * kSliceCols + c % kSliceCols] = slot[c];
}

hipError_t split_fill(const int32_t* sterm2, const int64_t* seg, const uint16_t* cid, const float* v32, int32_t T,
                      int32_t ktp, int64_t H, void* sval, hipStream_t s) {
    hipLaunchKernelGGL(k_split_rows, dim3((unsigned)(H * T)), dim3(256), 0, s, sterm2, seg, cid, v32, T, ktp, H,
                       (float*)sval);
    return hipGetLastError();
}

// ---------------------------------------------------------------- export to the paper's layout
__global__ void k_exp_counts(const int64_t* __restrict__ seg, const int32_t* __restrict__ mid, int64_t d, int32_t T,
                             int64_t* __restrict__ cnt, int32_t* __restrict__ split) {
    int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (t >= d) return;
    cnt[t] = seg[(t + 1) * T] - seg[t * T];
    int64_t sp = 0;
    for (int32_t tile = 0; tile < T; ++tile) sp += mid[t * T + tile];
    if (split) split[t] = (int32_t)sp;
}

__global__ void k_exp_fill(const int64_t* __restrict__ seg, const int32_t* __restrict__ mid,
                           const uint16_t* __restrict__ cid, const double* __restrict__ v64, int64_t d, int32_t T,
                           int32_t kt, const int32_t* __restrict__ perm, const int64_t* __restrict__ tptr,
                           int32_t* __restrict__ p_cid,
                           double* __restrict__ p_val) {
    const int lane = threadIdx.x & 63;
    const int64_t wave = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6;
    const int64_t nw = ((int64_t)gridDim.x * blockDim.x) >> 6;
    for (int64_t t = wave; t < d; t += nw) {
        int64_t o = tptr[t];
        for (int part = 0; part < 2; ++part) {
            for (int32_t tile = 0; tile < T; ++tile) {
                int64_t s0 = seg[t * T + tile], s1 = seg[t * T + tile + 1], sm = s0 + mid[t * T + tile];
                int64_t lo = part ? sm : s0, hi = part ? s1 : sm;
                for (int64_t p = lo + lane; p < hi; p += 64) {
                    if (p_cid) p_cid[o + (p - lo)] = perm[(int32_t)cid[p] + tile * kt];
                    if (p_val) p_val[o + (p - lo)] = v64[p];
                }
                o += hi - lo;
            }
        }
    }
}

hipError_t ivf_export(const sivf_ivf* f, int64_t* term_ptr, int32_t* split, int32_t* p_cid, double* p_val,
                      int64_t* ws_counts, int64_t* scan_ws, hipStream_t s) {
    const int64_t d = f->d;
    hipLaunchKernelGGL(k_exp_counts, dim3((unsigned)((d + 255) / 256)), dim3(256), 0, s, f->seg, f->mid, d, f->T,
                       ws_counts, split);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (!term_ptr) return hipSuccess;
    e = exclusive_scan_i64(ws_counts, term_ptr, d, scan_ws, s);
    if (e != hipSuccess) return e;
    if (!p_cid && !p_val) return hipSuccess;
    int64_t blocks = (d * 64 + 255) / 256;
    if (blocks > 16384) blocks = 16384;
    hipLaunchKernelGGL(k_exp_fill, dim3((unsigned)blocks), dim3(256), 0, s, f->seg, f->mid, f->cid, f->v64, d, f->T,
                       f->kt, f->perm, term_ptr, p_cid, p_val);
    return hipGetLastError();
}

}  // namespace sivf
