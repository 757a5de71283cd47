// Update step (Alg. 1 update; Alg. 5 mean computation) on CDNA.
//
// 1. Stable radix sort of the objects by cluster (sort.h): every cluster's
//    members in ascending object id.  (Per-block histograms and a bitonic sort
//    of 4,096 objects per workgroup took 115 us for 10,000 objects and 0.46 ms
//    for 1M at k = 1,000; this takes 30 us and 0.1 ms.)
// 2. One workgroup per cluster sums its members' values term by term in
//    ascending object id (k_upd_fold: tiles of nonzeros sorted by term in
//    LDS; k_upd_members: row by row), q_t = w_t / |C_j|, support = {t : q_t != 0}; then s = s + q_t*q_t
//    sequentially in ascending term order and u_t = q_t / sqrt(s)
//    (k_upd_norm).  Clusters with no members, or with unchanged members
//    (flag 1), keep their previous centroid bitwise (it would be recomputed
//    to the same bits).
#include <algorithm>

#include "internal.h"
#include "sort.h"
#include "tile_sort.h"
#include "wave.h"

#pragma clang fp contract(off)

namespace sivf {

// cluster sizes and member row lengths from the sorted objects: one workgroup
// per cluster
__global__ __launch_bounds__(256) void k_upd_sizes(int32_t k, const int64_t* __restrict__ cstart,
                                                   const int32_t* __restrict__ perm, const int64_t* __restrict__ rp,
                                                   int64_t* __restrict__ ccount, int64_t* __restrict__ memnnz) {
    __shared__ int64_t sh[4];
    for (int64_t j = blockIdx.x; j < k; j += gridDim.x) {
        const int64_t q0 = cstart[j], q1 = cstart[j + 1];
        int64_t n = 0;
        for (int64_t q = q0 + threadIdx.x; q < q1; q += 256) {
            const int64_t i = perm[q];
            n += rp[i + 1] - rp[i];
        }
        n = wave_sum_i64(n);
        __syncthreads();
        if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = n;
        __syncthreads();
        if (threadIdx.x == 0) {
            ccount[j] = q1 - q0;
            memnnz[j] = (sh[0] + sh[1]) + (sh[2] + sh[3]);
        }
    }
}

hipError_t upd_sort(const int32_t* a, int64_t n, int32_t k, const int64_t* rp, const SortWs<float>& sw, UpdateWs* w,
                    hipStream_t s) {
    SortIn<float> in{};
    in.kind = kSortIota;
    in.n = n;
    in.key = a;
    const int32_t* key = nullptr;
    const float* none = nullptr;
    hipError_t e = sort_entries(in, k, sw, &key, &w->perm, &none, s);
    if (e == hipSuccess) e = sort_starts(key, n, k, w->cstart, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_upd_sizes, dim3((unsigned)std::min<int64_t>(k, 65536)), dim3(256), 0, s, k, w->cstart, w->perm,
                       rp, w->ccount, w->memnnz);
    return hipGetLastError();
}

// Entry bound per cluster, and the plan of the member sums: a cluster of at
// least kFoldBigTiles tiles that holds more than 1 / kFoldBig of all nonzeros
// (half a workgroup's share: fewer than kFoldBig clusters can) is cut into
// term ranges that run side by side: up to kFoldRanges, a tile and about 8
// nonzeros of a row each.  members: see upd_members.
__global__ void k_upd_bounds(int32_t k, int64_t d, int64_t nnz_all, int64_t members, const uint8_t* __restrict__ lam,
                             int allow_copy, Store prev, UpdateWs w) {
    const int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (j >= k) return;
    const int64_t cnt = w.ccount[j], nnz = w.memnnz[j];
    const bool copy = cnt == 0 || (allow_copy && lam[j]);
    w.ub[j] = copy ? prev.nnz[j] : min(d, nnz);
    int32_t slot = -1;
    if (!copy && nnz > kFoldTile && cnt <= members) {
        slot = kByMembers;
    } else if (!copy && nnz >= (int64_t)kFoldBigTiles * kFoldTile && nnz > nnz_all / kFoldBig) {
        const int64_t R = min(min((int64_t)kFoldRanges, nnz / kFoldTile), nnz / (8 * cnt));
        if (R >= 2) {
            const unsigned long long b = atomicAdd(&w.work[1], 1ull);
            if (b < (unsigned long long)kFoldBig) {
                slot = (int32_t)b;
                w.bigc[slot] = (int32_t)j;
                w.bigr[slot] = (int32_t)R;
                const unsigned long long at = atomicAdd(&w.work[2], (unsigned long long)R);
                for (int r = 0; r < R; ++r) w.jobs[at + r] = slot * kFoldRanges + r;
            }
        }
    }
    w.bigslot[j] = slot;
}

hipError_t upd_bounds(int32_t k, int64_t n, int64_t d, int64_t nnz, const uint8_t* lam, int allow_copy, const Store prev,
                      UpdateWs w, hipStream_t s) {
    hipError_t e = fill_u64(w.work, 0ull, 3, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_upd_bounds, dim3((unsigned)((k + 255) / 256)), dim3(256), 0, s, k, d, nnz,
                       upd_members(n, nnz, d, k), lam, allow_copy, prev, w);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    return exclusive_scan_i64(w.ub, w.ubscan, k, w.scan_ws, s);
}

// ---------------------------------------------------------------------------
// Member sums.  The order of the additions is part of the result: w_t adds the
// members' values in ascending object id.  Only additions to the same term are
// ordered, so a workgroup takes kFoldTile nonzeros of a cluster's members at a
// time (in member order), sorts them stably by term in LDS (radix passes of at
// most 9 bits), and every run of one term is folded by a thread of its own, in
// member order:
//   * a cluster of at most kFoldTile nonzeros is done after one tile;
//   * a longer one carries its sums from tile to tile in a dense FP64 row of
//     the workgroup (d doubles), one read and one write per term and tile, and
//     marks the terms it touched in a bitmap; the touched terms are emitted in
//     ascending order at the end, the row and the bitmap are cleared as read.
// What bounds it: the sort's LDS passes and their barriers.  Folding member by
// member (a wave per cluster, each member waiting for the previous one's sums)
// was bound by that chain, about 7 us a member: N = 1M, k = 1,000, D = 100,000
// 14.7 -> 3.1 ms; N = 2M, k = 10,000, D = 140,000 19.7 -> 7.5 ms.
// Cluster sizes are uneven (the largest of these has 14 times the mean), so
// large clusters are cut into term ranges that run side by side (k_upd_split);
// whole, the largest one alone held the kernel to 11 ms at N = 1M.
// 4,096 nonzeros and 512 threads keep two workgroups on a CU (58 KB of LDS each
// with FP32 values).

template <typename V>
struct FoldLds {
    uint32_t key[kFoldTile];         // terms by position (member order)
    V val[kFoldTile + 4];            // values, by position, then in sorted order
    uint16_t ia[kFoldTile + 8];      // positions in sorted order, double-buffered
    uint16_t ib[kFoldTile + 8];
    TileSortLds s;
    int64_t rb[kFoldThreads];        // first nonzero of each member of the tile
    int32_t pre[kFoldThreads + 1];   // its position in the tile
    int32_t wcnt[kFoldTile / 64];
    int64_t job;
    int32_t nskip;
};

// Positions of the flagged entries among all flagged ones, in entry order:
// entry (i, thread) is number i * kFoldThreads + threadIdx.x; mask[i] is the
// wave's flag mask of window i.  base[i] + lanes_below(mask[i]) is the
// position.  Returns the total.
__device__ inline int32_t fold_compact(const unsigned long long (&mask)[kFoldPer], int32_t (&base)[kFoldPer],
                                       int32_t* wcnt) {
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    __syncthreads();   // wcnt free
    if (lane == 0) {
#pragma unroll
        for (int i = 0; i < kFoldPer; ++i) wcnt[i * kFoldWaves + wid] = __popcll(mask[i]);
    }
    __syncthreads();
    static_assert(kFoldTile / 64 == 64, "one window count per lane");
    const int32_t c = wcnt[lane];
    const int32_t inc = wave_incl_scan_i32(c);
#pragma unroll
    for (int i = 0; i < kFoldPer; ++i) base[i] = __shfl(inc - c, i * kFoldWaves + wid, 64);
    return __shfl(inc, 63, 64);
}

// first entry in [lo, hi) of an ascending row whose column is >= t
__device__ inline int64_t row_lower(const int32_t* __restrict__ col, int64_t lo, int64_t hi, int64_t t) {
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (col[mid] < t) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// Stage the next nonzeros of up to kFoldThreads members: thread tid holds
// member tid's nonzeros [b, b + len) (len 0: none; more than kFoldTile counts
// as kFoldTile + 1).  Members are taken in order until kFoldTile nonzeros are
// in; the last one may be taken in part.  Returns the nonzeros staged;
// *ndone: members taken whole, *part: nonzeros taken of the next one.
template <typename V, bool VALUES>
__device__ inline int fold_stage(FoldLds<V>& L, const Csr& X, int64_t b, int32_t len, int* ndone, int* part) {
    const int tid = threadIdx.x;
    const V* __restrict__ xv = (const V*)X.val;
    int32_t total;
    const int32_t at = tile_scan(len, L.s.wsum, &total);
    L.rb[tid] = b;
    L.pre[tid] = at;
    if (tid == 0) {
        L.pre[kFoldThreads] = total;
        L.nskip = 0;
    }
    *ndone = __syncthreads_count(at + len <= kFoldTile);   // a prefix of the threads
    if (tid == *ndone) L.nskip = max(0, kFoldTile - at);
    const int ne = min(total, kFoldTile);
    uint32_t t[kFoldPer];
    V v[kFoldPer];
#pragma unroll
    for (int i = 0; i < kFoldPer; ++i) {
        const int s = i * kFoldThreads + tid;
        t[i] = 0u;
        v[i] = (V)0;
        if (s >= ne) continue;
        // last member starting at or before s (empty ones before it share its start)
        int lo = 0;
#pragma unroll
        for (int step = kFoldThreads / 2; step > 0; step >>= 1)
            if (L.pre[lo + step] <= s) lo += step;
        const int64_t p = L.rb[lo] + (s - L.pre[lo]);
        t[i] = (uint32_t)X.col[p];
        if (VALUES) v[i] = xv[p];
    }
#pragma unroll
    for (int i = 0; i < kFoldPer; ++i) {
        const int s = i * kFoldThreads + tid;
        L.key[s] = t[i];
        if (VALUES) L.val[s] = v[i];
    }
    __syncthreads();
    *part = L.nskip;
    return ne;
}

// Stable sort of the staged positions by term; returns the sorted order.
template <typename V>
__device__ inline const uint16_t* fold_sort(FoldLds<V>& L, int ne, int passes, int nbits) {
    const uint16_t* cur = nullptr;
    for (int ps = 0; ps < passes; ++ps) {
        uint16_t* dst = (ps & 1) ? L.ib : L.ia;
        tile_radix(L.s, L.key, cur, dst, ne, ps * nbits, nbits);
        cur = dst;
    }
    return cur;
}

// The touched terms (bits) of the sums W in ascending order: q_t = w_t / dc
// where not zero into next at o.  W and bits are left zero.  Returns the
// entries written.  Every mark must be in memory, the whole workgroup calls.
template <typename V>
__device__ inline int64_t fold_emit(FoldLds<V>& L, double* W, unsigned long long* bits, int64_t d, double dc,
                                    const Store& next, int64_t o) {
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int tid = threadIdx.x;
    const int64_t nwords = (d + 63) / 64;
    int64_t eo = 0;
    for (int64_t wb = 0; wb < nwords; wb += kFoldThreads) {
        unsigned long long word = 0;
        if (wb + tid < nwords) word = atomicExch(&bits[wb + tid], 0ull);
        int32_t total;
        const int32_t at = tile_scan(__popcll(word), L.s.wsum, &total);
        if (total == 0) continue;   // workgroup-uniform
        // at most kFoldTile terms at a time: all words, or one wave's 64 words
        const int nsub = total <= kFoldTile ? 1 : kFoldWaves;
        for (int sub = 0; sub < nsub; ++sub) {
            int32_t from = 0, n = total;
            if (nsub > 1) {
                for (int x = 0; x < sub; ++x) from += L.s.wsum[x];
                n = L.s.wsum[sub];
            }
            if (nsub == 1 || wid == sub) {
                int p = at - from;
                while (word) {
                    L.key[p++] = (uint32_t)((wb + tid) * 64 + __builtin_ctzll(word));
                    word &= word - 1;
                }
            }
            __syncthreads();
            uint32_t t[kFoldPer];
            double acc[kFoldPer];
            unsigned long long mask[kFoldPer];
            int32_t base[kFoldPer];
#pragma unroll
            for (int i = 0; i < kFoldPer; ++i) {
                const int e = i * kFoldThreads + tid;
                t[i] = e < n ? L.key[e] : 0u;
                acc[i] = e < n ? W[t[i]] : 0.0;
            }
#pragma unroll
            for (int i = 0; i < kFoldPer; ++i) {
                const bool in = i * kFoldThreads + tid < n;
                if (in) W[t[i]] = 0.0;
                acc[i] = acc[i] / dc;
                mask[i] = ballot(in && acc[i] != 0.0);
            }
            const int32_t got = fold_compact(mask, base, L.wcnt);
#pragma unroll
            for (int i = 0; i < kFoldPer; ++i) {
                if ((mask[i] >> lane) & 1ull) {
                    const int64_t to = o + eo + base[i] + lanes_below(mask[i]);
                    next.term[to] = (int32_t)t[i];
                    next.val[to] = acc[i];
                }
            }
            eo += got;
            __syncthreads();
        }
    }
    return eo;
}

// Term ranges of the large clusters (k_upd_bounds lists them): the quantiles
// of a sample of at most kFoldTile member nonzeros, so the ranges hold about
// the same number of nonzeros whatever the terms' frequencies.
template <typename V>
__global__ __launch_bounds__(kFoldThreads) void k_upd_split(Csr X, UpdateWs w, int passes, int nbits) {
    extern __shared__ __align__(16) unsigned char fold_smem[];
    FoldLds<V>& L = *reinterpret_cast<FoldLds<V>*>(fold_smem);
    const int tid = threadIdx.x;
    const int nbig = min((int)w.work[1], kFoldBig);
    for (int slot = blockIdx.x; slot < nbig; slot += gridDim.x) {
        const int64_t j = w.bigc[slot], cnt = w.ccount[j];
        const int R = w.bigr[slot];
        // evenly spaced members, as many as fill a tile on average
        const int64_t want = kFoldTile * cnt / max((int64_t)1, w.memnnz[j]);
        const int nm = (int)max((int64_t)1, min(min((int64_t)kFoldThreads, cnt), want));
        int64_t b = 0;
        int32_t len = 0;
        if (tid < nm) {
            const int64_t i = w.perm[w.cstart[j] + tid * cnt / nm];
            b = X.rp[i];
            len = (int32_t)min((int64_t)kFoldTile + 1, X.rp[i + 1] - b);
        }
        int ndone, part;
        const int ne = fold_stage<V, false>(L, X, b, len, &ndone, &part);
        const uint16_t* cur = fold_sort(L, ne, passes, nbits);
        if (tid <= R)
            w.splits[slot * (kFoldRanges + 1) + tid] =
                tid == 0 ? 0 : tid == R ? (int32_t)min(X.d, (int64_t)INT32_MAX)
                                        : (ne ? (int32_t)L.key[cur[(int64_t)ne * tid / R]] : 0);
        __syncthreads();
    }
}

// Sums, means and supports of the recomputed clusters: q_t = w_t / |C_j| for
// the terms with q_t != 0, ascending, into next at the cluster's offset (not
// yet normalised; k_upd_norm follows).  Persistent workgroups take the ranges
// of the large clusters first (their sums stay in the cluster's row for
// k_upd_emit), then the other clusters whole.
template <typename V>
__global__ __launch_bounds__(kFoldThreads) __attribute__((amdgpu_waves_per_eu(4))) void k_upd_fold(
    Csr X, int32_t k, const uint8_t* __restrict__ lam, int allow_copy, Store next, UpdateWs w, int passes, int nbits) {
    extern __shared__ __align__(16) unsigned char fold_smem[];
    FoldLds<V>& L = *reinterpret_cast<FoldLds<V>*>(fold_smem);
    const int lane = threadIdx.x & 63;
    const int tid = threadIdx.x;
    const int64_t nwords = (X.d + 63) / 64;
    const int64_t njobs = min((int64_t)w.work[2], (int64_t)kFoldBig * kFoldRanges);
    for (;;) {
        __syncthreads();
        if (tid == 0) L.job = (int64_t)atomicAdd(w.work, 1ull);
        __syncthreads();
        const int64_t job = L.job;
        if (job >= njobs + k) break;
        int64_t j = job - njobs, row = blockIdx.x;   // the cluster, its row of sums
        int64_t t0 = 0, t1 = X.d;                    // its range of terms
        const bool ranged = job < njobs;
        if (ranged) {
            const int32_t code = w.jobs[job];
            const int slot = code / kFoldRanges, r = code - slot * kFoldRanges;
            j = w.bigc[slot];
            row = w.nslots + slot;
            t0 = w.splits[slot * (kFoldRanges + 1) + r];
            t1 = w.splits[slot * (kFoldRanges + 1) + r + 1];
            if (t0 >= t1) continue;
        } else if (w.bigslot[j] >= 0) {
            continue;
        }
        const int64_t cnt = w.ccount[j];
        if (cnt == 0 || (allow_copy && lam[j])) continue;
        double* W = w.W + row * X.d;
        unsigned long long* bits = w.touched + row * nwords;
        const double dc = (double)cnt;
        const int64_t q0 = w.cstart[j], o = w.ubscan[j];
        const bool single = !ranged && w.memnnz[j] <= kFoldTile && cnt <= kFoldThreads;
        int64_t m0 = 0, skip = 0;   // next member, nonzeros of it already taken
        bool first = true;
        int64_t eo = 0;
        // the nonzeros [mb, me) of member m0 + tid inside the range
        int64_t mb = 0, me = 0;
        auto fetch = [&]() {
            mb = me = 0;
            if (m0 + tid < cnt) {
                const int64_t i = w.perm[q0 + m0 + tid];
                me = X.rp[i + 1];
                mb = X.rp[i];
                if (ranged) {
                    if (t1 < X.d) me = row_lower(X.col, mb, me, t1);
                    if (t0 > 0) mb = row_lower(X.col, mb, me, t0);
                }
                if (tid == 0) mb += skip;
            }
        };
        fetch();
        while (m0 < cnt) {
            int ndone, part;
            const int ne = fold_stage<V, true>(L, X, mb, (int32_t)min((int64_t)kFoldTile + 1, me - mb), &ndone, &part);
            // threads past the last member count as done
            skip = ndone < kFoldThreads ? (ndone == 0 ? skip : 0) + part : 0;
            m0 += ndone;
            fetch();   // the next tile's members, ahead of this one's sort
            if (ne == 0) continue;
            const uint16_t* cur = fold_sort(L, ne, passes, nbits);
            uint16_t* hp = cur == L.ia ? L.ib : L.ia;   // first sorted position of each run
            // ---- runs of one term, their values moved into sorted order
            unsigned long long mask[kFoldPer];
            int32_t base[kFoldPer];
            V sv[kFoldPer];
#pragma unroll
            for (int i = 0; i < kFoldPer; ++i) {
                const int s = i * kFoldThreads + tid;
                bool hd = false;
                sv[i] = (V)0;
                if (s < ne) {
                    const int c = cur[s];
                    hd = s == 0 || L.key[c] != L.key[cur[s - 1]];
                    sv[i] = L.val[c];
                }
                mask[i] = ballot(hd);
            }
            const int nrun = fold_compact(mask, base, L.wcnt);   // its barriers end the reads of val
#pragma unroll
            for (int i = 0; i < kFoldPer; ++i) {
                L.val[i * kFoldThreads + tid] = sv[i];
                if ((mask[i] >> lane) & 1ull) hp[base[i] + lanes_below(mask[i])] = (uint16_t)(i * kFoldThreads + tid);
            }
            if (tid == 0) hp[nrun] = (uint16_t)ne;
            __syncthreads();
            // ---- fold every run onto the sum carried so far
            uint32_t t[kFoldPer];
            double acc[kFoldPer];
#pragma unroll
            for (int i = 0; i < kFoldPer; ++i) {
                const int r = i * kFoldThreads + tid;
                t[i] = r < nrun ? L.key[cur[hp[r]]] : 0u;
                acc[i] = !first && r < nrun ? W[t[i]] : 0.0;
            }
#pragma unroll
            for (int i = 0; i < kFoldPer; ++i) {
                const int r = i * kFoldThreads + tid;
                if (r >= nrun) continue;
                const bool fresh = acc[i] == 0.0;
                const int s1 = hp[r + 1];
                double a = acc[i];
                for (int s = hp[r]; s < s1; s += 4) {
                    V x[4];   // reads past the run stay inside the tile's padding
#pragma unroll
                    for (int u = 0; u < 4; ++u) x[u] = L.val[s + u];
                    a = a + (double)x[0];
#pragma unroll
                    for (int u = 1; u < 4; ++u) {
                        const double n = a + (double)x[u];
                        a = s + u < s1 ? n : a;
                    }
                }
                acc[i] = a;
                if (!single) {
                    W[t[i]] = a;
                    if (fresh) atomicOr(&bits[t[i] >> 6], 1ull << (t[i] & 63));
                }
            }
            first = false;
            if (single) {
                // ---- the only tile: emit from registers
#pragma unroll
                for (int i = 0; i < kFoldPer; ++i) {
                    acc[i] = acc[i] / dc;
                    mask[i] = ballot(i * kFoldThreads + tid < nrun && acc[i] != 0.0);
                }
                eo = fold_compact(mask, base, L.wcnt);
#pragma unroll
                for (int i = 0; i < kFoldPer; ++i) {
                    if ((mask[i] >> lane) & 1ull) {
                        const int64_t at = o + base[i] + lanes_below(mask[i]);
                        next.term[at] = (int32_t)t[i];
                        next.val[at] = acc[i];
                    }
                }
            }
            __syncthreads();
        }
        if (ranged) continue;
        if (!single) {
            __threadfence();   // every mark in memory before the words are taken
            __syncthreads();
            eo = fold_emit(L, W, bits, X.d, dc, next, o);
        }
        if (tid == 0) {
            next.start[j] = o;
            next.nnz[j] = eo;
        }
    }
}

// the large clusters' entries, from their rows of sums
__global__ __launch_bounds__(kFoldThreads) void k_upd_emit(int64_t d, Store next, UpdateWs w) {
    __shared__ FoldLds<float> L;
    const int nbig = min((int)w.work[1], kFoldBig);
    for (int slot = blockIdx.x; slot < nbig; slot += gridDim.x) {
        const int64_t j = w.bigc[slot], row = w.nslots + slot, o = w.ubscan[j];
        __syncthreads();
        const int64_t eo = fold_emit(L, w.W + row * d, w.touched + row * ((d + 63) / 64), d, (double)w.ccount[j], next, o);
        if (threadIdx.x == 0) {
            next.start[j] = o;
            next.nnz[j] = eo;
        }
    }
}

// Clusters of more than a tile and few members over a vocabulary whose FP64 sums
// fit LDS: a wave each adds its members' rows one after the other (a row's terms
// are distinct, and a wave's LDS operations complete in order), then emits the
// sums in ascending order.  Bound by that chain, 0.4 us a member with the bounds of
// 64 members and the nonzeros of the next one loaded ahead, instead of by the sort's
// passes: 400,000 rows of 200 of 4,000 terms, k = 3,000 (130 members a cluster) whole
// update 2.71 -> 1.33 ms.
template <typename V>
__global__ __launch_bounds__(64) void k_upd_members(Csr X, int32_t k, Store next, UpdateWs w) {
    extern __shared__ double sums[];   // zero between clusters
    constexpr int kAhead = 4;          // 64 nonzeros each
    const int lane = threadIdx.x;
    const V* __restrict__ xv = (const V*)X.val;
    for (int64_t t = lane; t < X.d; t += 64) sums[t] = 0.0;
    for (int64_t j = blockIdx.x; j < k; j += gridDim.x) {
        if (w.bigslot[j] != kByMembers) continue;
        const int64_t cnt = w.ccount[j], q0 = w.cstart[j], o = w.ubscan[j];
        for (int64_t m0 = 0; m0 < cnt; m0 += 64) {
            int64_t mb = 0, me = 0;   // of member m0 + lane
            if (m0 + lane < cnt) {
                const int64_t i = w.perm[q0 + m0 + lane];
                mb = X.rp[i];
                me = X.rp[i + 1];
            }
            const int nm = (int)min((int64_t)64, cnt - m0);
            int32_t t[kAhead], tn[kAhead];
            V v[kAhead], vn[kAhead];
            // unconditional loads: a branch would wait for them
            auto load = [&](int m, int32_t (&tt)[kAhead], V (&vv)[kAhead]) {
                const int64_t b = bcast_i64(mb, m), e = bcast_i64(me, m);
#pragma unroll
                for (int c = 0; c < kAhead; ++c) {
                    const int64_t p = b + c * 64 + lane, at = min(p, X.nnz - 1);
                    const int32_t col = X.col[at];
                    vv[c] = xv[at];
                    tt[c] = p < e ? col : -1;
                }
            };
            load(0, t, v);
            for (int m = 0; m < nm; ++m) {
                load(min(m + 1, nm - 1), tn, vn);
                double a[kAhead];
#pragma unroll
                for (int c = 0; c < kAhead; ++c) a[c] = sums[max(t[c], 0)];
#pragma unroll
                for (int c = 0; c < kAhead; ++c)
                    if (t[c] >= 0) sums[t[c]] = a[c] + (double)v[c];
                const int64_t e = bcast_i64(me, m);
                for (int64_t p = bcast_i64(mb, m) + kAhead * 64 + lane; p < e; p += 64)
                    sums[X.col[p]] = sums[X.col[p]] + (double)xv[p];
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int c = 0; c < kAhead; ++c) {
                    t[c] = tn[c];
                    v[c] = vn[c];
                }
            }
        }
        const double dc = (double)cnt;
        int64_t eo = 0;
        for (int64_t p0 = 0; p0 < X.d; p0 += 64) {
            const int64_t p = p0 + lane;
            const double q = p < X.d ? sums[p] / dc : 0.0;
            if (p < X.d) sums[p] = 0.0;
            const unsigned long long mask = ballot(q != 0.0);
            if (q != 0.0) {
                const int64_t at = o + eo + lanes_below(mask);
                next.term[at] = (int32_t)p;
                next.val[at] = q;
            }
            eo += __popcll(mask);
        }
        if (lane == 0) {
            next.start[j] = o;
            next.nnz[j] = eo;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
}

// u_t = q_t / sqrt(s) with s = s + q_t * q_t sequentially in ascending t, or a
// copy of the previous centroid for unchanged and empty clusters; and the
// centroid's norm bound (as k_centroid_norms).  One workgroup per cluster: all
// waves square kNormChunk values into LDS, the first wave folds the previous
// chunk, every lane reading the same squares (16-byte broadcasts, 16 ahead).
// Bound: the dependent FP64 additions of the longest centroid.  Against lane
// reads of the squares out of registers: 0.98 -> 0.61 ms at N = 1M, k = 1,000.
constexpr int kNormChunk = 1024;

__global__ __launch_bounds__(256) void k_upd_norm(int32_t k, const uint8_t* __restrict__ lam, int allow_copy,
                                                  Store prev, Store next, UpdateWs w, double* __restrict__ cnorm) {
    __shared__ alignas(16) double sq[2][kNormChunk];
    __shared__ double sh_nr;
    __shared__ double sh_part[4];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    for (int64_t j = blockIdx.x; j < k; j += gridDim.x) {
        const bool copy = w.ccount[j] == 0 || (allow_copy && lam[j]);
        int64_t o, m;
        double part = 0.0;
        if (copy) {
            const int64_t ps = prev.start[j];
            o = w.ubscan[j];
            m = prev.nnz[j];
            for (int64_t p = threadIdx.x; p < m; p += 256) {
                const double u = prev.val[ps + p];
                next.term[o + p] = prev.term[ps + p];
                next.val[o + p] = u;
                part = part + u * u;
            }
            if (threadIdx.x == 0) {
                next.start[j] = o;
                next.nnz[j] = m;
            }
        } else {
            o = next.start[j];
            m = next.nnz[j];
            double s = 0.0;
            int buf = 0;
            for (int64_t p0 = 0; p0 < m + kNormChunk; p0 += kNormChunk, buf ^= 1) {
                if (p0 < m) {
#pragma unroll
                    for (int u = 0; u < kNormChunk / 256; ++u) {
                        const int64_t p = p0 + u * 256 + threadIdx.x;
                        const double v = p < m ? next.val[o + p] : 0.0;   // + 0.0 leaves the sum as it is
                        sq[buf][u * 256 + threadIdx.x] = v * v;
                    }
                }
                if (wid == 0 && p0 > 0) {
                    const double2* q = reinterpret_cast<const double2*>(sq[buf ^ 1]);
                    const int n = (int)min((int64_t)kNormChunk, m - (p0 - kNormChunk));
                    double2 x[8], y[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) x[u] = q[u];
                    for (int b = 0; b < n; b += 32) {
#pragma unroll
                        for (int u = 0; u < 8; ++u) y[u] = q[b / 2 + 8 + u];
#pragma unroll
                        for (int u = 0; u < 8; ++u) {
                            s = s + x[u].x;
                            s = s + x[u].y;
                        }
                        const int nb = b + 32 < kNormChunk ? b + 32 : 0;
#pragma unroll
                        for (int u = 0; u < 8; ++u) x[u] = q[nb / 2 + u];
#pragma unroll
                        for (int u = 0; u < 8; ++u) {
                            s = s + y[u].x;
                            s = s + y[u].y;
                        }
                    }
                }
                __syncthreads();
            }
            if (threadIdx.x == 0) sh_nr = sqrt(s);
            __syncthreads();
            const double nr = sh_nr;
            for (int64_t p = threadIdx.x; p < m; p += 256) {
                const double u = next.val[o + p] / nr;
                next.val[o + p] = u;
                part = part + u * u;
            }
        }
        part = wave_sum_f64(part);
        if (lane == 0) sh_part[wid] = part;
        __syncthreads();
        if (threadIdx.x == 0) cnorm[j] = centroid_norm_bound((sh_part[0] + sh_part[1]) + (sh_part[2] + sh_part[3]));
        __syncthreads();
    }
}

int upd_fold_groups(int n_cu) { return n_cu * 2; }

template <typename V>
static hipError_t upd_means_t(const Csr& X, int32_t k, const uint8_t* lam, int allow_copy, Store next,
                              const UpdateWs& w, hipStream_t s) {
    int passes, nbits;
    tile_sort_plan(X.d, &passes, &nbits);
    const unsigned groups = (unsigned)w.nslots;
    const size_t lds = sizeof(FoldLds<V>);
    if (lds > 65536) {
        for (const void* fn : {(const void*)k_upd_fold<V>, (const void*)k_upd_split<V>}) {
            const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            if (e != hipSuccess) return e;
        }
    }
    if (X.nnz >= (int64_t)kFoldBigTiles * kFoldTile)
        hipLaunchKernelGGL(k_upd_split<V>, dim3(kFoldBig), dim3(kFoldThreads), lds, s, X, w, passes, nbits);
    hipLaunchKernelGGL(k_upd_fold<V>, dim3(groups), dim3(kFoldThreads), lds, s, X, k, lam, allow_copy, next, w, passes,
                       nbits);
    if (upd_members(X.n, X.nnz, X.d, k) > 0) {
        const size_t room = (size_t)X.d * 8;
        int nb = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_upd_members<V>, 64, room) != hipSuccess || nb < 1) nb = 1;
        const unsigned waves = (unsigned)std::min<int64_t>(k, (int64_t)groups / 2 * nb);
        hipLaunchKernelGGL(k_upd_members<V>, dim3(waves), dim3(64), room, s, X, k, next, w);
    }
    if (X.nnz >= (int64_t)kFoldBigTiles * kFoldTile)
        hipLaunchKernelGGL(k_upd_emit, dim3(kFoldBig), dim3(kFoldThreads), 0, s, X.d, next, w);
    return hipGetLastError();
}

hipError_t upd_means(const Csr& X, int32_t k, const uint8_t* lam, int allow_copy, const Store prev, Store next,
                     UpdateWs w, double* cnorm, hipStream_t s) {
    hipError_t e = X.f64 ? upd_means_t<double>(X, k, lam, allow_copy, next, w, s)
                         : upd_means_t<float>(X, k, lam, allow_copy, next, w, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_upd_norm, dim3((unsigned)std::min<int64_t>(k, 1 << 16)), dim3(256), 0, s, k, lam, allow_copy,
                       prev, next, w, cnorm);
    return hipGetLastError();
}

}  // namespace sivf
