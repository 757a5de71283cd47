// Utility kernels: device-wide exclusive scan, fills, CSR validation, and the
// centroid-store helpers (gather of initial rows, import from CSR, export,
// per-centroid norm bounds).
#include <algorithm>

#include "internal.h"
#include "wave.h"

#pragma clang fp contract(off)

namespace sivf {

// ---------------------------------------------------------------- fills
template <typename T>
__global__ void k_fill(T* __restrict__ p, T v, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

template <typename T>
static hipError_t fill_any(T* p, T v, int64_t n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    int64_t blocks = (n + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(k_fill<T>, dim3((unsigned)blocks), dim3(256), 0, s, p, v, n);
    return hipGetLastError();
}
hipError_t fill_u8(uint8_t* p, uint8_t v, int64_t n, hipStream_t s) { return fill_any(p, v, n, s); }
hipError_t fill_u64(unsigned long long* p, unsigned long long v, int64_t n, hipStream_t s) { return fill_any(p, v, n, s); }
hipError_t fill_i64(int64_t* p, int64_t v, int64_t n, hipStream_t s) { return fill_any(p, v, n, s); }
hipError_t fill_i32(int32_t* p, int32_t v, int64_t n, hipStream_t s) { return fill_any(p, v, n, s); }

// ---------------------------------------------------------------- scan
// out[i] = sum_{j < i} in[j] for i in [0, n], three phases: per-chunk totals,
// scan of the totals (one workgroup), per-chunk local scan plus carry-in.
constexpr int kScanThreads = 256;
constexpr int kScanPer = 16;
constexpr int kScanChunk = kScanThreads * kScanPer;

int64_t scan_ws_elems(int64_t n) { return (n + kScanChunk - 1) / kScanChunk + 1; }

__device__ inline int64_t block_excl_scan(int64_t v, int64_t* sh, int64_t* total) {
    // sh: kScanThreads/64 entries
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    int64_t inc = wave_incl_scan_i64(v);
    if (lane == 63) sh[wid] = inc;
    __syncthreads();
    int64_t off = 0, tot = 0;
    for (int w = 0; w < kScanThreads / 64; ++w) {
        int64_t x = sh[w];
        if (w < wid) off += x;
        tot += x;
    }
    __syncthreads();
    *total = tot;
    return off + inc - v;
}

__global__ void k_scan_totals(const int64_t* __restrict__ in, int64_t n, int64_t* __restrict__ bsum) {
    __shared__ int64_t sh[kScanThreads / 64];
    int64_t base = (int64_t)blockIdx.x * kScanChunk + (int64_t)threadIdx.x * kScanPer;
    int64_t acc = 0;
    for (int q = 0; q < kScanPer; ++q) {
        int64_t i = base + q;
        if (i < n) acc += in[i];
    }
    int64_t tot;
    block_excl_scan(acc, sh, &tot);
    if (threadIdx.x == 0) bsum[blockIdx.x] = tot;
}

__global__ void k_scan_bsum(int64_t* __restrict__ bsum, int64_t nb) {
    __shared__ int64_t sh[kScanThreads / 64];
    int64_t carry = 0;
    for (int64_t b0 = 0; b0 < nb; b0 += kScanThreads) {
        int64_t i = b0 + threadIdx.x;
        int64_t v = i < nb ? bsum[i] : 0;
        int64_t tot;
        int64_t ex = block_excl_scan(v, sh, &tot);
        if (i < nb) bsum[i] = carry + ex;
        carry += tot;
    }
    if (threadIdx.x == 0) bsum[nb] = carry;
}

__global__ void k_scan_apply(const int64_t* __restrict__ in, int64_t n, const int64_t* __restrict__ bsum,
                             int64_t nb, int64_t* __restrict__ out) {
    __shared__ int64_t sh[kScanThreads / 64];
    int64_t base = (int64_t)blockIdx.x * kScanChunk + (int64_t)threadIdx.x * kScanPer;
    int64_t loc[kScanPer];
    int64_t acc = 0;
    for (int q = 0; q < kScanPer; ++q) {
        int64_t i = base + q;
        loc[q] = i < n ? in[i] : 0;
        acc += loc[q];
    }
    int64_t tot;
    int64_t ex = block_excl_scan(acc, sh, &tot) + bsum[blockIdx.x];
    for (int q = 0; q < kScanPer; ++q) {
        int64_t i = base + q;
        if (i < n) out[i] = ex;
        ex += loc[q];
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) out[n] = bsum[nb];
}

// The whole scan by one workgroup: a launch costs more than a few more rounds
// (up to 16,384 elements: one launch of about 5 us for three of 4).
constexpr int64_t kScanSmall = 16384;

__global__ __launch_bounds__(1024) void k_scan_small(const int64_t* __restrict__ in, int64_t n, int64_t* __restrict__ out) {
    __shared__ int64_t sh[2][16];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    int64_t carry = 0;
    int buf = 0;
    for (int64_t b = 0; b < n; b += 4096, buf ^= 1) {
        const int64_t i0 = b + 4 * (int64_t)threadIdx.x;
        int64_t v[4], acc = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            v[q] = i0 + q < n ? in[i0 + q] : 0;
            acc += v[q];
        }
        const int64_t inc = wave_incl_scan_i64(acc);
        if (lane == 63) sh[buf][wid] = inc;
        __syncthreads();
        int64_t ex = carry + inc - acc;
        for (int w = 0; w < 16; ++w) {
            const int64_t x = sh[buf][w];
            if (w < wid) ex += x;
            carry += x;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (i0 + q < n) out[i0 + q] = ex;
            ex += v[q];
        }
    }
    if (threadIdx.x == 0) out[n] = carry;
}

hipError_t exclusive_scan_i64(const int64_t* in, int64_t* out, int64_t n, int64_t* bsum, hipStream_t s) {
    if (n <= 0) {
        hipLaunchKernelGGL(k_fill<int64_t>, dim3(1), dim3(64), 0, s, out, (int64_t)0, (int64_t)1);
        return hipGetLastError();
    }
    if (n <= kScanSmall) {
        hipLaunchKernelGGL(k_scan_small, dim3(1), dim3(1024), 0, s, in, n, out);
        return hipGetLastError();
    }
    int64_t nb = (n + kScanChunk - 1) / kScanChunk;
    hipLaunchKernelGGL(k_scan_totals, dim3((unsigned)nb), dim3(kScanThreads), 0, s, in, n, bsum);
    hipLaunchKernelGGL(k_scan_bsum, dim3(1), dim3(kScanThreads), 0, s, bsum, nb);
    hipLaunchKernelGGL(k_scan_apply, dim3((unsigned)nb), dim3(kScanThreads), 0, s, in, n, bsum, nb, out);
    return hipGetLastError();
}

// ---------------------------------------------------------------- validation
// flags[0]: bit0 unsorted/row_ptr decreasing, bit1 column out of range,
//           bit2 non-finite value, bit3 row_ptr inconsistent with nnz
// flags[1]: smallest offending row, complemented (0: none; k_validate_rows only)
// flags[2]: 1 if some value is negative
// flags[3]: descents of col that are not at the start of a row (0 if every
//           row's columns ascend strictly)
// All zero before the launch.
//
// The check is one pass over the nonzeros in memory order, independent of how
// they fall into rows, so a few long rows (a centroid matrix) and many short
// ones fill the chip alike.  A descent is a p >= 1 with col[p] <= col[p - 1].
// With consistent row bounds, rows ascend strictly exactly if every descent
// lies at the start of a (non-empty) row, so the pass counts all descents,
// takes away those at row starts, and the rows ascend iff nothing is left.
// The arrays hold row_ptr[n] nonzeros: no more are read if more are stated.
// Bound: one read of X.  Each thread takes 4 consecutive nonzeros (16-byte
// loads where the arrays allow).  Against one wave per 64 rows walking their
// nonzeros 64 at a time (32 waves for 2,000 long centroid rows), a restart of
// 200,000 objects, k = 2,000, takes 4.2 instead of 7.9 ms.
__device__ inline unsigned long long wave_or_u64(unsigned long long v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v |= __shfl_xor(v, o, 64);
    return v;
}

__device__ inline bool finite_bits(float v) { return (__float_as_uint(v) & 0x7f800000u) != 0x7f800000u; }
__device__ inline bool finite_bits(double v) {
    return ((unsigned)((unsigned long long)__double_as_longlong(v) >> 32) & 0x7ff00000u) != 0x7ff00000u;
}

// Workgroups are large because each adds its count to one word, 15 ns in turn: with
// 2,048 of 256 threads a whole check of 5,000,000 rows of one nonzero took 59 us, of
// 200,000 rows of 60 58; so 41 and 40.  Small inputs, whose groups are few, take
// 256 (the kernel, 256 and 1,024 threads: 8,000 nonzeros 3.1 and 3.3 us, 32,000 3.2
// and 3.7, 64,000 3.5 both, 130,000 4.0 and 3.7, 520,000 8.5 and 4.7).
template <typename V, int T>
__global__ __launch_bounds__(T) void k_validate(const int64_t* __restrict__ rp, const int32_t* __restrict__ col,
                                                const V* __restrict__ val, int64_t n, int64_t d, int64_t stated,
                                                int vec, unsigned long long* flags) {
    __shared__ int sh_diff[T / 64];
    __shared__ unsigned sh_bad[T / 64];
    const int64_t nnz = min(stated, rp[n]);   // negative: none
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int64_t t0 = blockIdx.x * (int64_t)blockDim.x + threadIdx.x, nt = (int64_t)gridDim.x * blockDim.x;
    unsigned bad = 0;   // flags[0]'s bits, bit 4: a negative value
    int diff = 0;       // descents less those at row starts, seen by this thread
    for (int64_t q0 = 4 * (t0 - lane); q0 < nnz; q0 += 4 * nt) {   // a wave's 256 nonzeros
        const int64_t q = q0 + 4 * lane;
        int32_t c[4];
        V v[4];
        const int m = (int)max((int64_t)0, min((int64_t)4, nnz - q));
        if (vec && m == 4) {
            const int4 cc = *reinterpret_cast<const int4*>(col + q);
            c[0] = cc.x;
            c[1] = cc.y;
            c[2] = cc.z;
            c[3] = cc.w;
            if (sizeof(V) == 4) {
                const float4 f = *reinterpret_cast<const float4*>(val + q);
                v[0] = f.x;
                v[1] = f.y;
                v[2] = f.z;
                v[3] = f.w;
            } else {
                const double2 f = *reinterpret_cast<const double2*>(val + q);
                const double2 g = *reinterpret_cast<const double2*>(val + q + 2);
                v[0] = (V)f.x;
                v[1] = (V)f.y;
                v[2] = (V)g.x;
                v[3] = (V)g.y;
            }
        } else {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                c[u] = u < m ? col[q + u] : 0;
                v[u] = u < m ? val[q + u] : (V)0;
            }
        }
        int32_t left = __shfl_up(c[3], 1, 64);
        if (lane == 0) left = q > 0 ? col[q - 1] : -1;
        if (q == 0) left = INT32_MIN;   // the first nonzero opens a row: no descent
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (u < m) {
                if (c[u] < 0 || c[u] >= d) bad |= 2;
                if (!finite_bits(v[u])) bad |= 4;
                if (v[u] < (V)0) bad |= 16;
                if (c[u] <= left) ++diff;
            }
            left = c[u];
        }
    }
    for (int64_t i = t0; i < n; i += nt) {
        const int64_t b = rp[i], e = rp[i + 1];
        if (i == 0 && b != 0) bad |= 8;
        if (i == n - 1 && e != stated) bad |= 8;
        if (e < b || b < 0 || e > nnz) bad |= 1;
        else if (b < e && b > 0 && col[b] <= col[b - 1]) --diff;
    }
    diff = (int)wave_sum_i64(diff);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) bad |= (unsigned)__shfl_xor((int)bad, o, 64);
    if (lane == 0) {
        sh_diff[wid] = diff;
        sh_bad[wid] = bad;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        int dsum = 0;
        unsigned b = 0;
#pragma unroll
        for (int w = 0; w < T / 64; ++w) {
            dsum += sh_diff[w];
            b |= sh_bad[w];
        }
        if (dsum) atomicAdd(&flags[3], (unsigned long long)(long long)dsum);
        if (b & 15u) atomicOr(&flags[0], (unsigned long long)(b & 15u));
        if (b & 16u) atomicOr(&flags[2], 1ull);
    }
}

// The failing matrix once more, row by row, for the row to report (flags[1])
// and the kind of every fault (flags[0]); runs only after k_validate found one.
//
// One wave per group of 64 consecutive rows: lane l holds the bounds of row
// g*64 + l, and the wave reads the group's nonzeros as one contiguous range,
// 64 at a time (coalesced).  For each such window the lanes OR together the
// bits of the row starts that fall in it, so a lane knows whether its element
// opens a row; otherwise its column must exceed its left neighbour's (taken
// by a shuffle, lane 0 from the previous window).  Row bounds that are out of
// order are reported as such and their group's elements are not inspected; nor
// are any past row_ptr[n], which the arrays need not hold.
__global__ __launch_bounds__(256) void k_validate_rows(const int64_t* __restrict__ rp, const int32_t* __restrict__ col,
                                                       const void* __restrict__ val, int f64, int64_t n, int64_t d,
                                                       int64_t nnz, unsigned long long* flags) {
    const int lane = threadIdx.x & 63;
    const int64_t wave = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6;
    const int64_t nw = ((int64_t)gridDim.x * blockDim.x) >> 6;
    const int64_t ngroups = (n + 63) / 64, held = rp[n];
    for (int64_t g = wave; g < ngroups; g += nw) {
        const int64_t i = g * 64 + lane;
        const bool row = i < n;
        int64_t b = 0, e = 0;
        unsigned long long bad = 0;
        if (row) {
            b = rp[i];
            e = rp[i + 1];
            if (i == 0 && b != 0) bad |= 8;
            if (i == n - 1 && e != nnz) bad |= 8;
            if (e < b || b < 0 || e > nnz) bad |= 1;
        }
        int64_t first_bad_row = bad ? i : INT64_MAX;
        const bool bounds_ok = ballot(bad != 0 || e > held) == 0ull;
        unsigned long long ebad = 0;
        if (bounds_ok) {
            // the group's nonzeros: [rp[g*64], rp[min(g*64+64, n)])
            const int64_t lo = bcast_i64(b, 0);
            const int last_lane = (int)min<int64_t>(63, n - 1 - g * 64);
            const int64_t hi = bcast_i64(e, last_lane);
            int32_t prev_last = -1;
            for (int64_t q = lo; q < hi; q += 64) {
                // rows (non-empty) starting inside [q, q + 64)
                const unsigned long long sb =
                    (row && b < e && b >= q && b < q + 64) ? (1ull << (int)(b - q)) : 0ull;
                const unsigned long long starts = wave_or_u64(sb);
                const int64_t p = q + lane;
                const bool in = p < hi;
                int32_t c = in ? col[p] : 0;
                int32_t left = __shfl_up(c, 1, 64);
                if (lane == 0) left = prev_last;
                unsigned long long eb = 0;
                if (in) {
                    if (c < 0 || c >= d) eb |= 2;
                    if (!((starts >> lane) & 1ull) && c <= left) eb |= 1;
                    const double v = f64 ? ((const double*)val)[p] : (double)((const float*)val)[p];
                    if (!isfinite(v)) eb |= 4;
                }
                prev_last = __shfl(c, 63, 64);
                if (ballot(eb != 0)) {
                    // error path: the row of each offending element (the last
                    // row of the group starting at or before it)
                    int64_t rbad = INT64_MAX;
                    for (int l = 0; l < 64 && g * 64 + l < n; ++l) {
                        const int64_t bl = bcast_i64(b, l), el = bcast_i64(e, l);
                        if (eb && p >= bl && p < el) rbad = g * 64 + l;
                    }
                    first_bad_row = min(first_bad_row, rbad);
                    ebad |= eb;
                }
            }
        }
        bad |= ebad;
        if (bad) {
            atomicOr(&flags[0], bad);
            atomicMax(&flags[1], ~(unsigned long long)first_bad_row);
        }
    }
}

hipError_t validate_csr(const int64_t* rp, const int32_t* col, const void* val, int f64, int64_t n, int64_t d,
                        int64_t nnz, unsigned long long* flags, hipStream_t s) {
    hipError_t e = fill_u64(flags, 0ull, 8, s);
    if (e != hipSuccess || n <= 0) return e;
    // 16-byte loads need both arrays aligned to them (a caller may pass slices)
    const int vec = (((uintptr_t)col | (uintptr_t)val) & 15) == 0;
    const int64_t want = std::max<int64_t>((nnz + 3) / 4, n);   // threads
    const int T = want <= (1 << 14) ? 256 : 1024;
    const dim3 grid((unsigned)std::min<int64_t>(512, (want + T - 1) / T));
    const float* f = (const float*)val;
    const double* g = (const double*)val;
    if (f64 && T == 256)
        hipLaunchKernelGGL((k_validate<double, 256>), grid, dim3(T), 0, s, rp, col, g, n, d, nnz, vec, flags);
    else if (f64)
        hipLaunchKernelGGL((k_validate<double, 1024>), grid, dim3(T), 0, s, rp, col, g, n, d, nnz, vec, flags);
    else if (T == 256)
        hipLaunchKernelGGL((k_validate<float, 256>), grid, dim3(T), 0, s, rp, col, f, n, d, nnz, vec, flags);
    else
        hipLaunchKernelGGL((k_validate<float, 1024>), grid, dim3(T), 0, s, rp, col, f, n, d, nnz, vec, flags);
    return hipGetLastError();
}

hipError_t validate_csr_rows(const int64_t* rp, const int32_t* col, const void* val, int f64, int64_t n, int64_t d,
                             int64_t nnz, unsigned long long* flags, hipStream_t s) {
    int64_t blocks = ((n + 63) / 64 + 3) / 4;
    if (blocks > 8192) blocks = 8192;
    hipLaunchKernelGGL(k_validate_rows, dim3((unsigned)blocks), dim3(256), 0, s, rp, col, val, f64, n, d, nnz, flags);
    return hipGetLastError();
}

// *flag |= 1 if some a[i] is outside [0, k)
__global__ void k_range_i32(const int32_t* __restrict__ a, int64_t n, int32_t k, unsigned long long* flags) {
    bool bad = false;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        bad |= (a[i] < 0 || a[i] >= k);
    if (__ballot(bad) && (threadIdx.x & 63) == 0) atomicOr(&flags[0], 1ull);
}

hipError_t range_check_i32(const int32_t* a, int64_t n, int32_t k, unsigned long long* flags, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    int64_t blocks = (n + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(k_range_i32, dim3((unsigned)blocks), dim3(256), 0, s, a, n, k, flags);
    return hipGetLastError();
}

// ---------------------------------------------------------------- centroid store helpers
// phase 0: lens_out[j] = nnz of row ids[j]; phase 1: copy the rows (values
// widened to FP64) to st.start[j] and set st.nnz[j].  One wave per centroid.
__global__ void k_gather_rows(const int64_t* __restrict__ rp, const int32_t* __restrict__ col,
                              const void* __restrict__ val, int f64, const int32_t* __restrict__ ids, int32_t k,
                              Store st, int64_t* lens_out, int phase) {
    const int lane = threadIdx.x & 63;
    const int64_t wave = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6;
    const int64_t nw = ((int64_t)gridDim.x * blockDim.x) >> 6;
    for (int64_t j = wave; j < k; j += nw) {
        int64_t i = ids[j];
        int64_t b = rp[i], e = rp[i + 1];
        if (phase == 0) {
            if (lane == 0) lens_out[j] = e - b;
            continue;
        }
        int64_t o = st.start[j];
        for (int64_t p = b + lane; p < e; p += 64) {
            st.term[o + (p - b)] = col[p];
            st.val[o + (p - b)] = f64 ? ((const double*)val)[p] : (double)((const float*)val)[p];
        }
        if (lane == 0) st.nnz[j] = e - b;
    }
}

hipError_t gather_rows(const Csr& X, const int32_t* ids, int32_t k, Store st, int64_t* lens_out, hipStream_t s,
                       int phase) {
    int64_t blocks = ((int64_t)k * 64 + 255) / 256;
    if (blocks > 8192) blocks = 8192;
    hipLaunchKernelGGL(k_gather_rows, dim3((unsigned)blocks), dim3(256), 0, s, X.rp, X.col, X.val, X.f64, ids, k,
                       st, lens_out, phase);
    return hipGetLastError();
}

// Entries are copied in pieces of 1,024 (one wave each), wherever the rows
// begin: a wave per centroid left 1,000 waves with 30,000 entries each
// (1.05 ms to export k = 1,000, D = 100,000; 0.11 now).
constexpr int kCopyPiece = 1024;

__global__ __launch_bounds__(256) void k_csr_to_store(const int64_t* __restrict__ ptr, const int32_t* __restrict__ col,
                                                      const double* __restrict__ val, int32_t k, int64_t nnz, Store st) {
    const int64_t t0 = blockIdx.x * (int64_t)blockDim.x + threadIdx.x, nt = (int64_t)gridDim.x * blockDim.x;
    for (int64_t p = t0; p < nnz; p += nt) {
        st.term[p] = col[p];
        st.val[p] = val[p];
    }
    for (int64_t j = t0; j < k; j += nt) {
        st.start[j] = ptr[j];
        st.nnz[j] = ptr[j + 1] - ptr[j];
    }
}

hipError_t csr_to_store(const int64_t* ptr, const int32_t* col, const double* val, int32_t k, int64_t nnz, Store st,
                        hipStream_t s) {
    const int64_t blocks = std::min<int64_t>(4096, std::max<int64_t>((nnz + 1023) / 1024, ((int64_t)k + 255) / 256));
    hipLaunchKernelGGL(k_csr_to_store, dim3((unsigned)blocks), dim3(256), 0, s, ptr, col, val, k, nnz, st);
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void k_store_export(Store st, int32_t k, const int64_t* __restrict__ c_ptr,
                                                      int32_t* c_col, double* c_val) {
    const int64_t n = c_ptr[k], nw = ((int64_t)gridDim.x * blockDim.x) >> 6;
    const int64_t wave = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6;
    for (int64_t p0 = wave * kCopyPiece; p0 < n; p0 += nw * kCopyPiece) {
        piece_entries(c_ptr, k, p0, min(n, p0 + kCopyPiece), [&](int64_t j, int64_t a, int64_t e, int first, int step) {
            const int64_t b = st.start[j] - c_ptr[j];
            for (int64_t p = a + first; p < e; p += step) {
                if (c_col) c_col[p] = st.term[b + p];
                if (c_val) c_val[p] = st.val[b + p];
            }
        });
    }
}

hipError_t store_export(const Store st, int32_t k, const int64_t* c_ptr, int32_t* c_col, double* c_val, hipStream_t s) {
    const int64_t blocks = std::min<int64_t>(4096, std::max<int64_t>(1, (st.cap + 4 * kCopyPiece - 1) / (4 * kCopyPiece)));
    hipLaunchKernelGGL(k_store_export, dim3((unsigned)blocks), dim3(256), 0, s, st, k, c_ptr, c_col, c_val);
    return hipGetLastError();
}

// cnorm[j] >= ||mu_j||_2 (the update computes its own while normalising).
__global__ __launch_bounds__(256) void k_centroid_norms(Store st, int32_t k, double* __restrict__ cnorm) {
    __shared__ double sh[4];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    for (int64_t j = blockIdx.x; j < k; j += gridDim.x) {
        const int64_t b = st.start[j], m = st.nnz[j];
        double acc = 0.0;
        for (int64_t p = threadIdx.x; p < m; p += 256) {
            const double v = st.val[b + p];
            acc = acc + v * v;
        }
        acc = wave_sum_f64(acc);
        __syncthreads();
        if (lane == 0) sh[wid] = acc;
        __syncthreads();
        if (threadIdx.x == 0) cnorm[j] = centroid_norm_bound((sh[0] + sh[1]) + (sh[2] + sh[3]));
    }
}

hipError_t centroid_norms(const Store st, int32_t k, double* cnorm, hipStream_t s) {
    hipLaunchKernelGGL(k_centroid_norms, dim3((unsigned)std::min<int32_t>(k, 65536)), dim3(256), 0, s, st, k, cnorm);
    return hipGetLastError();
}

}  // namespace sivf
