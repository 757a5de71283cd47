// Soft spherical assignment (the differentiable form of the assignment step):
//   S = X C^T, lse_i = log sum_j exp(S_ij / tau), loss = -sum_i lse_i,
//   backward: P = exp(S/tau - lse), dS = -g P / tau, dC = dS^T X,
//             dX_it = sum_j dS_ij C_jt on X's nonzeros (sampled dense-dense product).
//
// Every pass gathers rows (of C^T per object nonzero, of dS per CSC entry) and
// moves the same bytes, nnz * k * 4, so what counts is where they come from.
// Zipf terms make narrow slices of the rows cacheable: the columns are cut
// into blocks of 64 (C^T) or 32 (dS), each block's slices of all rows are one
// contiguous array, and the 8 XCDs (workgroup b runs on XCD b mod 8) work on 8
// blocks at a time, one each, block after block over all rows.  An XCD's 4 MB
// L2 then holds 256-byte slices of up to 16,384 terms (72% of a row's slices
// come from L1 or L2 at Zipf 1.1, D = 100,000; 56% with 512-column slices),
// and a block's dS slices of 24,576 rows.
//
// A wave takes one (row, block): its four 16-lane DPP rows gather four terms'
// 256-byte slices at once, 16 bytes a lane; a term's address and value sit in
// one lane and reach its DPP row by a row broadcast, so a step is one address
// instruction, one load and four fused multiply-adds.  No LDS, no barriers.
//
// Nothing of size N x k is kept: the backward recomputes S per row and
// materialises dS only for a chunk of rows, from which dC is accumulated
// term-major over a CSC copy of X whose lists are in ascending row order,
// chunk after chunk.  Every sum has a fixed order, so results are run-to-run
// deterministic.
#include <algorithm>
#include <utility>

#include "internal.h"
#include "slices.h"
#include "soft.h"
#include "wave.h"

namespace sivf {

constexpr int kBlk = kSoftBlk;   // columns of a C^T block (one 256-byte slice per term)
constexpr int kSub = kSoftSub;   // columns of a dS / dC^T block (128-byte slices)

// ---------------------------------------------------------------- block layouts
// out[b][t][c] = C[64 b + c][t] (0 past the last centroid), 64x64 tiles via LDS
__global__ __launch_bounds__(256) void k_soft_pack(const float* __restrict__ C, float* __restrict__ out, int64_t k,
                                                   int64_t d) {
    __shared__ float tile[64][65];
    const int64_t t0 = (int64_t)blockIdx.x * 64, j0 = (int64_t)blockIdx.y * kBlk;
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;   // 64 x 4
    for (int y = ty; y < 64; y += 4) {
        const int64_t j = j0 + y, t = t0 + tx;
        tile[y][tx] = (j < k && t < d) ? C[j * d + t] : 0.0f;
    }
    __syncthreads();
    float* o = out + (int64_t)blockIdx.y * d * kBlk;
    for (int y = ty; y < 64; y += 4)
        if (t0 + y < d) o[(t0 + y) * kBlk + tx] = tile[tx][y];
}

// dC[64 b + c][t] from the 32-column blocks [sb][t][32]
__global__ __launch_bounds__(256) void k_soft_unpack(const float* __restrict__ dCT, float* __restrict__ dC, int64_t k,
                                                     int64_t d) {
    __shared__ float tile[64][65];
    const int64_t t0 = (int64_t)blockIdx.x * 64, j0 = (int64_t)blockIdx.y * kBlk;
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
    const float* in = dCT + ((int64_t)blockIdx.y * 2 + (tx >> 5)) * d * kSub + (tx & 31);
    for (int y = ty; y < 64; y += 4)
        tile[y][tx] = (t0 + y < d && j0 + tx < k) ? in[(t0 + y) * kSub] : 0.0f;
    __syncthreads();
    for (int y = ty; y < 64; y += 4) {
        const int64_t j = j0 + y, t = t0 + tx;
        if (j < k && t < d) dC[j * d + t] = tile[tx][y];
    }
}

hipError_t soft_pack(const float* C, float* out, int64_t k, int64_t d, hipStream_t s) {
    const dim3 grid((unsigned)((d + 63) / 64), (unsigned)((k + kBlk - 1) / kBlk));
    hipLaunchKernelGGL(k_soft_pack, grid, dim3(256), 0, s, C, out, k, d);
    return hipGetLastError();
}

hipError_t soft_unpack(const float* dCT, float* dC, int64_t k, int64_t d, hipStream_t s) {
    const dim3 grid((unsigned)((d + 63) / 64), (unsigned)((k + kBlk - 1) / kBlk));
    hipLaunchKernelGGL(k_soft_unpack, grid, dim3(256), 0, s, dCT, dC, k, d);
    return hipGetLastError();
}

// ---------------------------------------------------------------- work split
// workgroups (a multiple of 8) for `items` wave-sized items per block
static unsigned share_grid(const void* fn, int64_t items, int64_t nblk, int threads, int n_cu) {
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, fn, threads, 0) != hipSuccess || nb < 1) nb = 1;
    const int64_t want = (items * std::min<int64_t>(nblk, kXcds) * 64 + threads - 1) / threads;
    const int64_t most = (int64_t)n_cu * nb;
    return (unsigned)(((std::max<int64_t>(1, std::min(want, most)) + kXcds - 1) / kXcds) * kXcds);
}

// The same for the passes over rows: few rows against many blocks leave most of
// the chip idle in every phase, and a phase starts with loads that nothing hides,
// so phases run side by side (*lanes) while a wave has at least 8 rows of one, or
// each row has a wave, and the slices they touch stay in L2 (`touched` rows of C^T).
// Forward in us with one lane and so, 40 terms a row, k = 20,000: 4 rows 307 and
// 241, 300 rows 409 and 379, 1,000 rows 509 and 492.
static unsigned share_grid_rows(const void* fn, int64_t rows, int64_t nblk, int64_t touched, int n_cu, int* lanes) {
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, fn, 256, 0) != hipSuccess || nb < 1) nb = 1;
    const int64_t most = std::max<int64_t>(1, (int64_t)n_cu * nb / kXcds);   // workgroups per XCD
    const int64_t phases = (nblk + kXcds - 1) / kXcds;
    const int64_t fit = std::max<int64_t>(1, (3ll << 20) / (std::max<int64_t>(touched, 1) * kBlk * 4));
    const int64_t l = std::max<int64_t>(1, std::min({phases, fit, most, 8 * 4 * most / std::max<int64_t>(rows, 1)}));
    if (l == 1) {
        *lanes = 1;
        return share_grid(fn, rows, nblk, 256, n_cu);
    }
    const int64_t groups = std::max<int64_t>(1, std::min(most / l, (rows + 3) / 4));
    *lanes = (int)l;
    return (unsigned)(groups * l * kXcds);
}

// ---------------------------------------------------------------- lane moves
template <int CTRL>
__device__ inline float dpp(float v) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, true));
}
template <int S>
__device__ inline uint32_t row_bcast(uint32_t v) {   // lane S of every 16-lane row
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x150 + S, 0xf, 0xf, true);
}
template <int S>
__device__ inline uint64_t row_bcast(uint64_t v) {
    return (uint64_t)row_bcast<S>((uint32_t)v) | ((uint64_t)row_bcast<S>((uint32_t)(v >> 32)) << 32);
}
template <int S>
__device__ inline float row_bcast(float v) {
    return __uint_as_float(row_bcast<S>(__float_as_uint(v)));
}

// sums over lanes 16 and 32 apart (every lane gets the total of its 4)
__device__ inline float sum_rows(float v) {
    auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ inline float max_rows(float v) {
    auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
    r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ inline float4 sum_rows4(float4 a) {
    return make_float4(sum_rows(a.x), sum_rows(a.y), sum_rows(a.z), sum_rows(a.w));
}
// over the whole wave: the 16 lanes of a row by rotations (8, 4, 2, 1), then the rows
__device__ inline float wave_sum(float v) {
    v = v + dpp<0x128>(v);
    v = v + dpp<0x124>(v);
    v = v + dpp<0x122>(v);
    v = v + dpp<0x121>(v);
    return sum_rows(v);
}
__device__ inline float wave_max(float v) {
    v = fmaxf(v, dpp<0x128>(v));
    v = fmaxf(v, dpp<0x124>(v));
    v = fmaxf(v, dpp<0x122>(v));
    v = fmaxf(v, dpp<0x121>(v));
    return max_rows(v);
}

__device__ inline float4 zero4() { return make_float4(0.0f, 0.0f, 0.0f, 0.0f); }
__device__ inline void fma4(float4& a, float v, const float4& g) {
    a.x = fmaf(v, g.x, a.x);
    a.y = fmaf(v, g.y, a.y);
    a.z = fmaf(v, g.z, a.z);
    a.w = fmaf(v, g.w, a.w);
}
__device__ inline float pick4(const float4& a, int i) { return i == 0 ? a.x : i == 1 ? a.y : i == 2 ? a.z : a.w; }

// ---------------------------------------------------------------- gathering a row's slices
// Up to 64 of a row's terms: lane (sub = lane / 16, q = lane % 16) holds the
// byte offset of term 4 q + sub's slice in the block and the term's value, so
// that step s broadcasts lane s of every DPP row to it and the wave gathers
// terms 4 s .. 4 s + 3.  Lanes past the row's end hold an offset outside the
// block, which reads as 0 without touching memory.
template <typename OFF>
struct Terms {
    OFF off;
    float v;
};

template <typename OFF>
__device__ inline Terms<OFF> load_terms(const int32_t* __restrict__ col, const float* __restrict__ xv, int64_t p0,
                                        int rem, int lane) {
    const int e = 4 * (lane & 15) + (lane >> 4);
    Terms<OFF> t;
    t.off = (OFF)~(OFF)0xff;
    t.v = 0.0f;
    if (e < rem) {
        t.off = (OFF)(uint32_t)col[p0 + e] * (OFF)(kBlk * 4);
        t.v = xv[p0 + e];
    }
    return t;
}

typedef unsigned int u32x4s __attribute__((ext_vector_type(4)));

// A block's slices.  While they span less than 4 GiB (OFF = uint32_t) they are
// read through a buffer descriptor, whose range check gives the zeros.
template <typename OFF>
struct Slices;
template <>
struct Slices<uint32_t> {
    __amdgpu_buffer_rsrc_t r;
    __device__ Slices(const float* base, int64_t d)
        : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base), (short)0, (int)(uint32_t)(d * (kBlk * 4)), 0x00020000)) {}
    __device__ float4 get(uint32_t off) const {
        const u32x4s v = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0);
        return make_float4(__uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z), __uint_as_float(v.w));
    }
};
template <>
struct Slices<uint64_t> {
    const char* base;
    __device__ Slices(const float* b, int64_t) : base((const char*)b) {}
    __device__ float4 get(uint64_t off) const {
        if ((off >> 63) != 0) return zero4();
        return *reinterpret_cast<const float4*>(base + off);
    }
};

template <typename OFF, int... S>
__device__ inline void gather_steps(float4* g, const Slices<OFF>& src, OFF off, uint32_t q16,
                                    std::integer_sequence<int, S...>) {
    ((g[S] = src.get(row_bcast<S>(off) | (OFF)q16)), ...);
}
template <int... S>
__device__ inline void fma_steps(float4& acc, const float4* g, float v, std::integer_sequence<int, S...>) {
    ((fma4(acc, row_bcast<S>(v), g[S]), (S % 4 == 3 ? __builtin_amdgcn_sched_barrier(0) : (void)0)), ...);
}

template <int G>
using Four = std::integer_sequence<int, 4 * G, 4 * G + 1, 4 * G + 2, 4 * G + 3>;

// acc += sum of the chunk's v * slice, steps in order; g keeps the slices
// (groups of four steps past the row's end are skipped, g is not set there)
template <typename OFF>
__device__ inline void gather_chunk(float4& acc, float4 (&g)[16], const Slices<OFF>& src, const Terms<OFF>& t,
                                    uint32_t q16, int rem) {
    if (0 < rem) gather_steps(g, src, t.off, q16, Four<0>{});
    if (16 < rem) gather_steps(g, src, t.off, q16, Four<1>{});
    if (32 < rem) gather_steps(g, src, t.off, q16, Four<2>{});
    if (48 < rem) gather_steps(g, src, t.off, q16, Four<3>{});
    if (0 < rem) fma_steps(acc, g, t.v, Four<0>{});
    if (16 < rem) fma_steps(acc, g, t.v, Four<1>{});
    if (32 < rem) fma_steps(acc, g, t.v, Four<2>{});
    if (48 < rem) fma_steps(acc, g, t.v, Four<3>{});
}

// ---------------------------------------------------------------- forward
// Per (row, block): the maximum of S / tau and the sum of exp(S / tau - max).
// Bound: L1 misses on random 256-byte slices (every slice from L2: 24 TB/s;
// with the rare terms' slices from the memory-side cache 15.6 TB/s).
// N = 262,144, D = 100,000, 100 terms a row, k = 4,096: 27.5 ms (28.4 with a
// workgroup per row and 512 columns); N = 20,011, k = 1,021: 0.36 ms (2.6: rows
// of k floats that no 16-byte load could read, now padded blocks).
template <typename OFF>
__global__ __launch_bounds__(256) void k_soft_fwd(int64_t c0, int64_t c1, const int64_t* __restrict__ rp,
                                                  const int32_t* __restrict__ col, const float* __restrict__ xv,
                                                  const float* __restrict__ CT, int64_t d, int32_t k, float inv_tau,
                                                  int lanes, float* __restrict__ pmax, float* __restrict__ psum) {
    const int lane = threadIdx.x & 63, q = lane & 15, sub = lane >> 4;
    const uint32_t q16 = 16 * q;
    const int64_t nblk = ((int64_t)k + kBlk - 1) / kBlk, n = c1 - c0;
    for (int64_t ph = phase_lane(lanes); ph * kXcds < nblk; ph += lanes) {
        const Share sh = phase_share(ph, nblk, lanes);
        const Slices<OFF> src(CT + sh.blk * d * kBlk, d);
        const bool mine = sh.blk * kBlk + 4 * q + sub < k;   // the column this lane exponentiates
        if (sh.first >= n) continue;
        // the next row's bounds and first terms are fetched ahead
        int64_t r0 = rp[c0 + sh.first];
        int m = (int)(rp[c0 + sh.first + 1] - r0);
        Terms<OFF> t = load_terms<OFF>(col, xv, r0, m, lane);
        for (int64_t i = sh.first; i < n; i += sh.step) {
            const int64_t in = min(i + sh.step, n - 1);
            const int64_t nr0 = rp[c0 + in];
            const int nm = (int)(rp[c0 + in + 1] - nr0);
            const Terms<OFF> nt = load_terms<OFF>(col, xv, nr0, nm, lane);
            float4 acc = zero4(), g[16];
            Terms<OFF> u = t;
            for (int h = 0; h < m; h += 64) {
                Terms<OFF> un = u;
                if (h + 64 < m) un = load_terms<OFF>(col, xv, r0 + h + 64, m - h - 64, lane);
                gather_chunk(acc, g, src, u, q16, m - h);
                u = un;
            }
            acc = sum_rows4(acc);
            const float x = mine ? pick4(acc, sub) * inv_tau : -INFINITY;
            const float mx = wave_max(x);
            const float z = wave_sum(mine ? expf(x - (mx == -INFINITY ? 0.0f : mx)) : 0.0f);
            if (lane == 0) {
                pmax[sh.blk * n + i] = mx;
                psum[sh.blk * n + i] = z;
            }
            r0 = nr0;
            m = nm;
            t = nt;
        }
    }
}

// lse_i = M + log sum_b psum_b exp(pmax_b - M), M = max_b pmax_b, blocks in
// order, and the FP64 sum of each workgroup's lse in a fixed order.  U blocks'
// values are loaded at a time: few rows of many blocks wait for little else (U =
// 16 against 1: 300 rows, k = 20,000: forward 379 -> 280 us; 2,000 rows, k = 4,096:
// 179 -> 156; of two blocks U = 16 takes 3.8 us for 3.0).
template <int U>
__global__ __launch_bounds__(256) void k_soft_lse(int64_t n, int64_t nblk, const float* __restrict__ pmax,
                                                  const float* __restrict__ psum, float* __restrict__ lse,
                                                  double* __restrict__ part) {
    __shared__ double sh[4];
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    double l = 0.0;
    if (i < n) {
        float M = -INFINITY;
        for (int64_t b = 0; b < nblk; b += U) {
            float px[U];
#pragma unroll
            for (int u = 0; u < U; ++u) px[u] = b + u < nblk ? pmax[(b + u) * n + i] : -INFINITY;
#pragma unroll
            for (int u = 0; u < U; ++u) M = fmaxf(M, px[u]);
        }
        float z = 0.0f;
        for (int64_t b = 0; b < nblk; b += U) {
            float px[U], ps[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                px[u] = b + u < nblk ? pmax[(b + u) * n + i] : -INFINITY;
                ps[u] = b + u < nblk ? psum[(b + u) * n + i] : 0.0f;
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (px[u] > -INFINITY) z += ps[u] * expf(px[u] - M);
                else if (ps[u] != 0.0f) z += ps[u];   // not a number
            }
        }
        const float v = M + logf(z);
        lse[i] = v;
        l = (double)v;
    }
    l = wave_sum_f64(l);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = l;
    __syncthreads();
    if (threadIdx.x == 0) part[blockIdx.x] = (sh[0] + sh[1]) + (sh[2] + sh[3]);
}

// loss = -(sum of the partial sums), each thread a contiguous range, then a tree
__global__ __launch_bounds__(1024) void k_soft_loss(const double* __restrict__ part, int64_t m, double* __restrict__ out) {
    __shared__ double sh[1024];
    const int64_t per = (m + 1023) / 1024;
    const int64_t lo = (int64_t)threadIdx.x * per, hi = min(m, lo + per);
    double acc = 0.0;
    for (int64_t i = lo; i < hi; ++i) acc += part[i];
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int s = 512; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) sh[threadIdx.x] += sh[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = -sh[0];
}

// ---------------------------------------------------------------- forward, the commonest terms in LDS
// Larger calls read the slices of the 608 commonest terms (56% of the nonzeros
// at Zipf 1.1, D = 100,000) from LDS: the gather's L1 misses were all of its
// time, and those slices were most of its L2 hits.  Which terms they are is
// counted on a sample of the nonzeros; any choice gives the same sums up to
// their order.  N = 262,144, D = 100,000, 100 terms a row, k = 4,096: 27.5 ->
// 16.5 ms (0.3 of it choosing and sorting the terms).

// counts of terms in 1024 runs of 64 nonzeros
__global__ __launch_bounds__(256) void k_soft_sample(const int32_t* __restrict__ col, int64_t nnz,
                                                     uint32_t* __restrict__ count) {
    const int64_t p = (blockIdx.x * 4 + (threadIdx.x >> 6)) * (nnz / 1024) + (threadIdx.x & 63);
    if (p < nnz) atomicAdd(&count[col[p]], 1u);
}

// one workgroup: the commonest terms' slots (slot[t], -1: none; term[slot]; *nhot)
__global__ __launch_bounds__(1024) void k_soft_hot(const uint32_t* __restrict__ count, int64_t d,
                                                   int32_t* __restrict__ slot, int32_t* __restrict__ term,
                                                   int32_t* __restrict__ nhot) {
    __shared__ uint32_t sh[258];
    __shared__ uint32_t nh;
    if (threadIdx.x == 0) nh = 0;
    const uint32_t x = top_weights(count, d, kSplitHot, sh);
    each_weight(count, d, [&](uint32_t v, int64_t t) {
        if (t >= d) return;
        int32_t q = -1;
        if (v >= x) {
            q = (int32_t)atomicAdd(&nh, 1u);
            term[q] = (int32_t)t;
        }
        slot[t] = q;
    });
    __syncthreads();
    if (threadIdx.x == 0) *nhot = (int32_t)nh;
}

// A wave per row of the chunk: its pairs and header (slices.h), the slot's or the
// term's slice as code.  Row o's pairs start at 32 + (nonzeros before it) + 32 o.
__global__ __launch_bounds__(256) void k_soft_prep(int64_t c0, int64_t n, const int64_t* __restrict__ rp,
                                                   const int32_t* __restrict__ col, const float* __restrict__ xv,
                                                   const int32_t* __restrict__ slot, const int32_t* __restrict__ nhot,
                                                   uint2* __restrict__ ent, uint2* __restrict__ hdr) {
    const int lane = threadIdx.x & 63;
    const int64_t p0 = rp[c0];
    const uint2 fill_hot = make_uint2((uint32_t)*nhot * kSliceBytes, 0u), fill_cold = make_uint2(kOutside, 0u);
    if (blockIdx.x == 0 && threadIdx.x < 32) ent[threadIdx.x] = threadIdx.x < 16 ? fill_hot : fill_cold;
    for (int64_t o = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); o < n; o += (int64_t)gridDim.x * 4) {
        const int64_t r0 = rp[c0 + o];
        const int m = (int)(rp[c0 + o + 1] - r0);
        int nh = 0;
        for (int h = lane; h - lane < m; h += 64) nh += __popcll(ballot(h < m && slot[col[r0 + min(h, m - 1)]] >= 0));
        const int nc = m - nh, ph = 16 * chunks16(nh), pc = 16 * chunks16(nc);
        const int64_t to = 32 + (r0 - p0) + 32 * o;
        uint2* out = ent + to;
        if (lane < 16) {
            if (nh + lane < ph) out[nh + lane] = fill_hot;
            if (nc + lane < pc) out[ph + nc + lane] = fill_cold;
        }
        int ah = 0, ac = ph;
        for (int h0 = 0; h0 < m; h0 += 64) {
            const int h = h0 + lane;
            const int32_t t = h < m ? col[r0 + h] : 0, q = h < m ? slot[t] : -1;
            const unsigned long long mh = ballot(q >= 0), mc = ballot(h < m && q < 0);
            if (h < m)
                out[q >= 0 ? ah + lanes_below(mh) : ac + lanes_below(mc)] =
                    make_uint2((uint32_t)(q >= 0 ? q : t) * kSliceBytes, __float_as_uint(xv[r0 + h]));
            ah += __popcll(mh);
            ac += __popcll(mc);
        }
        if (lane == 0) hdr[o] = make_uint2((uint32_t)to, ((uint32_t)nc << 12) | ((uint32_t)nh << 2));
    }
}

// k_soft_fwd's results for a chunk of rows, four rows to a wave (dense_groups).
// Four partial sums: dX, which takes exp of S from here and S from the backward,
// is off by 1.3e-6 of its largest value with one, 0.8e-6 with four.
__global__ __launch_bounds__(kDenseThreads) void k_soft_fwd_lds(int n, const uint2* __restrict__ ent, uint32_t npairs,
                                                                const uint2* __restrict__ hdr,
                                                                const int32_t* __restrict__ term,
                                                                const int32_t* __restrict__ nhot,
                                                                const float* __restrict__ CT, int64_t d, int32_t k,
                                                                float inv_tau, float* __restrict__ pmax,
                                                                float* __restrict__ psum) {
    extern __shared__ u32x4 panel[];
    const int q = threadIdx.x & 15, sub = (threadIdx.x & 63) >> 4, nh = *nhot;
    const __amdgpu_buffer_rsrc_t ents = bytes_rsrc(ent, npairs * (uint32_t)sizeof(uint2));
    uint32_t loads = 0;
    each_block((k + kBlk - 1) / kBlk, (n + 3) / 4, [&](int blk, int g0, int g1) {
        const char* src = (const char*)(CT + (int64_t)blk * d * kBlk);
        __syncthreads();
        for (int e = threadIdx.x; e < nh * 16; e += kDenseThreads)
            panel[e] = *reinterpret_cast<const u32x4*>(src + (int64_t)term[e >> 4] * kSliceBytes + 16 * (e & 15));
        if (threadIdx.x < 16) panel[nh * 16 + threadIdx.x] = u32x4{0u, 0u, 0u, 0u};
        __syncthreads();
        const int cols = k - blk * kBlk - 4 * q;   // of the lane's four, those that exist
        dense_groups<4>(
            g0, g1, ents, panel, bytes_rsrc(src, (uint32_t)(d * kSliceBytes)), loads,
            [&](int g) { return hdr[min(4 * g + sub, n - 1)]; }, [&](int g, const uint2&) { return 4 * g + sub < n; },
            [&](int g, const float4& acc, bool want) {
                const float x0 = cols > 0 ? acc.x * inv_tau : -INFINITY, x1 = cols > 1 ? acc.y * inv_tau : -INFINITY;
                const float x2 = cols > 2 ? acc.z * inv_tau : -INFINITY, x3 = cols > 3 ? acc.w * inv_tau : -INFINITY;
                float mx = fmaxf(fmaxf(x0, x1), fmaxf(x2, x3));
                mx = fmaxf(mx, dpp<0x128>(mx));
                mx = fmaxf(mx, dpp<0x124>(mx));
                mx = fmaxf(mx, dpp<0x122>(mx));
                mx = fmaxf(mx, dpp<0x121>(mx));
                const float b = mx == -INFINITY ? 0.0f : mx;
                float z = (cols > 0 ? expf(x0 - b) : 0.0f) + (cols > 1 ? expf(x1 - b) : 0.0f);
                z = z + ((cols > 2 ? expf(x2 - b) : 0.0f) + (cols > 3 ? expf(x3 - b) : 0.0f));
                z = z + dpp<0x128>(z);
                z = z + dpp<0x124>(z);
                z = z + dpp<0x122>(z);
                z = z + dpp<0x121>(z);
                if (want && q == 0) {
                    pmax[(int64_t)blk * n + 4 * g + sub] = mx;
                    psum[(int64_t)blk * n + 4 * g + sub] = z;
                }
            });
    });
}

// 32-bit slice offsets reach every term of a block (and one past is outside)
static bool narrow_offsets(int64_t d) { return d * (kBlk * 4) <= (int64_t)0xffffff00u; }

int64_t soft_lds_rows(int64_t N, int64_t nnz, int64_t d, int32_t k) {
    constexpr int64_t kRows = 65536;
    // headers hold 20 bits of a row's nonzeros
    if (!soft_lds_pays(nnz, k) || !narrow_offsets(d) || d >= (1 << 20) ||
        split_pairs(nnz, kRows) > kSplitMaxPairs)
        return 0;
    return std::min(N, kRows);
}

hipError_t soft_forward(int64_t N, int64_t nnz, const int64_t* rp, const int32_t* col, const float* xv, const float* C, int64_t d,
                        int32_t k, float tau, float* lse, double* loss_dev, SoftFwdWs w, int n_cu, hipStream_t s) {
    const int64_t nblk = ((int64_t)k + kBlk - 1) / kBlk;
    const bool narrow = narrow_offsets(d);
    const void* fn = narrow ? (const void*)k_soft_fwd<uint32_t> : (const void*)k_soft_fwd<uint64_t>;
    constexpr size_t lds = (size_t)(kSplitHot + 1) * kSliceBytes;
    if (w.ent) {
        hipError_t e = hipFuncSetAttribute((const void*)k_soft_fwd_lds, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e == hipSuccess) e = fill_i32((int32_t*)w.count, 0, d, s);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_soft_sample, dim3(256), dim3(256), 0, s, col, w.nnz, w.count);
        hipLaunchKernelGGL(k_soft_hot, dim3(1), dim3(1024), 0, s, w.count, d, w.slot, w.term, w.nhot);
    }
    int64_t parts = 0;
    for (int64_t c0 = 0; c0 < N; c0 += w.rows) {
        const int64_t c1 = std::min(N, c0 + w.rows), n = c1 - c0;
        if (w.ent) {
            const int64_t blocks = std::max<int64_t>(1, std::min<int64_t>((n + 3) / 4, (int64_t)n_cu * 8));
            hipLaunchKernelGGL(k_soft_prep, dim3((unsigned)blocks), dim3(256), 0, s, c0, n, rp, col, xv, w.slot, w.nhot,
                               w.ent, w.hdr);
        }
        for (int64_t b0 = 0; b0 < nblk; b0 += w.blocks) {
            const int32_t kg = (int32_t)std::min<int64_t>(w.blocks * kBlk, k - b0 * kBlk);
            int lanes;
            const unsigned grid = share_grid_rows(fn, n, std::min(w.blocks, nblk - b0), std::min(d, nnz), n_cu, &lanes);
            float *pmax = w.pmax + b0 * n, *psum = w.psum + b0 * n;
            if (c0 == 0 || w.blocks < nblk) {
                const hipError_t e = soft_pack(C + b0 * kBlk * d, w.CT, kg, d, s);
                if (e != hipSuccess) return e;
            }
            if (w.ent)
                hipLaunchKernelGGL(k_soft_fwd_lds, dim3((unsigned)((n_cu + kXcds - 1) / kXcds * kXcds)), dim3(kDenseThreads),
                                   lds, s, (int)n, w.ent, (uint32_t)split_pairs(w.nnz, w.rows), w.hdr, w.term, w.nhot, w.CT,
                                   d, kg, 1.0f / tau, pmax, psum);
            else if (narrow)
                hipLaunchKernelGGL(k_soft_fwd<uint32_t>, dim3(grid), dim3(256), 0, s, c0, c1, rp, col, xv, w.CT, d, kg,
                                   1.0f / tau, lanes, pmax, psum);
            else
                hipLaunchKernelGGL(k_soft_fwd<uint64_t>, dim3(grid), dim3(256), 0, s, c0, c1, rp, col, xv, w.CT, d, kg,
                                   1.0f / tau, lanes, pmax, psum);
        }
        const int64_t wgs = (n + 255) / 256;
        hipLaunchKernelGGL(nblk <= 4 ? k_soft_lse<4> : k_soft_lse<16>, dim3((unsigned)wgs), dim3(256), 0, s, n, nblk, w.pmax, w.psum, lse + c0,
                           w.part + parts);
        parts += wgs;
    }
    hipLaunchKernelGGL(k_soft_loss, dim3(1), dim3(1024), 0, s, w.part, parts, loss_dev);
    return hipGetLastError();
}

// ---------------------------------------------------------------- backward, rows of one chunk
// Per (row, block): S again, dS = -g exp(S / tau - lse) / tau into the dS
// blocks, and the block's share of dX on the row's nonzeros.  The slices of a
// row of at most 128 terms stay in registers between S and dX (longer rows
// are gathered a second time).  dX: each lane dots its four columns with the step's
// slice; 16 steps' dots are summed over the 16 lanes of their DPP row by
// exchanging halves (mirror 16, mirror 8, quad reversal, pair swap), after which
// lane q holds step q's sum, the term that lane loaded.  Blocks are added in
// order by k_soft_dx_combine.
// Bound: L1 misses, as the forward.  At its two shapes 31.5 ms and 0.50 ms
// (37.4 and 1.88 with a workgroup per row, slices of 64 columns and LDS sums).
template <int CTRL>
__device__ inline float exchange(float lo, float hi, bool upper) {
    return (upper ? hi : lo) + dpp<CTRL>(upper ? lo : hi);
}

__device__ inline float row_transpose_sum(float (&p)[16], int q) {
    float a[8], b[4], c[2];
#pragma unroll
    for (int s = 0; s < 8; ++s) a[s] = exchange<0x140>(p[s], p[s + 8], q >= 8);
#pragma unroll
    for (int s = 0; s < 4; ++s) b[s] = exchange<0x141>(a[s], a[s + 4], (q & 7) >= 4);
#pragma unroll
    for (int s = 0; s < 2; ++s) c[s] = exchange<0x1b>(b[s], b[s + 2], (q & 3) >= 2);
    return exchange<0xb1>(c[0], c[1], (q & 1) != 0);
}

// dX of a chunk's terms in this block, its first STEPS steps: lane (sub, q)
// gets term 4 q + sub's
template <int STEPS>
__device__ inline float chunk_dx(const float4* g, const float4& ds, int q) {
    float p[16];
#pragma unroll
    for (int s = 0; s < 16; ++s) {
        p[s] = 0.0f;
        if (s < STEPS) {
            p[s] = ds.x * g[s].x;
            p[s] = fmaf(ds.y, g[s].y, p[s]);
            p[s] = fmaf(ds.z, g[s].z, p[s]);
            p[s] = fmaf(ds.w, g[s].w, p[s]);
        }
    }
    return row_transpose_sum(p, q);
}

// dS of columns 4 q .. 4 q + 3 from the sub-sums of S: every lane takes one
// exponential and the four of a column group exchange them
__device__ inline float4 row_ds(float4 acc, bool mine, float inv_tau, float neg_g_over_tau, float l, int sub, int q) {
    acc = sum_rows4(acc);
    const float ds1 = mine ? neg_g_over_tau * expf(pick4(acc, sub) * inv_tau - l) : 0.0f;
    return make_float4(__shfl(ds1, q, 64), __shfl(ds1, q + 16, 64), __shfl(ds1, q + 32, 64), __shfl(ds1, q + 48, 64));
}

// what a (row, block) needs besides its terms
struct RowCtx {
    bool mine;               // this lane's column (the block's 4 q + sub) exists
    float inv_tau, neg_g_over_tau, l;
    uint32_t q16;
    int q, sub;
    float4* dsrow;           // the lane's four columns of dS, or nullptr
    float* out;              // the row's share of dX, or nullptr
};

// a row of at most 16 G terms, 64 in tA and the rest in tB; all slices in registers
template <int G, typename OFF>
__device__ inline void row_in_registers(const Slices<OFF>& src, const Terms<OFF>& tA, const Terms<OFF>& tB, int m,
                                        const RowCtx& c) {
    constexpr int A = G < 4 ? 4 * G : 16, B = 4 * G - A;   // steps of the two chunks
    float4 g[4 * G], acc = zero4();
    // the barriers keep the scheduler from moving every broadcast ahead of the
    // loads it waits for, which would not fit the registers
    gather_steps(g, src, tA.off, c.q16, std::make_integer_sequence<int, A>{});
    gather_steps(g + A, src, tB.off, c.q16, std::make_integer_sequence<int, B>{});
    __builtin_amdgcn_sched_barrier(0);
    fma_steps(acc, g, tA.v, std::make_integer_sequence<int, A>{});
    __builtin_amdgcn_sched_barrier(0);
    fma_steps(acc, g + A, tB.v, std::make_integer_sequence<int, B>{});
    __builtin_amdgcn_sched_barrier(0);
    const float4 ds = row_ds(acc, c.mine, c.inv_tau, c.neg_g_over_tau, c.l, c.sub, c.q);
    if (c.dsrow && c.sub == 0) *c.dsrow = ds;
    if (!c.out) return;
    const int e = 4 * c.q + c.sub;
    const float xa = chunk_dx<A>(g, ds, c.q);
    if (e < m) c.out[e] = xa;
    __builtin_amdgcn_sched_barrier(0);
    if (B > 0) {
        const float xb = chunk_dx<B>(g + A, ds, c.q);
        if (64 + e < m) c.out[64 + e] = xb;
    }
}

template <typename OFF>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_soft_bwd_rows(
    int64_t c0, int64_t c1, int64_t p0, int64_t pn, const int64_t* __restrict__ rp, const int32_t* __restrict__ col,
    const float* __restrict__ xv, const float* __restrict__ CT, int64_t d, int32_t k, float inv_tau,
    float neg_g_over_tau, int lanes, const float* __restrict__ lse, float* __restrict__ dS, float* __restrict__ dxp) {
    const int lane = threadIdx.x & 63;
    const int64_t nblk = ((int64_t)k + kBlk - 1) / kBlk, n = c1 - c0;
    RowCtx c;
    c.q = lane & 15;
    c.sub = lane >> 4;
    c.q16 = 16 * c.q;
    c.inv_tau = inv_tau;
    c.neg_g_over_tau = neg_g_over_tau;
    const int e0 = 4 * c.q + c.sub;   // this lane's column of a block and term of a chunk
    for (int64_t ph = phase_lane(lanes); ph * kXcds < nblk; ph += lanes) {
        const Share sh = phase_share(ph, nblk, lanes);
        const Slices<OFF> src(CT + sh.blk * d * kBlk, d);
        c.mine = sh.blk * kBlk + e0 < k;
        if (sh.first >= n) continue;
        // the next row's bounds and first terms are fetched ahead
        int64_t r0 = rp[c0 + sh.first];
        int m = (int)(rp[c0 + sh.first + 1] - r0);
        Terms<OFF> tA = load_terms<OFF>(col, xv, r0, m, lane);
        for (int64_t i = sh.first; i < n; i += sh.step) {
            const Terms<OFF> tB = load_terms<OFF>(col, xv, r0 + 64, m - 64, lane);
            const int64_t in = min(i + sh.step, n - 1);
            const int64_t nr0 = rp[c0 + in];
            const int nm = (int)(rp[c0 + in + 1] - nr0);
            const Terms<OFF> nt = load_terms<OFF>(col, xv, nr0, nm, lane);
            c.l = lse[c0 + i];
            c.dsrow = dS ? reinterpret_cast<float4*>(dS + ((sh.blk * 2 + (c.q >> 3)) * n + i) * kSub + 4 * (c.q & 7))
                         : nullptr;
            c.out = dxp ? dxp + sh.blk * pn + (r0 - p0) : nullptr;
            switch ((m + 15) >> 4) {
                case 0:
                case 1: row_in_registers<1>(src, tA, tB, m, c); break;
                case 2: row_in_registers<2>(src, tA, tB, m, c); break;
                case 3: row_in_registers<3>(src, tA, tB, m, c); break;
                case 4: row_in_registers<4>(src, tA, tB, m, c); break;
                case 5: row_in_registers<5>(src, tA, tB, m, c); break;
                case 6: row_in_registers<6>(src, tA, tB, m, c); break;
                case 7: row_in_registers<7>(src, tA, tB, m, c); break;
                case 8: row_in_registers<8>(src, tA, tB, m, c); break;
                default: {
                    float4 acc = zero4(), g[16];
                    for (int h = 0; h < m; h += 64)
                        gather_chunk(acc, g, src, load_terms<OFF>(col, xv, r0 + h, m - h, lane), c.q16, m - h);
                    const float4 ds = row_ds(acc, c.mine, inv_tau, neg_g_over_tau, c.l, c.sub, c.q);
                    if (c.dsrow && c.sub == 0) *c.dsrow = ds;
                    for (int h = 0; c.out && h < m; h += 64) {
                        const Terms<OFF> t = load_terms<OFF>(col, xv, r0 + h, m - h, lane);
                        gather_steps(g, src, t.off, c.q16, std::make_integer_sequence<int, 16>{});
                        const float x = chunk_dx<16>(g, ds, c.q);
                        if (h + e0 < m) c.out[h + e0] = x;
                    }
                }
            }
            r0 = nr0;
            m = nm;
            tA = nt;
        }
    }
}

// dxv[p] = (add ? dxv[p] : 0) + sum over the blocks, in order, of dxp[b][p]
__global__ void k_soft_dx_combine(int64_t pn, int64_t nblk, bool add, const float* __restrict__ dxp,
                                  float* __restrict__ dxv) {
    const int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (p >= pn) return;
    float a = add ? dxv[p] + dxp[p] : dxp[p];
    for (int64_t b = 1; b < nblk; ++b) a = a + dxp[b * pn + p];
    dxv[p] = a;
}

hipError_t soft_bwd_rows(int64_t c0, int64_t c1, int64_t p0, int64_t p1, const int64_t* rp, const int32_t* col,
                         const float* xv, const float* CT, int64_t d, int32_t k, float tau, float grad,
                         const float* lse, float* dS, float* dxp, float* dxv, bool add, int n_cu, hipStream_t s) {
    if (c1 <= c0) return hipSuccess;
    const int64_t nblk = ((int64_t)k + kBlk - 1) / kBlk, pn = p1 - p0;
    // where there is one block in all, its share is dX itself
    float* dx = !dxv ? nullptr : dxp ? dxp : dxv + p0;
    const bool narrow = narrow_offsets(d);
    const void* fn = narrow ? (const void*)k_soft_bwd_rows<uint32_t> : (const void*)k_soft_bwd_rows<uint64_t>;
    int lanes;
    const unsigned grid = share_grid_rows(fn, c1 - c0, nblk, std::min(d, pn), n_cu, &lanes);
    if (narrow)
        hipLaunchKernelGGL(k_soft_bwd_rows<uint32_t>, dim3(grid), dim3(256), 0, s, c0, c1, p0, pn, rp, col, xv, CT, d,
                           k, 1.0f / tau, -grad / tau, lanes, lse, dS, dx);
    else
        hipLaunchKernelGGL(k_soft_bwd_rows<uint64_t>, dim3(grid), dim3(256), 0, s, c0, c1, p0, pn, rp, col, xv, CT, d,
                           k, 1.0f / tau, -grad / tau, lanes, lse, dS, dx);
    if (dxv && dxp && pn > 0)
        hipLaunchKernelGGL(k_soft_dx_combine, dim3((unsigned)((pn + 255) / 256)), dim3(256), 0, s, pn, nblk, add, dxp,
                           dxv + p0);
    return hipGetLastError();
}

__global__ void k_chunk_offsets(const int64_t* __restrict__ rp, int64_t n, int64_t rc, int64_t nch,
                                int64_t* __restrict__ out) {
    const int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (j <= nch) out[j] = rp[min(j * rc, n)];
}

hipError_t soft_chunk_offsets(const int64_t* rp, int64_t n, int64_t rc, int64_t nch, int64_t* out, hipStream_t s) {
    hipLaunchKernelGGL(k_chunk_offsets, dim3((unsigned)((nch + 256) / 256)), dim3(256), 0, s, rp, n, rc, nch, out);
    return hipGetLastError();
}

// ---------------------------------------------------------------- dC^T, term-major, one chunk of rows
// dCT[sb][t][:] (+)= sum over rows i in [c0, c1) containing t, ascending CSC
// entries, of v_it * dS[sb][i - c0][:], 32 columns at a time: eight lanes (16
// bytes each) hold a row's 128-byte slice, and a wave gathers eight entries at
// once.  A term's entries inside the chunk are a range of its ascending CSC
// list.  Zipf frequencies make a few ranges as long as the chunk and most only
// a few entries, so there are three kinds:
//   * at most kTiny entries: eight terms per wave, a term's entries one after
//     another in its eight lanes, straight into dCT (k_dct_tiny);
//   * up to kPiece entries: a wave, eight partial sums added at the end,
//     straight into dCT; longer ones in pieces of kPiece entries into partial
//     rows (both k_dct_wave), which k_dct_combine adds into dCT.
// The chunk's slices of one block (24,576 rows, 3 MB) mostly stay in the XCD's
// L2 whatever the order of the rows.  What bounds it: L1 misses on random
// 128-byte slices (12 TB/s) and, for the rare terms, the read and write of dCT
// per chunk.  At the forward's shapes 42.7 and 0.50 ms (less the densest terms'
// entries 30.6, in chunks of 32,768 rows 28.6); with 512-column slices
// in chunks of 16,384 rows, cut at row blocks, 44 and 2.9 ms.
constexpr int kTiny = 8;
constexpr int kPiece = kSoftPiece;

__device__ inline int64_t row_lower_bound(const int32_t* __restrict__ xt_row, int64_t lo, int64_t hi, int64_t r) {
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (xt_row[mid] < r) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// The ranges of every term in the chunk ending at row c1 (`next` remembers
// where the previous chunk ended) and the lists of the longer ones.  List
// positions come from atomics: any order gives the same sums.
__global__ void k_dct_plan(int64_t d, int64_t c1, int fresh, const int64_t* __restrict__ colptr,
                           const int32_t* __restrict__ xt_row, DctWs w) {
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    int64_t lo = 0, len = 0;
    if (t < d) {
        lo = fresh ? colptr[t] : w.next[t];
        const int64_t end = colptr[t + 1];
        // most ranges are short: a few steps forward before the search
        int64_t hi = lo;
        for (int u = 0; u < 4 && hi < end && xt_row[hi] < c1; ++u) ++hi;
        if (hi == lo + 4) hi = row_lower_bound(xt_row, hi, end, c1);
        w.next[t] = hi;
        len = hi - lo;
        if (w.xd && w.slot[t] >= 0 && w.count[3] == 0) len = 0;   // k_dct_dense has it
        w.lo[t] = lo;
        w.len[t] = (int32_t)len;
    }
    const bool mid = len > kTiny && len <= kPiece;
    const unsigned long long m = ballot(mid);
    if (m) {
        int64_t at = 0;
        if (lanes_below(m) == 0 && mid) at = (int64_t)atomicAdd(&w.count[0], (unsigned long long)__popcll(m));
        at = bcast_i64(at, __builtin_ctzll(m));
        if (mid) w.mid[at + lanes_below(m)] = (int32_t)t;
    }
    if (len > kPiece) {
        const int64_t np = (len + kPiece - 1) / kPiece;
        const int64_t at = (int64_t)atomicAdd(&w.count[1], (unsigned long long)np);
        const int64_t l = (int64_t)atomicAdd(&w.count[2], 1ull);
        w.longt[l] = (int32_t)t;
        w.longp[l] = at;
        for (int64_t q = 0; q < np; ++q) w.piece[at + q] = lo + q * kPiece;
        for (int64_t q = 0; q < np; ++q) w.piece_len[at + q] = (int32_t)min((int64_t)kPiece, len - q * kPiece);
    }
}

__global__ __launch_bounds__(256) void k_dct_tiny(int64_t d, int64_t nsb, int64_t c0, int64_t n, int first,
                                                  const int32_t* __restrict__ xt_row, const float* __restrict__ xt_val,
                                                  const float* __restrict__ dS, float* __restrict__ dCT, DctWs w) {
    const int lane = threadIdx.x & 63, q = lane & 7, sub = lane >> 3;
    const int64_t groups = (d + 7) / 8;
    for (int64_t ph = 0; ph * kXcds < nsb; ++ph) {
        const Share sh = phase_share(ph, nsb);
        const char* base = (const char*)(dS + sh.blk * n * kSub);
        for (int64_t g = sh.first; g < groups; g += sh.step) {
            const int64_t t = g * 8 + sub;
            int32_t len = t < d ? w.len[t] : 0;
            const bool tiny = t < d && len <= kTiny && (len > 0 || first);
            if (!tiny) len = 0;
            uint32_t off = 0;
            float v = 0.0f;
            if (q < len) {
                const int64_t p = w.lo[t] + q;
                off = (uint32_t)(xt_row[p] - c0) * (kSub * 4);
                v = xt_val[p];
            }
            float4 acc = zero4();
            float4* out = reinterpret_cast<float4*>(dCT + (sh.blk * d + t) * kSub + 4 * q);
            if (tiny && !first) acc = *out;
            float4 x[kTiny];
            float vv[kTiny];
#pragma unroll
            for (int e = 0; e < kTiny; ++e) {
                const uint32_t o = (uint32_t)__shfl((int)off, (lane & ~7) + e, 64);
                vv[e] = __shfl(v, (lane & ~7) + e, 64);
                x[e] = zero4();
                if (e < len) x[e] = *reinterpret_cast<const float4*>(base + o + 16 * q);
            }
#pragma unroll
            for (int e = 0; e < kTiny; ++e) fma4(acc, vv[e], x[e]);
            if (tiny) *out = acc;
        }
    }
}

// sum of v * slice over CSC entries [lo, lo + len): lanes 0..7 (all subs alike)
__device__ inline float4 dct_range(const char* __restrict__ base, const int32_t* __restrict__ xt_row,
                                   const float* __restrict__ xt_val, int64_t c0, int64_t lo, int len, int lane) {
    const int q = lane & 7, sub = lane >> 3;
    float4 acc = zero4();
    for (int h = 0; h < len; h += 64) {
        uint32_t off = 0;
        float v = 0.0f;
        if (h + lane < len) {
            off = (uint32_t)(xt_row[lo + h + lane] - c0) * (kSub * 4);
            v = xt_val[lo + h + lane];
        }
        const int rem = len - h;
        float4 x[8];
        float vv[8];
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const uint32_t o = (uint32_t)__shfl((int)off, 8 * s + sub, 64);
            vv[s] = __shfl(v, 8 * s + sub, 64);
            x[s] = zero4();
            if (8 * s + sub < rem) x[s] = *reinterpret_cast<const float4*>(base + o + 16 * q);
        }
#pragma unroll
        for (int s = 0; s < 8; ++s) fma4(acc, vv[s], x[s]);
    }
    return acc;
}

// the eight entry lanes' sums, in a fixed tree
__device__ inline float sum_eight(float v) { return sum_rows(v + dpp<0x128>(v)); }

__global__ __launch_bounds__(256) void k_dct_wave(int64_t d, int64_t nsb, int64_t c0, int64_t n, int first,
                                                  const int32_t* __restrict__ xt_row, const float* __restrict__ xt_val,
                                                  const float* __restrict__ dS, float* __restrict__ dCT, DctWs w) {
    const int lane = threadIdx.x & 63;
    const int64_t nmid = (int64_t)w.count[0], np = min((int64_t)w.count[1], w.max_pieces);
    for (int64_t ph = 0; ph * kXcds < nsb; ++ph) {
        const Share sh = phase_share(ph, nsb);
        const char* base = (const char*)(dS + sh.blk * n * kSub);
        for (int64_t o = sh.first; o < np + nmid; o += sh.step) {
            const bool piece = o < np;   // the long pieces first
            const int32_t t = piece ? 0 : w.mid[o - np];
            const int64_t lo = piece ? w.piece[o] : w.lo[t];
            const int len = piece ? w.piece_len[o] : w.len[t];
            float4 a = dct_range(base, xt_row, xt_val, c0, lo, len, lane);
            a = make_float4(sum_eight(a.x), sum_eight(a.y), sum_eight(a.z), sum_eight(a.w));
            if (lane < 8) {
                float4* out = piece ? reinterpret_cast<float4*>(w.part + (sh.blk * w.max_pieces + o) * kSub + 4 * lane)
                                    : reinterpret_cast<float4*>(dCT + (sh.blk * d + t) * kSub + 4 * lane);
                if (!piece && !first) {
                    const float4 b = *out;
                    a = make_float4(b.x + a.x, b.y + a.y, b.z + a.z, b.w + a.w);
                }
                *out = a;
            }
        }
    }
}

// dCT[t] = (first ? 0 : dCT[t]) + partial rows of t's pieces: eight partial
// sums (every eighth piece in order), added in a fixed tree
__global__ __launch_bounds__(256) void k_dct_combine(int64_t d, int64_t nsb, int first, float* __restrict__ dCT, DctWs w) {
    const int lane = threadIdx.x & 63, q = lane & 7, sub = lane >> 3;
    const int64_t nlong = (int64_t)w.count[2];
    for (int64_t ph = 0; ph * kXcds < nsb; ++ph) {
        const Share sh = phase_share(ph, nsb);
        for (int64_t l = sh.first; l < nlong; l += sh.step) {
            const int32_t t = w.longt[l];
            const int64_t p0 = w.longp[l], np = ((int64_t)w.len[t] + kPiece - 1) / kPiece;
            const float* part = w.part + (sh.blk * w.max_pieces + p0) * kSub + 4 * q;
            float4 a = zero4();
            for (int64_t p = sub; p < np && p0 + p < w.max_pieces; p += 8) {
                const float4 x = *reinterpret_cast<const float4*>(part + p * kSub);
                a = make_float4(a.x + x.x, a.y + x.y, a.z + x.z, a.w + x.w);
            }
            a = make_float4(sum_eight(a.x), sum_eight(a.y), sum_eight(a.z), sum_eight(a.w));
            if (lane < 8) {
                float4* out = reinterpret_cast<float4*>(dCT + (sh.blk * d + t) * kSub + 4 * lane);
                if (!first) {
                    const float4 b = *out;
                    a = make_float4(b.x + a.x, b.y + a.y, b.z + a.z, b.w + a.w);
                }
                *out = a;
            }
        }
    }
}

// ---------------------------------------------------------------- dC^T of the densest terms
// A term in more than a few percent of the rows costs less as a row of a matrix
// product than entry by entry: dC^T = Xd^T dS with Xd the chunk's rows over the
// 256 densest terms (46% of the nonzeros at Zipf 1.1, D = 100,000, 100 terms a
// row), on the FP32 matrix cores.  An entry costs 0.4 ps of gathers per column, a
// place of Xd 0.015, so terms in 1/32 of the rows and more are taken.  N =
// 262,144, k = 4,096: 42.6 ms for dC before, 36.0 so (5.4 the products, at 104
// TFLOP/s of 149 that a library product reaches).

__global__ void k_dct_cands(int64_t N, int64_t d, const int64_t* __restrict__ colptr, int64_t room, DctWs w) {
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    const int64_t df = t < d ? colptr[t + 1] - colptr[t] : 0;
    const bool has = df * 32 >= N && df > 0;
    const unsigned long long m = ballot(has);
    if (t < d) w.slot[t] = -1;
    if (!m) return;
    int64_t at = 0;
    if ((threadIdx.x & 63) == 0) at = (int64_t)atomicAdd(&w.ndense[0], (unsigned long long)__popcll(m));
    at = bcast_i64(at, 0) + lanes_below(m);
    if (has && at < room) {
        w.cand[at] = (int32_t)t;
        w.cand_df[at] = (uint32_t)min(df, (int64_t)0xffffffffu);
    }
}

// the densest candidates, if their products pay
__global__ __launch_bounds__(1024) void k_dct_pick(int64_t N, int32_t k, int64_t room, DctWs w) {
    __shared__ uint32_t sh[258];
    __shared__ uint32_t taken;
    __shared__ unsigned long long entries;
    if (threadIdx.x == 0) {
        taken = 0;
        entries = 0;
    }
    const int64_t n = min(room, (int64_t)w.ndense[0]);
    const uint32_t x = top_weights(w.cand_df, n, kDctDense, sh);
    each_weight(w.cand_df, n, [&](uint32_t v, int64_t i) {
        if (i < n && v >= x) atomicAdd(&entries, (unsigned long long)v);
    });
    __syncthreads();
    if (!soft_prod_pays((double)entries, (double)N, (double)k)) return;   // ndense[1] stays 0, all slots -1
    each_weight(w.cand_df, n, [&](uint32_t v, int64_t i) {
        if (i >= n || v < x) return;
        const uint32_t q = atomicAdd(&taken, 1u);   // any numbering gives the same sums
        w.term[q] = w.cand[i];
        w.slot[w.cand[i]] = (int32_t)q;
    });
    __syncthreads();
    if (threadIdx.x == 0) w.ndense[1] = taken;
}

hipError_t dct_pick(int64_t N, int64_t d, int32_t k, const int64_t* colptr, DctWs w, hipStream_t s) {
    const int64_t room = dct_cands(w.nnz, N);
    hipLaunchKernelGGL(k_dct_cands, dim3((unsigned)((d + 255) / 256)), dim3(256), 0, s, N, d, colptr, room, w);
    hipLaunchKernelGGL(k_dct_pick, dim3(1), dim3(1024), 0, s, N, k, room, w);
    return hipGetLastError();
}

// a wave per row: its densest terms' values over zeros, in LDS, then written
__global__ __launch_bounds__(256) void k_dct_dense_rows(int64_t c0, int64_t n, const int64_t* __restrict__ rp,
                                                        const int32_t* __restrict__ col, const float* __restrict__ xv,
                                                        DctWs w) {
    __shared__ float4 buf[4][kDctDense / 4];
    if (w.ndense[1] == 0) return;   // no term qualified: nothing reads them
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    float* row = reinterpret_cast<float*>(buf[wid]);
    for (int64_t i = (int64_t)blockIdx.x * 4 + wid; i < n; i += (int64_t)gridDim.x * 4) {
        buf[wid][lane] = zero4();
        const int64_t r1 = rp[c0 + i + 1];
        for (int64_t p = rp[c0 + i] + lane; p < r1; p += 64) {
            const int32_t q = w.slot[col[p]];
            if (q >= 0) row[q] = xv[p];
        }
        reinterpret_cast<float4*>(w.xd + i * kDctDense)[lane] = buf[wid][lane];
    }
}

hipError_t dct_dense_rows(int64_t c0, int64_t c1, const int64_t* rp, const int32_t* col, const float* xv, DctWs w,
                          int n_cu, hipStream_t s) {
    const int64_t n = c1 - c0;
    const unsigned blocks = (unsigned)std::min<int64_t>((n + 3) / 4, (int64_t)n_cu * 8);
    hipLaunchKernelGGL(k_dct_dense_rows, dim3(blocks), dim3(256), 0, s, c0, n, rp, col, xv, w);
    return hipGetLastError();
}

// How a chunk of n rows is cut: about 512 workgroups of two dS blocks by a range
// of rows (a multiple of 32).
constexpr int kProdRows = 32;   // rows of Xd in LDS
struct ProdCut {
    int cgroups, rows, splits;
};
static ProdCut prod_cut(int64_t n, int32_t k) {
    ProdCut c;
    c.cgroups = (int)((((int64_t)k + kBlk - 1) / kBlk));
    const int64_t want = std::max<int64_t>(1, std::min<int64_t>(512 / c.cgroups, (n + kProdRows - 1) / kProdRows));
    c.rows = (int)(((n + want - 1) / want + kProdRows - 1) / kProdRows * kProdRows);
    c.splits = (int)((n + c.rows - 1) / c.rows);
    return c;
}
int64_t dct_prod_elems(int64_t rows, int32_t k) {
    const int64_t cg = ((int64_t)k + kBlk - 1) / kBlk;
    return std::max<int64_t>(1, std::min<int64_t>(512 / cg, (rows + kProdRows - 1) / kProdRows)) * cg * 2 * kDctDense * kSub;
}

// prod[split][sb][slot][32] = sum over the split's rows of xd[row][slot] dS[sb][row].
// Four waves: two dS blocks by two halves of the terms; a wave holds 128 terms x
// 32 columns of sums.  v_mfma_f32_32x32x2_f32 takes two rows a step: lane l gives
// term (or column) l % 32 of row l / 32, and holds rows 8 (r / 4) + 4 (l / 32) +
// r % 4 of column l % 32 in result r.  32 rows of Xd are in LDS (rows 288 floats
// apart: the two rows of a step use different banks), the next 32 and their dS on
// the way.  Sums of 32 rows are added to the running ones, which rounds less than
// one chain.  Zeros of Xd meet every dS: a dS that is not finite sets count[3],
// and the chunk's sums are then taken entry by entry.
typedef float f32x16 __attribute__((ext_vector_type(16)));

__global__ __launch_bounds__(256, 2) void k_dct_dense(int n, int nsb, ProdCut cut, const float* __restrict__ dS,
                                                      DctWs w) {
    constexpr int kStride = kDctDense + 32;
    __shared__ float tile[2][kProdRows * kStride];
    const int M = (int)w.ndense[1];
    if (M == 0) return;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, j = lane & 31, kk = lane >> 5;
    // the splits of an XCD are its own: their rows of Xd stay in its L2
    const int split = blockIdx.x % cut.splits, cg = blockIdx.x / cut.splits;
    const int sb = 2 * cg + (wid & 1), half = 128 * (wid >> 1);
    const int mt = __builtin_amdgcn_readfirstlane(min(4, max(0, (M - half + 31) / 32)));
    const int r0 = split * cut.rows, r1 = min(n, r0 + cut.rows);
    const float* ds = dS + (int64_t)sb * n * kSub + j;   // nsb is even: both blocks exist
    float4 a[8];
    float b[kProdRows / 2], nb[kProdRows / 2];
    auto fetch = [&](int base, float* bb) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int e = i * 256 + threadIdx.x, row = base + (e >> 6);
            a[i] = row < r1 ? reinterpret_cast<const float4*>(w.xd + (int64_t)row * kDctDense)[e & 63] : zero4();
        }
#pragma unroll
        for (int i = 0; i < kProdRows / 2; ++i) {
            const int row = base + 2 * i + kk;
            bb[i] = row < r1 ? ds[(int64_t)row * kSub] : 0.0f;
        }
    };
    auto put = [&](float* to) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int e = i * 256 + threadIdx.x;
            *reinterpret_cast<float4*>(to + (e >> 6) * kStride + 4 * (e & 63)) = a[i];
        }
    };
    f32x16 sum[4];
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int r = 0; r < 16; ++r) sum[m][r] = 0.0f;
    bool bad = false;
    fetch(r0, b);
    put(tile[0]);
    __syncthreads();
    int cur = 0;
    for (int base = r0; base < r1; base += kProdRows) {
        const bool more = base + kProdRows < r1;
        if (more) fetch(base + kProdRows, nb);
        const float* t = tile[cur] + kk * kStride + half + j;
#pragma unroll
        for (int i = 0; i < kProdRows / 2; ++i) bad |= (__float_as_uint(b[i]) & 0x7f800000u) == 0x7f800000u;
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            if (m >= mt) break;
            f32x16 c;
#pragma unroll
            for (int r = 0; r < 16; ++r) c[r] = 0.0f;
#pragma unroll
            for (int i = 0; i < kProdRows / 2; ++i)
                c = __builtin_amdgcn_mfma_f32_32x32x2f32(t[2 * i * kStride + 32 * m], b[i], c, 0, 0, 0);
#pragma unroll
            for (int r = 0; r < 16; ++r) sum[m][r] = sum[m][r] + c[r];
        }
        if (more) {
            put(tile[cur ^ 1]);
#pragma unroll
            for (int i = 0; i < kProdRows / 2; ++i) b[i] = nb[i];
        }
        cur ^= 1;
        __syncthreads();
    }
    if (ballot(bad) && lane == 0) atomicOr(&w.count[3], 1ull);
    float* out = w.prod + (((int64_t)split * nsb + sb) * kDctDense + half) * kSub + j;
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        if (m >= mt) break;
#pragma unroll
        for (int r = 0; r < 16; ++r) out[(32 * m + 8 * (r / 4) + 4 * kk + r % 4) * kSub] = sum[m][r];
    }
}

// dCT += the splits' products, in order
__global__ __launch_bounds__(256) void k_dct_dense_add(int64_t d, int nsb, int nsb2, int splits, float* __restrict__ dCT, DctWs w) {
    const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;   // (sb, slot, q)
    const int64_t rowi = e >> 3;
    const int slot = (int)(rowi % kDctDense);
    const int64_t sb = rowi / kDctDense;
    if (sb >= nsb || slot >= (int)w.ndense[1] || w.count[3] != 0) return;
    const float4* p = reinterpret_cast<const float4*>(w.prod) + e;
    float4 a = p[0];
    for (int s = 1; s < splits; ++s) {
        const float4 x = p[(int64_t)s * nsb2 * kDctDense * (kSub / 4)];
        a = make_float4(a.x + x.x, a.y + x.y, a.z + x.z, a.w + x.w);
    }
    float4* out = reinterpret_cast<float4*>(dCT + (sb * d + w.term[slot]) * kSub) + (e & 7);
    const float4 o = *out;
    *out = make_float4(o.x + a.x, o.y + a.y, o.z + a.z, o.w + a.w);
}

hipError_t soft_dct(int64_t d, int32_t k, int64_t c0, int64_t c1, int first, int fresh, const int64_t* colptr,
                    const int32_t* xt_row, const float* xt_val, const float* dS, float* dCT, DctWs w, int n_cu,
                    hipStream_t s) {
    const int64_t nsb = ((int64_t)k + kSub - 1) / kSub, n = c1 - c0;
    const ProdCut cut = prod_cut(n, k);
    const int nsb2 = 2 * cut.cgroups;   // dS and dCT have an even number of blocks
    if (w.xd) hipLaunchKernelGGL(k_dct_dense, dim3((unsigned)(cut.splits * cut.cgroups)), dim3(256), 0, s, (int)n, nsb2, cut, dS, w);
    hipLaunchKernelGGL(k_dct_plan, dim3((unsigned)((d + 255) / 256)), dim3(256), 0, s, d, c1, fresh, colptr, xt_row, w);
    const unsigned gt = share_grid((const void*)k_dct_tiny, (d + 7) / 8, nsb, 256, n_cu);
    const unsigned gw = share_grid((const void*)k_dct_wave, d, nsb, 256, n_cu);
    const unsigned gc = share_grid((const void*)k_dct_combine, std::min<int64_t>(d, w.max_pieces), nsb, 256, n_cu);
    hipLaunchKernelGGL(k_dct_wave, dim3(gw), dim3(256), 0, s, d, nsb, c0, n, first, xt_row, xt_val, dS, dCT, w);
    hipLaunchKernelGGL(k_dct_tiny, dim3(gt), dim3(256), 0, s, d, nsb, c0, n, first, xt_row, xt_val, dS, dCT, w);
    if (w.max_pieces > 0)
        hipLaunchKernelGGL(k_dct_combine, dim3(gc), dim3(256), 0, s, d, nsb, first, dCT, w);
    if (w.xd)
        hipLaunchKernelGGL(k_dct_dense_add, dim3((unsigned)(nsb * kDctDense * 8 / 256)), dim3(256), 0, s, d, (int)nsb,
                           nsb2, cut.splits, dCT, w);
    return hipGetLastError();
}

}  // namespace sivf
