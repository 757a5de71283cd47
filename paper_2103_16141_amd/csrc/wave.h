// Wavefront-level helpers for 64-lane CDNA waves.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace sivf {

__device__ inline int lane_id() { return (int)(threadIdx.x & 63); }

// Number of set bits of `mask` in lanes below the calling lane.
__device__ inline int lanes_below(unsigned long long mask) {
    return (int)__builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0u));
}

__device__ inline unsigned long long ballot(bool p) { return __ballot(p); }

// Wave-uniform value of lane `l` (l must be wave-uniform).
__device__ inline int32_t bcast_i32(int32_t v, int l) { return __builtin_amdgcn_readlane(v, l); }
__device__ inline float bcast_f32(float v, int l) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}
__device__ inline int64_t bcast_i64(int64_t v, int l) {
    uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, l);
    uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)v >> 32), l);
    return (int64_t)(((uint64_t)hi << 32) | lo);
}
__device__ inline double bcast_f64(double v, int l) {
    return __longlong_as_double(bcast_i64(__double_as_longlong(v), l));
}

// Work grab: lane 0 adds `amount`, every lane gets the old value.  (One lane:
// atomics of 64 lanes on one address take 64 turns, about 40 ns a wave.)
__device__ inline int64_t wave_grab(unsigned long long* counter, unsigned long long amount) {
    unsigned long long old = 0;
    if (lane_id() == 0) old = atomicAdd(counter, amount);
    return bcast_i64((int64_t)old, 0);
}

__device__ inline int64_t wave_incl_scan_i64(int64_t v) {
    const int lane = lane_id();
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        int64_t u = __shfl_up(v, o, 64);
        if (lane >= o) v += u;
    }
    return v;
}

__device__ inline int32_t wave_incl_scan_i32(int32_t v) {
    const int lane = lane_id();
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        int32_t u = __shfl_up(v, o, 64);
        if (lane >= o) v += u;
    }
    return v;
}

// Butterfly sums: the same fixed association on every call, so results are
// run-to-run deterministic.  Every lane receives the total.
__device__ inline double wave_sum_f64(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

__device__ inline int64_t wave_sum_i64(int64_t v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

__device__ inline double wave_max_f64(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
    return v;
}

__device__ inline int32_t wave_min_i32(int32_t v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = min(v, __shfl_xor(v, o, 64));
    return v;
}

// A bound >= ||mu||_2 from the FP64 sum of squares acc (any order, relative
// error <= nnz * 2^-53): square root, then a 2^-30 relative margin.
__device__ inline double centroid_norm_bound(double acc) { return sqrt(acc) * (1.0 + 0x1p-30) + 0x1p-1000; }

// last centroid in [lo, hi] whose entries start at or before p (start ascends;
// empty ones share their successor's)
__device__ inline int64_t start_before(const int64_t* __restrict__ start, int64_t lo, int64_t hi, int64_t p) {
    while (lo < hi) {
        const int64_t mid = (lo + hi + 1) >> 1;
        if (start[mid] <= p) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// Calls f(centroid j, first entry, past the last, lane, lanes) for the entries
// [p0, p1) of k centroids starting at start[j], by one wave: centroid by centroid
// with all lanes, or, where the piece holds many short ones, an entry per lane
// (600 centroids of one entry: export 385 -> 150 us).
template <typename F>
__device__ inline void piece_entries(const int64_t* __restrict__ start, int64_t k, int64_t p0, int64_t p1, F f) {
    const int lane = lane_id();
    const int64_t lo = start_before(start, 0, k - 1, p0), hi = start_before(start, lo, k - 1, p1 - 1);
    if (hi - lo >= 16) {
        for (int64_t p = p0 + lane; p < p1; p += 64) f(start_before(start, lo, hi, p), p, p + 1, 0, 1);
        return;
    }
    for (int64_t j = lo; j <= hi; ++j) {
        const int64_t a = max(p0, start[j]), e = min(p1, start[j + 1]);
        if (a < e) f(j, a, e, lane, 64);
    }
}

constexpr int kXcds = 8;   // workgroup b runs on XCD b mod 8

// Blocks run in phases of up to 8, one block per XCD; in a phase with fewer
// blocks than XCDs, XCDs share a block and split its rows.  A wave takes items
// first, first + step, ... of block `blk`.  The workgroups are in `lanes` groups
// (a divisor of those of an XCD), which take every lanes-th phase each.
struct Share {
    int64_t blk, first, step;
};

__device__ inline int phase_lane(int lanes) { return (int)((blockIdx.x / kXcds) / (gridDim.x / kXcds / lanes)); }

__device__ inline Share phase_share(int64_t phase, int64_t nblk, int lanes = 1) {
    const int x = blockIdx.x % kXcds;
    const unsigned groups = gridDim.x / kXcds / lanes;   // workgroups of an XCD and lane
    const int64_t wave =
        __builtin_amdgcn_readfirstlane((int)((blockIdx.x / kXcds) % groups * (blockDim.x >> 6) + (threadIdx.x >> 6)));
    const int64_t waves = (int64_t)groups * (blockDim.x >> 6);
    const int nb = (int)min((int64_t)kXcds, nblk - phase * kXcds);
    const int b = x % nb, sharers = (kXcds - 1 - b) / nb + 1;
    return {phase * kXcds + b, wave * sharers + x / nb, waves * sharers};
}

// bf16 storage <-> f32: the 16 high bits of an IEEE binary32.
__device__ __host__ inline float bf16_to_f32(uint16_t b) {
    uint32_t u = (uint32_t)b << 16;
    float f;
    __builtin_memcpy(&f, &u, 4);
    return f;
}

// Round a finite binary32 to bf16, nearest-even (format definition: keep the
// top 16 bits, add half an ulp of bf16 plus the tie-to-even bit).
__device__ __host__ inline uint16_t f32_to_bf16_rne(float f) {
    uint32_t u;
    __builtin_memcpy(&u, &f, 4);
    uint32_t lsb = (u >> 16) & 1u;
    u += 0x7FFFu + lsb;
    return (uint16_t)(u >> 16);
}

}  // namespace sivf
