// Stable sorting of a tile of kFoldTile 32-bit keys in LDS by one workgroup of
// kFoldThreads threads: counting passes of at most kFoldBits bits.
#pragma once

#include "internal.h"
#include "wave.h"

namespace sivf {

constexpr int kFoldThreads = 512;
constexpr int kFoldWaves = kFoldThreads / 64;
constexpr int kFoldPer = kFoldTile / kFoldThreads;   // entries per thread: window i * 8 + wave, 64 wide
constexpr int kFoldBits = 9;
constexpr int kFoldBins = 1 << kFoldBits;            // one per thread
static_assert(kFoldBins == kFoldThreads, "one bin per thread");

struct TileSortLds {
    uint16_t cnt[kFoldWaves][kFoldBins];
    uint16_t base[kFoldBins];
    int32_t wsum[kFoldWaves];
};

// passes and bits per pass that sort keys below n
inline void tile_sort_plan(int64_t n, int* passes, int* nbits) {
    int bits = 1;
    while (bits < 31 && ((int64_t)1 << bits) < n) ++bits;
    *passes = (bits + kFoldBits - 1) / kFoldBits;
    *nbits = (bits + *passes - 1) / *passes;
}

// exclusive block scan of one value per thread; *total: the sum
__device__ inline int32_t tile_scan(int32_t v, int32_t* wsum, int32_t* total) {
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int32_t inc = wave_incl_scan_i32(v);
    __syncthreads();   // wsum free
    if (lane == 63) wsum[wid] = inc;
    __syncthreads();
    int32_t off = 0, tot = 0;
#pragma unroll
    for (int x = 0; x < kFoldWaves; ++x) {
        const int32_t s = wsum[x];
        if (x < wid) off += s;
        tot += s;
    }
    *total = tot;
    return off + inc - v;
}

// One stable counting pass over `ne` sorted positions: src order (nullptr:
// identity) by nbits bits of key from `shift` up, into dst.  Afterwards
// L.base[digit] is the position of the digit's first entry.
__device__ inline void tile_radix(TileSortLds& L, const uint32_t* key, const uint16_t* src, uint16_t* dst, int ne,
                                  int shift, int nbits) {
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const uint32_t dm = (1u << nbits) - 1u;
    // each wave owns a contiguous part of the order, so ranks are stable
    const int per = ((ne + kFoldThreads - 1) / kFoldThreads) * 64;
    const int lo = wid * per, hi = min(ne, lo + per);
    volatile uint16_t* cnt = L.cnt[wid];
#pragma unroll
    for (int b = 0; b < kFoldBins; b += 64) cnt[b + lane] = 0;
    uint32_t rk[kFoldPer];   // digit << 16 | rank
    uint16_t id[kFoldPer];
#pragma unroll
    for (int i = 0; i < kFoldPer; ++i) {
        const int s = lo + i * 64 + lane;
        const bool in = s < hi;
        const int p = in ? (src ? src[s] : s) : 0;
        id[i] = (uint16_t)p;
        rk[i] = ((key[p] >> shift) & dm) << 16;
    }
#pragma unroll
    for (int i = 0; i < kFoldPer; ++i) {
        if (lo + i * 64 >= hi) break;   // wave-uniform
        const bool in = lo + i * 64 + lane < hi;
        const uint32_t dg = rk[i] >> 16;
        unsigned long long m = ballot(in);
        for (int b = 0; b < nbits; ++b) {
            const unsigned long long v = ballot((dg >> b) & 1u);
            m &= ((dg >> b) & 1u) ? v : ~v;
        }
        const uint32_t old = in ? cnt[dg] : 0u;
        const int below = lanes_below(m);
        rk[i] |= old + (uint32_t)below;
        __builtin_amdgcn_wave_barrier();
        if (in && below == 0) cnt[dg] = (uint16_t)(old + (uint32_t)__popcll(m));
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    // per digit: exclusive over waves, then over digits
    uint32_t run = 0;
#pragma unroll
    for (int x = 0; x < kFoldWaves; ++x) {
        const uint32_t c = L.cnt[x][threadIdx.x];
        L.cnt[x][threadIdx.x] = (uint16_t)run;
        run += c;
    }
    int32_t total;
    L.base[threadIdx.x] = (uint16_t)tile_scan((int32_t)run, L.wsum, &total);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kFoldPer; ++i) {
        if (lo + i * 64 + lane < hi) {
            const uint32_t dg = rk[i] >> 16;
            dst[L.base[dg] + L.cnt[wid][dg] + (rk[i] & 0xffffu)] = id[i];
        }
    }
    __syncthreads();
}

}  // namespace sivf
