// Sums of v * slice over an object's terms, four objects to a wave: shared by
// the split walk and the soft forward.
//
// The slices are the 256-byte pieces (64 columns, FP32) of dense rows.  A
// workgroup of 16 waves holds the slices of the heaviest rows of one block of
// columns in LDS and takes four objects per wave, one per 16-lane DPP row: a
// term's code and value reach the row's lanes by a broadcast, each lane adds 16
// bytes of the slice (4 columns).  Slices are
// 256 bytes apart, so the 16 lanes of a DPP row read each LDS bank once.
#pragma once

#include <type_traits>

#include "wave.h"

namespace sivf {

constexpr int kDenseThreads = 1024;

// A pair is (code, value).  An object's pairs are in chunks of 16, those of LDS
// rows first (code: byte offset of the slice in LDS), then the others (byte
// offset in the block's slices); the last chunk of each is filled up with pairs
// that add nothing: LDS's row of zeros, or an offset past the block, where a
// buffer load gives 0.  Pairs 0 .. 31 of the array are two chunks of fill.
// Header: first pair; others << 12 | LDS rows << 2 | two flags.
constexpr uint32_t kOutside = 0xffffff00u;
__device__ inline int hdr_hot(const uint2& hd) { return (int)((hd.y >> 2) & 1023u); }
__device__ inline int hdr_cold(const uint2& hd) { return (int)(hd.y >> 12); }
__device__ inline int chunks16(int n) { return (n + 15) >> 4; }

__device__ inline __amdgpu_buffer_rsrc_t bytes_rsrc(const void* p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes, 0x00020000);
}

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

template <int S>
__device__ inline uint32_t drow_bcast(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x150 + S, 0xf, 0xf, true);
}

// acc += v[4 G + i] * u[i], i = 0 .. 3, v broadcast within each DPP row by the
// multiply-add itself (compiled from a broadcast and four fmaf it takes a move
// more per step).  A DPP operand may not be written by the two instructions
// before: hence the s_nop.
template <int G>
__device__ inline void dense_fma4(float4& acc, float v, const u32x4 (&u)[4]) {
#define STEP(S, A, B, C, D)                                                          \
    "v_fmac_f32_dpp %0, %4, " A " row_newbcast:" S " row_mask:0xf bank_mask:0xf\n\t" \
    "v_fmac_f32_dpp %1, %4, " B " row_newbcast:" S " row_mask:0xf bank_mask:0xf\n\t" \
    "v_fmac_f32_dpp %2, %4, " C " row_newbcast:" S " row_mask:0xf bank_mask:0xf\n\t" \
    "v_fmac_f32_dpp %3, %4, " D " row_newbcast:" S " row_mask:0xf bank_mask:0xf\n\t"
#define FOUR(S0, S1, S2, S3)                                                                                     \
    asm("s_nop 1\n\t" STEP(S0, "%5", "%6", "%7", "%8") STEP(S1, "%9", "%10", "%11", "%12")                       \
            STEP(S2, "%13", "%14", "%15", "%16") STEP(S3, "%17", "%18", "%19", "%20")                            \
        : "+v"(acc.x), "+v"(acc.y), "+v"(acc.z), "+v"(acc.w)                                                     \
        : "v"(v), "v"(u[0].x), "v"(u[0].y), "v"(u[0].z), "v"(u[0].w), "v"(u[1].x), "v"(u[1].y), "v"(u[1].z),     \
          "v"(u[1].w), "v"(u[2].x), "v"(u[2].y), "v"(u[2].z), "v"(u[2].w), "v"(u[3].x), "v"(u[3].y), "v"(u[3].z), \
          "v"(u[3].w))
    if (G == 0) FOUR("0", "1", "2", "3");
    if (G == 1) FOUR("4", "5", "6", "7");
    if (G == 2) FOUR("8", "9", "10", "11");
    if (G == 3) FOUR("12", "13", "14", "15");
#undef FOUR
#undef STEP
}

// The same into four sums, every fourth step each.
#define SIVF_STEP(S, A, B, C, D, U, V, W, X)                                              \
    "v_fmac_f32_dpp " A ", %8, " U " row_newbcast:" S " row_mask:0xf bank_mask:0xf\n\t" \
    "v_fmac_f32_dpp " B ", %8, " V " row_newbcast:" S " row_mask:0xf bank_mask:0xf\n\t" \
    "v_fmac_f32_dpp " C ", %8, " W " row_newbcast:" S " row_mask:0xf bank_mask:0xf\n\t" \
    "v_fmac_f32_dpp " D ", %8, " X " row_newbcast:" S " row_mask:0xf bank_mask:0xf\n\t"
#define SIVF_TWO(S0, S1, P, Q, U, V)                                                                 \
    asm("s_nop 1\n\t" SIVF_STEP(S0, "%0", "%1", "%2", "%3", "%9", "%10", "%11", "%12")               \
            SIVF_STEP(S1, "%4", "%5", "%6", "%7", "%13", "%14", "%15", "%16")                        \
        : "+v"(P.x), "+v"(P.y), "+v"(P.z), "+v"(P.w), "+v"(Q.x), "+v"(Q.y), "+v"(Q.z), "+v"(Q.w)     \
        : "v"(v), "v"(U.x), "v"(U.y), "v"(U.z), "v"(U.w), "v"(V.x), "v"(V.y), "v"(V.z), "v"(V.w))
template <int G>
__device__ inline void dense_fma4(float4 (&acc)[4], float v, const u32x4 (&u)[4]) {
    if (G == 0) {
        SIVF_TWO("0", "1", acc[0], acc[1], u[0], u[1]);
        SIVF_TWO("2", "3", acc[2], acc[3], u[2], u[3]);
    } else if (G == 1) {
        SIVF_TWO("4", "5", acc[0], acc[1], u[0], u[1]);
        SIVF_TWO("6", "7", acc[2], acc[3], u[2], u[3]);
    } else if (G == 2) {
        SIVF_TWO("8", "9", acc[0], acc[1], u[0], u[1]);
        SIVF_TWO("10", "11", acc[2], acc[3], u[2], u[3]);
    } else {
        SIVF_TWO("12", "13", acc[0], acc[1], u[0], u[1]);
        SIVF_TWO("14", "15", acc[2], acc[3], u[2], u[3]);
    }
}
#undef SIVF_TWO
#undef SIVF_STEP

typedef __attribute__((address_space(3))) const u32x4* lds_u32x4;

// steps 4 G .. 4 G + 3 of the 16 pairs e held by each DPP row: slices in LDS
// (panel16: the panel's address + 16 q) or in memory
template <int G>
__device__ inline void dense_hot_load4(u32x4 (&u)[4], uint32_t panel16, const uint2& e) {
    u[0] = *(lds_u32x4)(drow_bcast<4 * G + 0>(e.x) + panel16);
    u[1] = *(lds_u32x4)(drow_bcast<4 * G + 1>(e.x) + panel16);
    u[2] = *(lds_u32x4)(drow_bcast<4 * G + 2>(e.x) + panel16);
    u[3] = *(lds_u32x4)(drow_bcast<4 * G + 3>(e.x) + panel16);
}
template <int G>
__device__ inline void dense_cold_load4(u32x4 (&u)[4], __amdgpu_buffer_rsrc_t r, const uint2& e, uint32_t q16) {
    u[0] = __builtin_amdgcn_raw_buffer_load_b128(r, drow_bcast<4 * G + 0>(e.x) | q16, 0, 0);
    u[1] = __builtin_amdgcn_raw_buffer_load_b128(r, drow_bcast<4 * G + 1>(e.x) | q16, 0, 0);
    u[2] = __builtin_amdgcn_raw_buffer_load_b128(r, drow_bcast<4 * G + 2>(e.x) | q16, 0, 0);
    u[3] = __builtin_amdgcn_raw_buffer_load_b128(r, drow_bcast<4 * G + 3>(e.x) | q16, 0, 0);
}

// over the four DPP rows (v is the same in a row's lanes)
__device__ inline int rows_max(int v) {
    return max(max(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)),
               max(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
}

// A lane's place in a list of pairs: byte offset of its pair in the next chunk of
// 16, and the chunks left; then chunks of fill.
struct DenseList {
    uint32_t at;
    int left;
};

// Pairs are loaded through a descriptor of all pairs (less than 4 GiB), whether
// or not the list has any left: a load that may not happen would make the
// compiler wait for all before it.
__device__ inline uint2 next_pairs(__amdgpu_buffer_rsrc_t ents, DenseList& l, uint32_t fill) {
    const uint32_t at = l.left > 0 ? l.at : fill;
    l.at += 128;
    l.left -= 1;
    const auto v = __builtin_amdgcn_raw_buffer_load_b64(ents, at, 0, 0);
    return make_uint2(v[0], v[1]);
}

// 16 pairs of the LDS rows (e) and CQ groups of four of the others (c) of a
// wave's objects: the latter's slices and the next pairs are in flight while
// the former are added.  The two have sums of their own.  mh, mc: steps left.
template <int CQ>
__device__ inline void dense_round(float4& hot, float4& cold, uint2& c, uint2& e, int mh, int mc, __amdgpu_buffer_rsrc_t ents, DenseList& lc,
                                   DenseList& lh, uint32_t panel16, __amdgpu_buffer_rsrc_t rsrc, uint32_t q16,
                                   uint32_t q8) {
    u32x4 u0[4], u1[4], u2[4], u3[4], a[4];
    uint2 cn = c, en = e;
    if (CQ == 4 && mc > 16) cn = next_pairs(ents, lc, 128 + q8);
    if (mh > 16) en = next_pairs(ents, lh, q8);
    __builtin_amdgcn_sched_barrier(0);
    if (CQ > 0) dense_cold_load4<0>(u0, rsrc, c, q16);
    if (CQ > 1) dense_cold_load4<1>(u1, rsrc, c, q16);
    if (CQ > 2) dense_cold_load4<2>(u2, rsrc, c, q16);
    if (CQ > 3) dense_cold_load4<3>(u3, rsrc, c, q16);
    __builtin_amdgcn_sched_barrier(0);
    const float ev = __uint_as_float(e.y), cv = __uint_as_float(c.y);
    if (0 < mh) {
        dense_hot_load4<0>(a, panel16, e);
        dense_fma4<0>(hot, ev, a);
    }
    if (4 < mh) {
        dense_hot_load4<1>(a, panel16, e);
        dense_fma4<1>(hot, ev, a);
    }
    if (8 < mh) {
        dense_hot_load4<2>(a, panel16, e);
        dense_fma4<2>(hot, ev, a);
    }
    if (12 < mh) {
        dense_hot_load4<3>(a, panel16, e);
        dense_fma4<3>(hot, ev, a);
    }
    __builtin_amdgcn_sched_barrier(0);
    if (CQ > 0) dense_fma4<0>(cold, cv, u0);
    if (CQ > 1) dense_fma4<1>(cold, cv, u1);
    if (CQ > 2) dense_fma4<2>(cold, cv, u2);
    if (CQ > 3) dense_fma4<3>(cold, cv, u3);
    c = cn;
    e = en;
}

// The same with four sums, and eight slices in flight at a time.
template <int CQ>
__device__ inline void dense_round(float4 (&acc)[4], uint2& c, uint2& e, int mh, int mc, __amdgpu_buffer_rsrc_t ents,
                                   DenseList& lc, DenseList& lh, uint32_t panel16, __amdgpu_buffer_rsrc_t rsrc,
                                   uint32_t q16, uint32_t q8) {
    u32x4 u0[4], u1[4], a[4];
    uint2 cn = c, en = e;
    if (CQ == 4 && mc > 16) cn = next_pairs(ents, lc, 128 + q8);
    if (mh > 16) en = next_pairs(ents, lh, q8);
    __builtin_amdgcn_sched_barrier(0);
    const float ev = __uint_as_float(e.y), cv = __uint_as_float(c.y);
    if (CQ > 0) dense_cold_load4<0>(u0, rsrc, c, q16);
    if (CQ > 1) dense_cold_load4<1>(u1, rsrc, c, q16);
    __builtin_amdgcn_sched_barrier(0);
    if (0 < mh) {
        dense_hot_load4<0>(a, panel16, e);
        dense_fma4<0>(acc, ev, a);
    }
    if (4 < mh) {
        dense_hot_load4<1>(a, panel16, e);
        dense_fma4<1>(acc, ev, a);
    }
    __builtin_amdgcn_sched_barrier(0);
    if (CQ > 0) dense_fma4<0>(acc, cv, u0);
    if (CQ > 2) dense_cold_load4<2>(u0, rsrc, c, q16);
    if (CQ > 1) dense_fma4<1>(acc, cv, u1);
    if (CQ > 3) dense_cold_load4<3>(u1, rsrc, c, q16);
    __builtin_amdgcn_sched_barrier(0);
    if (8 < mh) {
        dense_hot_load4<2>(a, panel16, e);
        dense_fma4<2>(acc, ev, a);
    }
    if (12 < mh) {
        dense_hot_load4<3>(a, panel16, e);
        dense_fma4<3>(acc, ev, a);
    }
    __builtin_amdgcn_sched_barrier(0);
    if (CQ > 2) dense_fma4<2>(acc, cv, u0);
    if (CQ > 3) dense_fma4<3>(acc, cv, u1);
    c = cn;
    e = en;
}

// The workgroup's share of all (block, group of four objects): eight blocks at a
// time, one per XCD, over the same objects (their pairs are then read from
// memory once); of the rest's pairs, block-major, an XCD takes an eighth.  Calls
// f(block, first group, past the last), the same for a workgroup's waves.
// blocks * groups < 2^31.
template <typename F>
__device__ inline void each_block(int blocks, int groups, F f) {
    const int xcd = blockIdx.x % kXcds, whole = blocks / kXcds, rest = blocks % kXcds * groups;
    const int mine = (int)((int64_t)xcd * rest / kXcds);
    const int end = whole * groups + (int)((int64_t)(xcd + 1) * rest / kXcds) - mine;
    for (int at = 0; at < end;) {
        int blk = at / groups, g0 = at - blk * groups;
        if (blk < whole) {
            blk = blk * kXcds + xcd;
        } else {
            const int r = mine + at - whole * groups;
            blk = r / groups;
            g0 = r - blk * groups;
            blk += whole * kXcds;
        }
        const int g1 = min(groups, g0 + end - at);
        at += g1 - g0;
        f(blk, g0, g1);
    }
}

// This wave's groups among [g0, g1) of a block: header(g) loads the lane's
// object's header, wanted(g, header) says whether its sums are, done(g, sums,
// wanted) takes them (lane: columns 4 q .. 4 q + 3 of object 4 g + sub).  SUMS:
// partial sums, 2 (32 LDS rows' at a time, and the rest), or 4 of every fourth
// step each, which round less but take registers from slices in flight.  loads:
// += KB requested.
template <int SUMS, typename Header, typename Wanted, typename Done>
__device__ inline void dense_groups(int g0, int g1, __amdgpu_buffer_rsrc_t ents, const u32x4* panel,
                                    __amdgpu_buffer_rsrc_t rsrc, uint32_t& loads, Header header, Wanted wanted,
                                    Done done) {
    const uint32_t q = threadIdx.x & 15, q16 = 16u * q, q8 = 8u * q;
    const uint32_t panel16 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)(char*)panel + q16;
    const int wave = (blockIdx.x / kXcds) * (kDenseThreads / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int step = (gridDim.x / kXcds) * (kDenseThreads / 64);
    const int first = g0 + wave;
    if (first >= g1) return;
    // headers are fetched two groups ahead, first pairs one
    uint2 hd = header(first);
    int nh = 0, nc = 0;
    DenseList lh, lc;
    auto lists = [&](bool want) {
        nh = want ? hdr_hot(hd) : 0;
        nc = want ? hdr_cold(hd) : 0;
        lh = DenseList{hd.x * 8 + q8, chunks16(nh)};
        lc = DenseList{lh.at + 128 * lh.left, chunks16(nc)};
    };
    bool want = wanted(first, hd);
    lists(want);
    uint2 c = next_pairs(ents, lc, 128 + q8), e = next_pairs(ents, lh, q8);
    hd = header(first + step);
    int h;
    for (int g = first; g < g1; g += step) {
        const int mh = rows_max(nh), mc = rows_max(nc);
        const bool nwant = wanted(g + step, hd);
        DenseList mlh = lh, mlc = lc;
        lists(nwant);
        const uint2 cn = next_pairs(ents, lc, 128 + q8), en = next_pairs(ents, lh, q8);
        hd = header(g + 2 * step);
        float4 acc[SUMS];
#pragma unroll
        for (int i = 0; i < SUMS; ++i) acc[i] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        auto round = [&](auto cq) {
            constexpr int CQ = decltype(cq)::value;
            if constexpr (SUMS == 2) dense_round<CQ>(acc[0], acc[1], c, e, mh - h, mc - h, ents, mlc, mlh, panel16, rsrc, q16, q8);
            else dense_round<CQ>(acc, c, e, mh - h, mc - h, ents, mlc, mlh, panel16, rsrc, q16, q8);
        };
        for (h = 0; h < mc || h < mh; h += 16) {
            const int cq = min(4, max(0, mc - h + 3) >> 2);
            loads += 1 + 4u * cq;
            if (SUMS == 2 && (h & 31) == 0 && h > 0) {
                acc[1] = make_float4(acc[0].x + acc[1].x, acc[0].y + acc[1].y, acc[0].z + acc[1].z, acc[0].w + acc[1].w);
                acc[0] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            }
            if (cq == 0) round(std::integral_constant<int, 0>{});
            else if (cq == 1) round(std::integral_constant<int, 1>{});
            else if (cq == 2) round(std::integral_constant<int, 2>{});
            else if (cq == 3) round(std::integral_constant<int, 3>{});
            else round(std::integral_constant<int, 4>{});
        }
        if constexpr (SUMS == 2)
            done(g, make_float4(acc[0].x + acc[1].x, acc[0].y + acc[1].y, acc[0].z + acc[1].z, acc[0].w + acc[1].w), want);
        else
            done(g,
                 make_float4((acc[0].x + acc[1].x) + (acc[2].x + acc[3].x), (acc[0].y + acc[1].y) + (acc[2].y + acc[3].y),
                             (acc[0].z + acc[1].z) + (acc[2].z + acc[3].z), (acc[0].w + acc[1].w) + (acc[2].w + acc[3].w)),
                 want);
        want = nwant;
        c = cn;
        e = en;
    }
}

// f(w[i], i) for all i < n by a workgroup of 1024 threads, whole waves at a time
// (w = 0 and i >= n past the end), 16 bytes a lane; w is 16-byte aligned
template <typename F>
__device__ inline void each_weight(const uint32_t* __restrict__ w, int64_t n, F f) {
    const int64_t quads = n / 4;
#pragma unroll 2
    for (int64_t b = 0; b < quads; b += 1024) {
        const int64_t r = b + threadIdx.x;
        const u32x4 v = r < quads ? reinterpret_cast<const u32x4*>(w)[r] : u32x4{0u, 0u, 0u, 0u};
        const int64_t i = r < quads ? 4 * r : n;
        f(v.x, i);
        f(v.y, i + 1);
        f(v.z, i + 2);
        f(v.w, i + 3);
    }
    const int64_t r = 4 * quads + threadIdx.x;
    f(r < n ? w[r] : 0u, r);
}

// The x > 0 that makes {i : w[i] >= x} the largest such set of at most cap (the
// same on every run: all or none of equal weights).  One workgroup of 1024
// threads; sh: 258 words of LDS.
__device__ inline uint32_t top_weights(const uint32_t* __restrict__ w, int64_t n, uint32_t cap, uint32_t* sh) {
    uint32_t *hist = sh, *prefix = sh + 256, *left = sh + 257;
    const int lane = threadIdx.x & 63;
    if (threadIdx.x == 0) {
        *prefix = 0;
        *left = cap;   // rank of the weight sought among those with the prefix
    }
    // the cap-th largest weight, byte by byte; a wave adds its lanes of one
    // bucket at once (most weights are alike: 0.38 ms for 100,000 lane by lane)
    for (int shift = 24; shift >= 0; shift -= 8) {
        if (threadIdx.x < 256) hist[threadIdx.x] = 0;
        __syncthreads();
        const uint32_t pf = *prefix;
        each_weight(w, n, [&](uint32_t v, int64_t) {
            const uint32_t b = (v >> shift) & 255u;
            unsigned long long todo = ballot(v > 0 && (shift == 24 || (v >> (shift + 8)) == pf));
            while (todo) {
                const uint32_t first = (uint32_t)__builtin_amdgcn_readlane((int)b, __builtin_ctzll(todo));
                const unsigned long long same = ballot(b == first) & todo;
                if (lane == 0) atomicAdd(&hist[first], (uint32_t)__popcll(same));
                todo &= ~same;
            }
        });
        __syncthreads();
        if (threadIdx.x == 0) {
            uint32_t b = 255, before = 0;
            while (b > 0 && before + hist[b] < *left) before += hist[b--];
            *left -= before;
            *prefix = (pf << 8) | b;
        }
        __syncthreads();
    }
    // those at least as heavy: all if they fit, else only the heavier ones
    const uint32_t y = max(*prefix, 1u);
    uint32_t ge = 0;
    each_weight(w, n, [&](uint32_t v, int64_t) { ge += v >= y ? 1u : 0u; });
    ge = (uint32_t)wave_sum_i64(ge);
    if (threadIdx.x == 0) hist[0] = 0;
    __syncthreads();
    if (lane == 0) atomicAdd(&hist[0], ge);
    __syncthreads();
    return hist[0] <= cap ? y : y + 1;
}

}  // namespace sivf
