// plan.hpp -- how a force call on a list of rows is split: formed alike on the host and in the
// kernels (a block's length is known only on the device).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace nbody {

constexpr int WG = 256;      // work-items per workgroup
constexpr int TJ = 256;      // j-particles per tile (LDS tile of the lane split; fold interval)
constexpr int LONG_LIST = 7168;  // rows up to which block-step lists have a plane per tile (Spread::whole)

// ------------------------------------------------------------------------------------------
// Work decomposition of one force call, computed identically on host and device from the
// number of i-particles: i-blocks of WG*IPL particles times K contiguous j-ranges (whole
// tiles).  K > 1 only when the i-blocks alone cannot fill `target` work items.
// ------------------------------------------------------------------------------------------
struct ForcePlan {
    int32_t n_i, n_iblk, ntiles, tps, K, items;
    int32_t S;   // slices of a tile's j-slots an i-particle's lanes take (1: every lane all)
    int32_t H;   // helper lanes per slice (quad_tile); S * H lanes share one i-particle
    int32_t ib;  // i-particles per i-block
    int64_t P;   // padded i rows of one partial plane
};

__host__ __device__ inline int32_t log2i(int32_t v) { return 31 - __builtin_clz((uint32_t)v); }

// Lanes per i-particle for a list of n_i with one i per work-item: a workgroup of wg lanes is
// spread over the list, up to smax lanes (at most one wave) per i.
__host__ __device__ inline int32_t lane_split(int32_t n_i, int32_t smax = 64, int32_t wg = WG) {
    if (n_i >= wg) return 1;
    // wg over the least power of two not below n_i
    const int32_t S = n_i > 1 ? wg >> (32 - __builtin_clz((uint32_t)n_i - 1)) : wg;
    return S > smax ? smax : S;
}

// How an arithmetic's lists may be spread over more lanes than lane_split gives, on launches too
// small to fill the chip.  A lane's 256-j tile sum is a serial chain on a wave that issues one
// instruction every four cycles however idle its SIMD is (measured: 185-200 cycles per j, 21 us
// per tile, the same with one wave per SIMD as with four).  Predict + force of all rows, without
// and with the spread: N = 1024 FP32 49 and 19 us, FP64 36 and 15 us; 300 rows at N = 10000 FP32
// 33 and 19 us, double-single 164 and 32 us.
struct Spread {
    int32_t smax;     // most slices
    int32_t hmax;     // 4: helper lanes keep the order of the sums (FP32); 1: none
    int32_t fill;     // lanes per tile that fill the chip (0: lane_split alone)
    int32_t wg = WG;  // lanes that lane_split spreads over a list
    int32_t pack = 0; // lists longer than a workgroup take slices that leave less padding
    // Helpers double the instructions of a pair: a list takes them where a slice has 32 j-slots or
    // more and (tq) the busiest compute unit gets no more than three items, or four where it gets two
    // without them.  With and without: 600 rows of 20000 (4 items, 1 without) 37.7 and 34.0 us, 700 of
    // 16384 (3, 1) 31.9 and 33.6, 300 of 50000 (4, 2) 39.5 and 41.7; 10 of 100000, 16 slices of one
    // row each, 22 and 16.
    int32_t hslices = 8, hfill = 0;
    // More slices for a list: `most` of them, and (tq) only where they spread the work: an item
    // has half the pairs of one before, so twice the items on the busiest compute unit are no gain
    // once they keep its SIMDs busy.  DS 10 rows of 100000 (391 items, then 782) 27 us for 22 with a
    // second doubling of its lanes, 250 of 20000 (316, then 632) 52 for 59.  `scalar`: arithmetics
    // that leave their scalar j-loads with the first doubling; a second one pays only while no
    // compute unit has two items (fixed point, 400 rows: of 8000 17 us for 22, of 20000 31 for 27).
    // The others also look two doublings ahead (DS 40 of 100000, 2, 4 and 5 items: 52 us for 61), and
    // half the pairs on twice two items, four waves a SIMD, gain where a slice is long (DS 200 of
    // 100000 188 us for 200).
    int32_t most = 64;
    int32_t tq = 0;      // tiles per compute unit in 1/4096 (0: not looked at)
    int32_t scalar = 0;
    // Lists of up to so many rows sum every tile in a plane of its own, whatever the target: the blocks
    // that tiled runs take, whose order of sums that is.
    int32_t whole = 0;
};

// Items of n_i rows in S slices that the busiest compute unit gets.
__host__ __device__ inline int32_t items_per_cu(int32_t n_i, int32_t S, int32_t tq) {
    const int32_t ls = log2i(S), ib = WG >> ls;
    return (((n_i + ib - 1) >> (log2i(WG) - ls)) * tq + 4095) >> 12;
}
__host__ __device__ inline bool helpers_pay(int32_t n_i, int32_t S, int32_t tq) {
    const int32_t with = items_per_cu(n_i, 4 * S, tq);
    return with <= 3 || (with == 4 && items_per_cu(n_i, S, tq) >= 2);
}
// ITEMS false: sp.tq is known to be 0.
template <bool ITEMS>
__host__ __device__ inline bool more_slices(int32_t n_i, int32_t S, const Spread &sp) {
    if (S >= sp.most || n_i * S * 2 > sp.fill) return false;
    if (!ITEMS || sp.tq == 0) return true;
    const int32_t now = items_per_cu(n_i, S, sp.tq), then = items_per_cu(n_i, 2 * S, sp.tq);
    if (sp.scalar && S > 1) return then <= 1;
    const int32_t busy = now > 2 ? now : 2;
    if (then < 2 * busy) return true;
    if (sp.scalar) return false;
    if (S <= 2 && now == 2) return true;
    return S * 4 <= sp.most && n_i * S * 4 <= sp.fill && items_per_cu(n_i, 4 * S, sp.tq) < 4 * busy;
}

// Slices of a list longer than a workgroup that takes S: more, up to 4, where the i-blocks of
// fewer rows that they give leave at least 1/16 less padding (a padded row costs as much as a
// true one; below 1/16 the tile staging shared by fewer rows takes the gain).  FP64 and
// double-single only: FP32's tile sums fix the slices, and fixed point would leave its scalar
// j-loads (881 rows at N = 65536 105 and 111 us).  Without and with it: 520 rows at N = 65536
// FP64 106 and 92 us, double-single 335 and 246; 881 rows 127 and 118, 400 and 356; 257 rows at
// N = 524288 390 and 292, 1340 and 937 (calls one after the other, launches included).
__host__ __device__ inline int32_t pack_lanes(int32_t n_i, int32_t S) {
    const auto padded = [n_i](int32_t ib) { return (n_i + ib - 1) & -ib; };  // ib a power of two
    const int32_t r1 = padded(WG), r2 = padded(WG / 2), r4 = padded(WG / 4);
    int32_t rows = S == 1 ? r1 : S == 2 ? r2 : r4;
    const int32_t least = rows >> 4;
    if (S < 2 && rows - r2 >= least) { rows = r2; S = 2; }
    if (S < 4 && rows - r4 >= least) S = 4;
    return S;
}

// Slices S and helper lanes H of each of n_i rows.
template <bool ITEMS = true>
__host__ __device__ inline void row_lanes(int32_t n_i, Spread sp, int32_t &S, int32_t &H) {
    S = lane_split(n_i, sp.smax, sp.wg);
    H = 1;
    if (n_i <= sp.fill) {  // also keeps the products below in range
        if (sp.hmax > 1) {
            if (S <= sp.hslices && n_i * S * 4 <= sp.hfill && (!ITEMS || helpers_pay(n_i, S, sp.tq))) H = 4;
        } else {
            while (more_slices<ITEMS>(n_i, S, sp)) S *= 2;
        }
    }
    if (sp.pack && n_i > WG) S = pack_lanes(n_i, S);
}

// ib_max: WG * (i-particles per work-item).  Lists shorter than a workgroup take the lane
// split whatever the variant (one i per group of lanes), so that a short block costs work in
// proportion to its length.  Where the rows' lanes, on every tile, leave the chip unfilled (no
// more than sp.fill per tile), rows take more lanes: more slices where the order of the sums is
// free, helper lanes where the float tile sums fix it.
__host__ __device__ inline ForcePlan make_plan(int32_t n_i, int32_t n, int32_t ib_max,
                                               int32_t target, int32_t kmax,
                                               Spread sp = Spread{64, 1, 0}) {
    ForcePlan p;
    p.n_i = n_i;
    p.ntiles = (n + TJ - 1) / TJ;
    row_lanes(n_i, sp, p.S, p.H);
    const int32_t L = p.S * p.H;
    const int32_t ib = L > 1 ? WG >> log2i(L) : ib_max;  // powers of two: shifts, not divisions
    p.ib = ib;
    p.n_iblk = (n_i + ib - 1) >> log2i(ib);
    int32_t K = p.n_iblk > 0 ? target / p.n_iblk : 1;
    if (n_i <= sp.whole) K = p.ntiles;
    if (K > kmax) K = kmax;
    if (K > p.ntiles) K = p.ntiles;
    if (K < 1) K = 1;
    p.tps = (p.ntiles + K - 1) / K;
    p.K = (p.ntiles + p.tps - 1) / p.tps;
    p.items = p.n_iblk * p.K;
    p.P = (int64_t)p.n_iblk * ib;
    return p;
}

// Lengths of blocks: up to lo, and from hi + 1 to most.
struct BlockRows {
    int32_t lo, hi, most;
    __host__ __device__ bool has(int32_t rows) const { return rows <= most && (rows <= lo || rows > hi); }
};

// Lengths up to `most` of blocks for which the plan of a target and kmax sums every row tile by tile,
// each in a plane of its own, in the slices of `tiled`.  (A second range: the lists of several
// blocks that take more slices, pack_lanes, have more items and join tiles sooner.)
inline BlockRows rows_by_tiles(int32_t n, int32_t ib_max, int32_t target, int32_t kmax, Spread sp,
                               Spread tiled, int32_t most) {
    BlockRows r{-1, 0, 0};
    for (int32_t m = 1; m <= most; ++m) {
        const ForcePlan p = make_plan(m, n, ib_max, target, kmax, sp);
        int32_t S, H;
        row_lanes(m, tiled, S, H);
        const bool alike = p.K == p.ntiles && p.S == S;
        if (!alike && r.lo < 0) r.lo = m - 1;
        if (alike) r.most = m;
    }
    if (r.lo < 0) r.lo = r.most;
    for (int32_t m = r.lo + 1; m < r.most; ++m) {
        const ForcePlan p = make_plan(m, n, ib_max, target, kmax, sp);
        int32_t S, H;
        row_lanes(m, tiled, S, H);
        if (p.K != p.ntiles || p.S != S) r.hi = m;
    }
    return r;
}

}  // namespace nbody
