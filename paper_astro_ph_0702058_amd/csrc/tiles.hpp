// tiles.hpp -- gfx950 device code of whole block-step runs in one launch, for sets of up to
// TL_TILES tiles of TJ particles (too large for one workgroup's LDS, too small for a chain of
// launches per step to be worth its latency).
//
// Every tile of TJ consecutive particles belongs to a workgroup that keeps its FP64 state in
// LDS for the whole launch.  A block step (Sec. 2) is
//   select   each owner finds its tile's finest level, from it the tile's next block time and
//            that block's members, predicts them and publishes their records beside one word
//            (epoch, finest level, member count);
//   gather   every workgroup reads all owners' words: the finest level of all gives the block
//            time, the owners whose own next time is that time give the block, in ascending
//            particle order;
//   force    every workgroup predicts its tile and sums its pull on every block row (its share
//            of the i-blocks where R workgroups hold the same tile), one partial sum per row;
//   correct  the owners of block rows sum the rows' T partials in the order of the launch
//            chain (reduce_correct_level), correct their particles in LDS and give them new
//            levels.
// The R workgroups that hold one tile correct it alike, so their states stay equal.
//
// The workgroups meet twice a step, without fences: words, records and partial sums go through
// relaxed agent-scope atomics, which the eight XCDs' L2 caches do not keep, each producer waits
// for its stores to complete before it stores its word, and each consumer loads after it saw the
// word.  They meet only once all are resident (roll_call): where other work keeps some of them off
// the device, all leave before the first step and nb_run goes on by another path.  (Measured on
// MI355X with 256 workgroups: 2.6 us per meeting; with agent-scope release and acquire fences,
// which write back and invalidate a whole L2, 19 us, and 62 us with 16 KB of records read after
// it.)  Every wait gives up after TL_POLLS polls; the run then reports an error and leaves the
// state as it was before the launch.
//
// The histogram gives the block time only while every particle's t_i is the last multiple of its
// step not after the scheduler's time; then a block is never empty, somebody waits for all
// arrivals in every step, and no workgroup can be two epochs ahead of another (what the reuse of
// words, records and sums every second epoch needs).  The correctors keep it so; of the state that a
// run is given, which calls other than the block steps may have moved, run_start checks it, and the
// launch ends without a step if it does not hold (tile_end TL_MOVED).  (Checked by the owners, as a
// level finer than all in the first words, it cost every step 0.3 us: registers.)
//
// What bounds a step (MI355X, N = 16384 FP32, mean block 230, cycles at 2.15 GHz): the rows' tile
// sums 11000 (one wave's serial chain over 256 j), the two meetings 8000, record and partial-sum
// loads 4000, selection, prediction and the corrector 10000.  Only the waves that hold the tile
// select and only they and the row mappers read the owners' words (every wave for itself: 1000
// cycles of issue more); the corrector's addresses are formed where they are used (hoisted out of
// the step loop they spilled 32 registers): together 10.80 against 10.96 ms for the N = 16384 FP32
// run to t = 1/32, 8.18 against 8.36 ms for N = 5000 FP64 to 1/16.  Per block step against the launch
// chain: N = 2048 FP32 15 and 26 us, N = 5000 FP64 15 and 25 us, N = 16384 FP32 21 and 31 us,
// N = 65536 56 and 66 us.
#pragma once

#include <type_traits>

#include "ensemble.hpp"
#include "run_loop.hpp"

namespace nbody {

constexpr int TL_WG = 1024;          // work-items per workgroup
constexpr int TL_SUB = TL_WG / WG;   // force items a workgroup works on at a time
constexpr int TL_TILES = 256;        // most tiles (one workgroup per compute unit)
constexpr int TL_REPS = 16;          // most workgroups per tile
constexpr int TL_ROWS = 8192;        // most block rows of a step (row map in LDS)
constexpr int TL_WORDS = 8;          // doubles of a published record
constexpr int TL_SUMS = 7;           // doubles of a row's partial sums
constexpr uint32_t TL_POLLS = 1u << 24;  // about a quarter of a minute

// How a launch ended (DevControl::tile_end).
constexpr int32_t TL_RAN = 0;    // its steps, t_end, or a block of more rows than its limit
constexpr int32_t TL_MOVED = 1;  // without a step: a particle's time does not fit the scheduler's
constexpr int32_t TL_APART = 2;  // without a step: its workgroups did not start together

struct TilesArgs {
    StateRW g;           // the state
    JStreamView js;      // the j-particle stream, written at the end
    int32_t *active;
    int32_t T, R;        // tiles, workgroups per tile (grid T * R: tile = block % T)
    int32_t limit;       // most block rows
    BlockRows rows;      // the lengths taken (a block of another ends the launch)
    int32_t steps;       // most block steps
    uint64_t epoch;      // first epoch (above every epoch published before)
    uint64_t *word;      // [2][T] published words (epoch, level << 16 | count), by epoch parity
    uint64_t *roll;      // workgroups that ever started; at ROLL_VERDICT the last launch's verdict
    uint64_t present;    // workgroups that started once all of this launch did
    uint32_t polls;      // looks before a workgroup gives up on the others' start
    uint64_t *arrive;    // [T * R] epoch whose partial sums a workgroup has stored
    double *rec[2];      // [T][TJ][TL_WORDS] published records, by epoch parity
    double *part;        // [2][T][limit][TL_SUMS] partial sums, by epoch parity
    DevControl *ctl;
    double eps2, eta;
    int32_t lmin, lmax;
    Spread sp;           // lanes per block row, as in the launch chain
};

__device__ __forceinline__ uint64_t agent_load(const uint64_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void agent_store(uint64_t *p, uint64_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double agent_load(const double *p) {
    return __longlong_as_double((long long)agent_load((const uint64_t *)p));
}
__device__ __forceinline__ void agent_store(double *p, double v) {
    agent_store((uint64_t *)p, (uint64_t)__double_as_longlong(v));
}
// This wave's stores have completed (they are visible to agent-scope loads).
__device__ __forceinline__ void stores_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Polls *p until its epoch is at least `epoch`; false after TL_POLLS polls.
__device__ __forceinline__ bool wait_epoch(const uint64_t *p, uint64_t epoch, uint64_t &v) {
    for (uint32_t k = 0; k < TL_POLLS; ++k) {
        v = agent_load(p);
        if ((v >> TL_SHIFT) >= epoch) return true;
    }
    return false;
}

// Whether all workgroups of a launch run at the same time.  Each counts itself in as it starts; the
// one that completes the count says go, one that has looked `polls` times in vain says stop, and
// the first word holds for all (an exchange on the verdict, tagged with the launch's epoch), also
// for those that start when others have left.  By one work-item.
constexpr int ROLL_VERDICT = 16, ROLL_WORDS = 32;
__device__ __forceinline__ bool roll_count(uint64_t *roll, uint64_t present) {
    return __hip_atomic_fetch_add(roll, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1 == present;
}
__device__ __forceinline__ bool roll_call(uint64_t *roll, uint64_t epoch, bool complete, uint32_t polls) {
    uint64_t *verdict = roll + ROLL_VERDICT;
    const uint64_t stop = epoch << 1, said = stop | (complete ? 1 : 0);
    uint64_t v = agent_load(verdict);
    if (!complete)
        for (uint32_t k = 0; k < polls && v < stop; ++k) v = agent_load(verdict);
    while (v < stop)  // nobody has spoken; on failure v is what somebody said
        if (__hip_atomic_compare_exchange_strong(verdict, &v, said, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT))
            v = said;
    return v & 1;
}

// First multiple of the step of level l after t (the block time of particles on that level).
__device__ __forceinline__ int64_t level_time(int64_t t, int32_t l, int32_t lmax) {
    return ((t >> (lmax - l)) + 1) << (lmax - l);
}

// Inclusive scans over the 64 lanes of a wave by DPP row shifts and broadcasts (no LDS): sums,
// and the maximum of values >= 0 (the same in every lane).
template <int CTRL, int ROWS>
__device__ __forceinline__ int32_t dpp0(int32_t v) {
    return __builtin_amdgcn_update_dpp(0, v, CTRL, ROWS, 0xf, false);
}
__device__ __forceinline__ int32_t wave_scan_add(int32_t v) {
    v += dpp0<0x111, 0xf>(v);  // row_shr 1, 2, 4, 8
    v += dpp0<0x112, 0xf>(v);
    v += dpp0<0x114, 0xf>(v);
    v += dpp0<0x118, 0xf>(v);
    v += dpp0<0x142, 0xa>(v);  // row_bcast 15, 31
    v += dpp0<0x143, 0xc>(v);
    return v;
}
template <int CTRL, int ROWS>
__device__ __forceinline__ int32_t dpp_max(int32_t v) {
    const int32_t o = dpp0<CTRL, ROWS>(v);
    return o > v ? o : v;
}
__device__ __forceinline__ int32_t wave_max(int32_t v) {
    v = dpp_max<0x111, 0xf>(v);
    v = dpp_max<0x112, 0xf>(v);
    v = dpp_max<0x114, 0xf>(v);
    v = dpp_max<0x118, 0xf>(v);
    v = dpp_max<0x142, 0xa>(v);
    v = dpp_max<0x143, 0xc>(v);
    return __builtin_amdgcn_readlane(v, 63);
}

// j-stream records of a staged tile (after the last step, so that a force call may follow).
__device__ __forceinline__ void write_stream(const JStreamView &js, const ModeF32::Smem &s, int t, int32_t j) {
    js.px[j] = s.x[t]; js.py[j] = s.y[t]; js.pz[j] = s.z[t]; js.vm[j] = s.vm[t];
}
__device__ __forceinline__ void write_stream(const JStreamView &js, const ModeDS::Smem &s, int t, int32_t j) {
    js.q0[j] = s.q0[t]; js.q1[j] = s.q1[t]; js.q2[j] = s.q2[t]; js.q3[j] = s.q3[t];
}
__device__ __forceinline__ void write_stream(const JStreamView &js, const ModeF64::Smem &s, int t, int32_t j) {
    const ModeF64::Rec &r = s.r[t];
    js.px[j] = r.x; js.py[j] = r.y; js.pz[j] = r.z; js.pm[j] = r.m;
    js.vx[j] = r.vx; js.vy[j] = r.vy; js.vz[j] = r.vz;
}

// Sum over planes k = w, w + RW, ... of one of a row's partial sums, in the order of
// reduce_correct_level: four running sums, added 0..3.
__device__ __forceinline__ double planes_sum(const double *src, int64_t stride, int32_t w, int32_t T) {
    double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
    int32_t k = w;
    for (; k + 3 * RW < T; k += 4 * RW) {
        const double b0 = agent_load(src + k * stride), b1 = agent_load(src + (k + RW) * stride);
        const double b2 = agent_load(src + (k + 2 * RW) * stride), b3 = agent_load(src + (k + 3 * RW) * stride);
        s0 += b0; s1 += b1; s2 += b2; s3 += b3;
    }
    for (; k < T; k += RW) s0 += agent_load(src + k * stride);
    return ((s0 + s1) + s2) + s3;
}

// The kernel's arguments read again from the kernel-argument segment: what only the start and
// the end of a launch need does not stay in scalar registers through its steps.
__device__ __forceinline__ TilesArgs tiles_args() {
    auto *p = (const __attribute__((address_space(4))) TilesArgs *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    TilesArgs a;
    __builtin_memcpy(&a, (const TilesArgs *)p, sizeof a);
    return a;
}

// The start of a run to t_end.  levelled: as set_t_end.  check: whether every particle's time fits
// the scheduler's, that is whether its next time is the first multiple of its step after it
// (`moved` was cleared by the launch of sched_newlevel before).
__global__ void __launch_bounds__(WG) run_start(StateRW s, int32_t lmax, int64_t t_end, bool levelled,
                                                bool check, DevControl *ctl) {
    if (check) {
        const int64_t t = ctl->t_cur;
        for (int32_t i = blockIdx.x * WG + threadIdx.x; i < s.n; i += gridDim.x * WG) {
            const int32_t l = s.level[i];
            if (l < 0 || l > lmax || s.tick[i] + ((int64_t)1 << (lmax - l)) != level_time(t, l, lmax))
                ctl->moved = 1;
        }
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        ctl->t_end = t_end;
        ctl->done = 0;
        if (levelled) ctl->n_pending = 0;
    }
}

// The scheduler's time moved on to the state's (its latest particle time), for a launch that ended
// with TL_MOVED.  A particle whose next time lies before the first multiple of the finest step
// after the scheduler's time is behind it, as the launch chain reports.  One workgroup.
__global__ void __launch_bounds__(WG) tiles_time(StateRW s, int32_t lmax, DevControl *ctl) {
    __shared__ int64_t red[WG / 64];
    int64_t late = -ctl->t_cur, next = INT64_MAX, fine = 0;
    for (int32_t i = threadIdx.x; i < s.n; i += WG) {
        const int32_t l = s.level[i] < lmax ? s.level[i] : lmax;
        const int64_t tn = s.tick[i] + ((int64_t)1 << (lmax - l));
        late = -s.tick[i] < late ? -s.tick[i] : late;
        next = tn < next ? tn : next;
        fine = -(int64_t)l < fine ? -(int64_t)l : fine;
    }
    late = wg_min_i64(late, red);
    next = wg_min_i64(next, red);
    fine = wg_min_i64(fine, red);
    if (threadIdx.x == 0) {
        if (next < level_time(ctl->t_cur, (int32_t)-fine, lmax)) ctl->flag_sched = 1;
        else ctl->t_cur = -late;
        ctl->moved = 0;  // run_start looks again
    }
}

// Rows of 8 block rows a wave corrects at a time when the waves share the planes (below).
constexpr int TL_UNITS = 4;

template <class M, int UNR>
__global__ void __launch_bounds__(TL_WG) run_tiles(TilesArgs a) {
    __shared__ double lx[3 * TJ], lv[3 * TJ], la[3 * TJ], lk[3 * TJ], lm[TJ], lpot[TJ];
    __shared__ int64_t ltick[TJ], lnext[TJ];  // t_i, t_i + dt_i
    __shared__ int32_t llevel[TJ];
    __shared__ int32_t hist[NLEV];            // the tile's particles per level
    __shared__ int32_t lmem[2][TJ];           // the tile's block members, by epoch parity
    __shared__ typename M::Smem sm;
    __shared__ double stage[TL_WG / 64][64 * TL_WORDS];
    __shared__ uint8_t row_tile[TL_ROWS];
    __shared__ int32_t row_base[TL_TILES];
    __shared__ int32_t owner[TL_TILES];       // level << 16 | count of every owner
    __shared__ int32_t late, plan_rows;       // block rows and time, for every wave
    __shared__ int64_t plan_t;
    DevControl *ctl = a.ctl;
    const int32_t tid = threadIdx.x, lane = tid & 63;
    const int32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool complete = tid == 0 && roll_count(a.roll, a.present);
    if (ctl->done || ctl->moved) {  // the same for every workgroup
        if (blockIdx.x == 0 && tid == 0) {
            ctl->tile_steps = 0;
            ctl->tile_end = ctl->done ? TL_RAN : TL_MOVED;
        }
        return;
    }
    const int32_t T = a.T, R = a.R, G = T * R, lmax = a.lmax;
    const int32_t tile = (int32_t)blockIdx.x % T, rep = (int32_t)blockIdx.x / T;
    int32_t p0, n_t;
    if (tid < NLEV) hist[tid] = 0;
    if (tid < TL_TILES) owner[tid] = 0;
    if (tid == 0) late = 0;
    __syncthreads();
    {
        const StateRW g = tiles_args().g;
        p0 = tile * TJ;
        n_t = g.n - p0 < TJ ? g.n - p0 : TJ;
        for (int32_t e = tid; e < 3 * TJ; e += TL_WG) {
            const int32_t c = e / TJ, i = e % TJ;
            const int64_t src = c * (int64_t)g.n + p0 + i;
            const bool in = i < n_t;  // padding: at rest, without mass
            lx[e] = in ? g.x[src] : 0.0; lv[e] = in ? g.v[src] : 0.0;
            la[e] = in ? g.a[src] : 0.0; lk[e] = in ? g.k[src] : 0.0;
        }
        if (tid < TJ) {
            const bool in = tid < n_t;
            const int32_t l = in ? g.level[p0 + tid] & (NLEV - 1) : 0;
            lm[tid] = in ? g.m[p0 + tid] : 0.0;
            lpot[tid] = in ? g.pot[p0 + tid] : 0.0;
            ltick[tid] = in ? g.tick[p0 + tid] : 0;
            lnext[tid] = in ? ltick[tid] + ((int64_t)1 << (lmax - l)) : INT64_MAX;  // never a member
            llevel[tid] = l;
            if (in) atomicAdd(&hist[l], 1);
        }
    }
    StateRW s;
    s.x = lx; s.v = lv; s.a = la; s.k = lk; s.m = lm; s.pot = lpot; s.tick = ltick; s.level = llevel;
    s.n = TJ;
    s.tick_len = a.g.tick_len;
    const auto eps2 = eps_as<M>(a.eps2);
    int64_t t_cur = ctl->t_cur, act_sum = 0;
    const int64_t t_end = ctl->t_end;
    if (tid == 0 && !roll_call(a.roll, a.epoch, complete, a.polls)) late = 1;
    int32_t stepped = 0, n_last = 0, last_base = 0, last_cnt = 0, last_par = 0;
    bool done = false, bad = false, clamp = false, behind = false, lost = false;
    __syncthreads();
    if (late) {
        if (blockIdx.x == 0 && tid == 0) {
            ctl->tile_steps = 0;
            ctl->tile_end = TL_APART;
        }
        return;
    }
    while (stepped < a.steps) {
        const uint64_t epoch = a.epoch + (uint64_t)stepped;
        const int32_t par = (int32_t)(epoch & 1);
        uint64_t own_word = 0;
        // select: the tile's own next block time and its members (the waves that hold them)
        if (wave < TJ / 64) {
            const int32_t lf = 63 - __builtin_clzll(__ballot(hist[lane] > 0) | 1ull);
            const int64_t t_own = level_time(t_cur, lf, lmax);
            int32_t n_own = 0, below = 0;
            bool member = false;
            uint64_t mask = 0;
#pragma unroll
            for (int k = 0; k < TJ / 64; ++k) {
                const bool f = lnext[k * 64 + lane] == t_own;
                const uint64_t mk = __ballot(f);
                if (k == wave) {
                    member = f;
                    mask = mk;
                    below = n_own;
                }
                n_own += __popcll(mk);
            }
            if (tid == 0) own_word = epoch << TL_SHIFT | (uint64_t)lf << 16 | (uint64_t)n_own;
            if (member) {
                const int32_t m = below + __popcll(mask & ((1ull << lane) - 1ull));
                lmem[par][m] = tid;
                if (rep == 0) {
                    double xp[3], vp[3];
                    predicted(s, tid, t_own, xp, vp);
                    double *r = a.rec[par] + ((int64_t)p0 + m) * TL_WORDS;
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        agent_store(r + c, xp[c]);
                        agent_store(r + 3 + c, vp[c]);
                    }
                    agent_store(r + 6, lm[tid]);
                    agent_store((uint64_t *)(r + 7), (uint64_t)(p0 + tid));
                }
            }
            stores_done();
        }
        __syncthreads();
        if (rep == 0 && tid == 0) agent_store(a.word + par * T + tile, own_word);
        // gather: every owner's word, then (the waves that predict the tile and those that map
        // the rows, each for itself, four owners a lane) the block time and the block size
        if (tid < T) {
            uint64_t w;
            if (!wait_epoch(a.word + par * T + tid, epoch, w)) late = 1;
            owner[tid] = (int32_t)(w & 0xffffff);
        }
        __syncthreads();
        if (late) {
            lost = true;
            break;
        }
        if (wave < TJ / 64 || wave >= 12) {
            const int4 ow = ((const int4 *)owner)[lane];
            const int32_t o4[4] = {ow.x, ow.y, ow.z, ow.w};
            int32_t fine = 0;
#pragma unroll
            for (int k = 0; k < 4; ++k) fine = o4[k] >> 16 > fine ? o4[k] >> 16 : fine;
            fine = wave_max(fine);
            const int64_t tn = level_time(t_cur, fine, lmax);
            int32_t c4[4], sum = 0;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                c4[k] = level_time(t_cur, o4[k] >> 16, lmax) == tn ? o4[k] & 0xffff : 0;
                sum += c4[k];
            }
            const int32_t inc = wave_scan_add(sum);
            const int32_t rows = __builtin_amdgcn_readlane(inc, 63);
            const bool fits = a.rows.has(rows), taken = tn <= t_end && fits;
            if (wave >= 12) {  // the row map, one owner of each lane per wave
                if (tid == 12 * 64) {
                    plan_t = tn;
                    plan_rows = fits ? rows : 0;
                }
                int32_t b4[4];
                b4[0] = inc - sum;
#pragma unroll
                for (int k = 1; k < 4; ++k) b4[k] = b4[k - 1] + c4[k - 1];
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if (taken && wave == 12 + k) {
                        row_base[4 * lane + k] = b4[k];
                        for (int32_t m = 0; m < c4[k]; ++m) row_tile[b4[k] + m] = (uint8_t)(4 * lane + k);
                    }
            } else if (taken) {  // predict the tile
                double xp[3], vp[3];
                behind = behind || lnext[tid] < tn;
                predicted(s, tid, tn, xp, vp);
                M::put(sm, tid, xp, vp, lm[tid]);
            }
        }
        __syncthreads();
        const int64_t t_next = plan_t;
        if (t_next > t_end) {
            done = true;
            break;
        }
        const int32_t n_act = __builtin_amdgcn_readfirstlane(plan_rows);
        if (n_act == 0) break;  // not for this path
        // force: i-blocks of WG / L rows against the tile, TL_SUB at a time
        int32_t S, H;
        row_lanes<false>(n_act, a.sp, S, H);
        const int32_t L = S * H, ls = 31 - __builtin_clz(L);      // L = 1 << ls
        const int32_t ib = WG >> ls, n_iblk = (n_act + ib - 1) >> (8 - ls);
        const int32_t sub = wave >> 2, tt = tid & (WG - 1);
        const int32_t slice = (tt & (L - 1)) >> (H > 1 ? 2 : 0);  // H is 4 or 1
        double *part = a.part + ((int64_t)par * T + tile) * a.limit * TL_SUMS;
        for (int32_t iblk = rep + R * sub; iblk < n_iblk; iblk += R * TL_SUB) {
            const int32_t q = iblk * ib + (tt >> ls);
            const int32_t q0 = iblk * ib + ((tt & ~63) >> ls);    // the wave's first row
            if (__builtin_amdgcn_readfirstlane(q0) >= n_act) break;
            double xi[3] = {0.0, 0.0, 0.0}, vi[3] = {0.0, 0.0, 0.0}, mi = 0.0;
            int32_t own = -1;  // the row's own slot in the tile (none on padding)
            if (q < n_act) {
                const int32_t rt = row_tile[q];
                const double *r = a.rec[par] + ((int64_t)rt * TJ + (q - row_base[rt])) * TL_WORDS;
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    xi[c] = agent_load(r + c);
                    vi[c] = agent_load(r + 3 + c);
                }
                mi = agent_load(r + 6);
                own = (int32_t)agent_load((const uint64_t *)(r + 7)) - p0;
            }
            const typename M::I ii = M::make_i(xi, vi, mi);
            typename M::Sum F = M::sum_zero();
            tile_sums<M, UNR, true, std::is_same<M, ModeF32>::value>(ii, sm, slice, S, H, own, eps2, F);
            lanes_add<M>(F, L, H);
            // the wave's rows, transposed through its own LDS slice: lanes store consecutive words
            double *st = stage[wave];
            if ((lane & (L - 1)) == 0) {
                const Out7 o = M::out(F);
#pragma unroll
                for (int c = 0; c < 6; ++c) st[(lane >> ls) * TL_WORDS + c] = o.v[c];
                st[(lane >> ls) * TL_WORDS + 6] = -o.v[6];
            }
            __builtin_amdgcn_wave_barrier();
            for (int32_t e = lane; e < (64 >> ls) * TL_WORDS; e += 64) {
                const int32_t r = q0 + e / TL_WORDS, c = e % TL_WORDS;
                if (r < n_act && c < TL_SUMS) agent_store(part + (int64_t)r * TL_SUMS + c, st[e]);
            }
            __builtin_amdgcn_wave_barrier();
        }
        stores_done();
        __syncthreads();
        if (tid == 0) agent_store(a.arrive + blockIdx.x, epoch << TL_SHIFT);
        const int32_t mine = __builtin_amdgcn_readfirstlane(owner[tile]);
        const int32_t cnt = level_time(t_cur, mine >> 16, lmax) == t_next ? mine & 0xffff : 0;
        const int32_t base = __builtin_amdgcn_readfirstlane(row_base[tile]);
        if (cnt > 0) {
            uint64_t v;
            if (tid < G && !wait_epoch(a.arrive + tid, epoch, v)) late = 1;
            __syncthreads();
            if (late) {
                lost = true;
                break;
            }
            // correct: lane 8 r + c of a unit of 8 rows takes sum c of row r.  Few rows: wave w
            // adds the planes k = w mod RW of up to TL_UNITS units, and wave u adds unit u's RW
            // wave sums in order.  More rows: a wave takes whole units, the same sums in the
            // same order.
            int32_t lane_c = lane;  // opaque: addresses are formed here, not spilled all launch
            asm volatile("" : "+v"(lane_c));
            const int32_t units = (cnt + 7) / 8, c = lane_c & 7;
            const int64_t stride = (int64_t)a.limit * TL_SUMS;
            const double *src0 = a.part + (int64_t)par * T * stride + (int64_t)base * TL_SUMS + c;
            const bool spread = units <= TL_UNITS;
            if (spread) {
#pragma unroll
                for (int u = 0; u < TL_UNITS; ++u) {
                    const int32_t m = u * 8 + (lane_c >> 3);
                    if (u < units)
                        stage[wave][u * 64 + lane_c] =
                            m < cnt && c < 7 ? planes_sum(src0 + m * TL_SUMS, stride, wave, T) : 0.0;
                }
                __syncthreads();
            }
            for (int32_t u = wave; u < units; u += RW) {
                const int32_t m = u * 8 + (lane_c >> 3);
                const bool live = m < cnt && c < 7;
                double t = 0.0;
                if (spread) {
                    t = stage[0][u * 64 + lane_c];
#pragma unroll
                    for (int k = 1; k < RW; ++k) t += stage[k][u * 64 + lane_c];
                } else if (live) {
                    const double *src = src0 + m * TL_SUMS;
                    t = planes_sum(src, stride, 0, T);
#pragma unroll 1
                    for (int32_t k = 1; k < RW; ++k) t += planes_sum(src, stride, k, T);
                }
                bad = bad || (live && !__builtin_isfinite(t));
                double v7[7];
#pragma unroll
                for (int k = 0; k < 7; ++k) v7[k] = __shfl(t, (lane_c & ~7) + k, 64);
                if (c == 0 && m < cnt) {
                    const int32_t i = lmem[par][m];
                    // the step is a power of two (its level's), so is its reciprocal
                    const double dt = (double)(t_next - ltick[i]) * s.tick_len;
                    const double idt = __builtin_ldexp(1.0, llevel[i]);
                    const double a1[3] = {v7[0], v7[1], v7[2]}, k1[3] = {v7[3], v7[4], v7[5]};
                    double num, den;
                    const bool ok = correct_particle(s, i, dt, a1, k1, v7[6], t_next, nullptr, &num, &den, idt);
                    bad = bad || !ok;
                    const double dtn = den > 0.0 ? __builtin_sqrt(a.eta * num / den) : __builtin_inf();
                    bad = bad || __builtin_isnan(dtn);
                    clamp = clamp || dtn < s.tick_len;
                    const int32_t l0 = llevel[i], l1 = next_level(dtn, l0, t_next, a.lmin, lmax);
                    lnext[i] = t_next + ((int64_t)1 << (lmax - l1));
                    if (l1 != l0) {
                        llevel[i] = l1;
                        atomicAdd(&hist[l0], -1);
                        atomicAdd(&hist[l1], 1);
                    }
                }
            }
        }
        t_cur = t_next;
        act_sum += n_act;
        n_last = n_act;
        last_base = base; last_cnt = cnt; last_par = par;
        stepped += 1;
        __syncthreads();  // corrected times and levels precede the next selection
    }
    // every workgroup ends here with the same steps, or the state stays as it was
    if (!lost) {
        const uint64_t epoch = a.epoch + (uint64_t)a.steps;
        uint64_t v;
        if (tid == 0) agent_store(a.arrive + blockIdx.x, epoch << TL_SHIFT);
        if (tid < G && !wait_epoch(a.arrive + tid, epoch, v)) late = 1;
        __syncthreads();
        lost = late != 0;
    }
    if (lost) {
        if (tid == 0) ctl->flag_wait = 1;
        return;
    }
    if (bad) ctl->flag_nonfinite = 1;
    if (clamp) ctl->flag_dtmin = 1;
    if (behind) ctl->flag_sched = 1;
    if (blockIdx.x == 0 && tid == 0) {
        ctl->n_pending = 0;  // levels are current
        ctl->tile_steps = stepped;
        ctl->tile_end = TL_RAN;
        if (stepped > 0) {
            ctl->t_cur = t_cur;
            ctl->t_next = t_cur;
            ctl->n_steps += stepped;
            ctl->n_active_sum += act_sum;
        }
        ctl->n_act = done ? 0 : n_last;
        if (done) ctl->done = 1;
    }
    if (rep != 0 || stepped == 0) return;
    const TilesArgs ea = tiles_args();
    const StateRW g = ea.g;
    for (int32_t e = tid; e < 3 * TJ; e += TL_WG) {
        const int32_t c = e / TJ, i = e % TJ;
        if (i < n_t) {
            const int64_t dst = c * (int64_t)g.n + p0 + i;
            g.x[dst] = lx[e]; g.v[dst] = lv[e]; g.a[dst] = la[e]; g.k[dst] = lk[e];
        }
    }
    if (tid < n_t) {
        g.pot[p0 + tid] = lpot[tid]; g.tick[p0 + tid] = ltick[tid]; g.level[p0 + tid] = llevel[tid];
        write_stream(ea.js, sm, tid, p0 + tid);
    }
    for (int32_t m = tid; m < last_cnt; m += TL_WG)
        ea.active[last_base + m] = p0 + lmem[last_par][m];
}

}  // namespace nbody
