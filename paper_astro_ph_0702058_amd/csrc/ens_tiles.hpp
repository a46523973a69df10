// ens_tiles.hpp -- gfx950 device code of an ensemble's run in one launch.
//
// The clusters of an ensemble are independent, so a cluster needs no global step, only its own.
// A team of T resident workgroups takes one cluster of T tiles at a time and integrates it to the
// end (tiles.hpp's block step, one workgroup per tile, the FP64 state of a particle in the
// registers of its work-item), then takes the next cluster of that many tiles from their queue.
// Teams of different sizes run side by side; nothing waits outside a team once all workgroups are
// resident (roll_call), and every wait is bounded.
//
// What it replaces: global steps of two launches, in which every cluster shares the latency of
// every step (about 50 us) and the number of steps is that of the cluster with the most.  512
// clusters of 64 to 4096 particles (2411 tiles, 1024 workgroups resident) to t = 1/16, FP32: 33
// against 68 ms with the energies, to t = 1: 463 against 660 ms in two lanes.  A step takes a lone
// team 17-19 us (the meetings and loads of tiles.hpp, 32 rows per pass of 32 j a lane); with the
// device full 24-31 us, four waves a SIMD sharing its issue.  Four waves per SIMD in FP32 (103
// spilled registers, outside the pair loop) against three: 35 and 38 ms; FP64 43 and 40 ms.  The
// records and the partial sums share the planes that the global steps had (padded records and
// sums of their own took 1.3 times the workspace and 5 % less time).
#pragma once

#include "tiles.hpp"

namespace nbody {

constexpr int ET_TILES = 32;   // most tiles of a cluster (a byte of LDS per possible block row)
constexpr int ET_WGS = 1024;   // most workgroups of a launch
constexpr int ET_ROWS = ET_TILES * TJ;

struct EnsTeam {
    int32_t tiles;       // workgroups of the team
    int32_t first;       // place in the queue order of the team's first cluster
    int32_t cls;         // queue counter
    int32_t last;        // end of the queue
};

// The host's tables for one launch, in one array of words.
struct EnsTables {
    int32_t *queue;              // clusters by tiles, then decreasing work
    int32_t *wg_team, *wg_tile;  // [ET_WGS]
    EnsTeam *team;               // [ET_WGS]
    int32_t *next;               // [ET_TILES + 1] next place of each queue
    EnsTables() = default;
    __host__ EnsTables(int32_t *p, int32_t clusters)
        : queue(p), wg_team(p + ((clusters + 3) & ~3)), wg_tile(wg_team + ET_WGS),
          team((EnsTeam *)(wg_tile + ET_WGS)), next((int32_t *)(team + ET_WGS)) {}
    static size_t words(int32_t clusters) {
        return (size_t)((clusters + 3) & ~3) + 6 * ET_WGS + ET_TILES + 1;
    }
};

struct EnsTilesArgs {
    EnsView e;
    StateRW s;
    double eta;
    int32_t steps;               // most block steps of a cluster
    uint64_t epoch;              // first epoch (above every epoch published before)
    EnsTables t;
    uint64_t *assign;            // [teams] turn << TL_SHIFT | place: the team's current cluster
    uint64_t turn;               // first turn (above every turn published before)
    const int32_t *tile_off;     // tiles before each cluster
    uint64_t *roll;              // as TilesArgs'
    uint64_t present;
    uint32_t polls;
    uint64_t *word;              // [total tiles][3]: words by epoch parity, then the arrival
};

// The kernel's arguments read again from the kernel-argument segment (tiles_args).
__device__ __forceinline__ EnsTilesArgs ens_tiles_args() {
    auto *p = (const __attribute__((address_space(4))) EnsTilesArgs *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    EnsTilesArgs a;
    __builtin_memcpy(&a, (const EnsTilesArgs *)p, sizeof a);
    return a;
}

// A cluster's partial planes in a run by a team: [T][n_c] rows of 7 sums, the row of member m of
// tile t at t TJ + m.  A tile's pull on its own rows stays in its workgroup's LDS, and those rows
// of its plane hold the records that it publishes (7 words each).
constexpr int ET_WORDS = 7;

// Sum over the T partial planes of one of a row's sums, in plane order (ens_row_sums); own: that
// of plane `tile`.
__device__ __forceinline__ double ens_planes_sum(const double *src, int64_t stride, int32_t T,
                                                 int32_t tile, double own) {
    double o = 0.0;
    int32_t k = 0;
    for (; k + 8 <= T; k += 8) {
        double v[8];
#pragma unroll
        for (int r = 0; r < 8; ++r) v[r] = agent_load(src + (k + r) * stride);
#pragma unroll
        for (int r = 0; r < 8; ++r) o += k + r == tile ? own : v[r];
    }
    for (; k < T; ++k) {
        const double v = agent_load(src + k * stride);
        o += k == tile ? own : v;
    }
    return o;
}

template <class M>
struct EnsTilesSmem {
    typename M::Smem sm;
    double stage[WG / 64][64 * TL_WORDS / 8];  // at least 8 lanes share a row
    double sums[64][ET_WORDS];
    double own[TJ][ET_WORDS];                  // the tile's pull on its own block rows
    uint8_t mem[TJ];                           // the tile's block members
    uint8_t row_tile[ET_ROWS];
    int32_t row_base[64];
    int32_t owner[64];
    int32_t hist[NLEV];
    int32_t cnt[4];
    int32_t late;
    int32_t place;
};

// One cluster by its team; this workgroup owns tile `tile`.  False if the team did not meet.
template <class M>
__device__ bool ens_tiles_cluster(const EnsTilesArgs &a, EnsTilesSmem<M> &z, int32_t c, int32_t tile,
                                  int32_t T, bool &bad, bool &clamp, bool &behind) {
    const EnsView &e = a.e;
    const int32_t tid = threadIdx.x, lane = tid & 63;
    const int32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int32_t lo = e.off[c], n_c = e.off[c + 1] - lo, lmax = e.lmax;
    const int32_t p0 = lo + tile * TJ, n_t = lo + n_c - p0 < TJ ? lo + n_c - p0 : TJ;
    EnsCluster *cl = e.cl + c;
    const bool skip = cl->done;  // the same for the whole team, which still meets at the end
    const bool selected = cl->n_act > 0;  // a block selected before is stepped whatever t_end
    uint64_t *word = a.word + (int64_t)a.tile_off[c] * 3;  // [2][T], then arrivals [T]
    uint64_t *arrive = word + 2 * T;
    double *part = e.partial + e.part_off[c];              // [T][n_c][ET_WORDS]
    const int64_t stride = (int64_t)n_c * ET_WORDS;
    const auto eps2 = eps_as<M>(e.eps2[c]);
    // the particle of this work-item
    const bool in = tid < n_t;
    const int32_t g = p0 + (in ? tid : 0);
    double x[3], v[3], ac[3], k[3];
    double pot, m;
    int64_t tick;
    int32_t level;
    {
        const StateRW s = ens_tiles_args().s;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const int64_t ix = d * (int64_t)s.n + g;
            x[d] = in ? s.x[ix] : 0.0; v[d] = in ? s.v[ix] : 0.0;
            ac[d] = in ? s.a[ix] : 0.0; k[d] = in ? s.k[ix] : 0.0;
        }
        pot = s.pot[g];
        m = in ? s.m[g] : 0.0;
        tick = in ? s.tick[g] : 0;
        level = in ? s.level[g] & (NLEV - 1) : 0;
    }
    int64_t next = in ? tick + ((int64_t)1 << (lmax - level)) : INT64_MAX;  // padding: never
    __syncthreads();
    if (tid < NLEV) z.hist[tid] = 0;
    if (tid < 64) z.owner[tid] = 0;
    if (tid == 0) z.late = 0;
    __syncthreads();
    if (in) atomicAdd(&z.hist[level], 1);
    int64_t t_cur = cl->t_cur, act_sum = 0;
    int32_t stepped = 0;
    bool done = false;
    __syncthreads();
    while (!skip) {
        const uint64_t epoch = a.epoch + (uint64_t)stepped;
        const int32_t par = (int32_t)(epoch & 1);
        // select: the tile's own next block time and members
        const int32_t lf = 63 - __builtin_clzll(__ballot(z.hist[lane] > 0) | 1ull);
        const int64_t t_own = level_time(t_cur, lf, lmax);
        const bool member = next == t_own;
        const uint64_t mask = __ballot(member);
        if (lane == 0) z.cnt[wave] = __popcll(mask);
        __syncthreads();
        int32_t n_own = 0, row = 0;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            row += w < wave ? z.cnt[w] : 0;
            n_own += z.cnt[w];
        }
        row += __popcll(mask & ((1ull << lane) - 1ull));  // of a member, among the tile's
        if (member) {
            const double D = (double)(t_own - tick) * a.s.tick_len;
            // one set of records: if the tile had rows in the last block it waited until every
            // workgroup had read them, and else nobody reads them
            double *r = part + tile * (stride + TJ * ET_WORDS) + row * ET_WORDS;
            z.mem[row] = (uint8_t)tid;
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                double xp, vp;
                predict_one(D, x[d], v[d], ac[d], k[d], xp, vp);
                agent_store(r + d, xp);
                agent_store(r + 3 + d, vp);
            }
            agent_store(r + 6, m);
        }
        stores_done();
        __syncthreads();
        if (tid == 0)
            agent_store(word + par * T + tile, epoch << TL_SHIFT | (uint64_t)lf << 16 | (uint64_t)n_own);
        // gather: the block time and the block rows
        if (tid < T) {
            uint64_t w;
            if (!wait_epoch(word + par * T + tid, epoch, w)) z.late = 1;
            z.owner[tid] = (int32_t)(w & 0xffffff);
        }
        __syncthreads();
        if (z.late) return false;
        const int32_t ow = z.owner[lane];
        const int64_t t_next = level_time(t_cur, wave_max(ow >> 16), lmax);
        if (t_next > e.t_end && !(selected && stepped == 0)) {
            done = true;
            break;
        }
        const int32_t oc = level_time(t_cur, ow >> 16, lmax) == t_next ? ow & 0xffff : 0;
        const int32_t inc = wave_scan_add(oc);
        const int32_t n_act = __builtin_amdgcn_readlane(inc, 63), ob = inc - oc;
        const int32_t base = __builtin_amdgcn_readlane(ob, tile);
        const bool mine = t_own == t_next;  // this tile has block rows
        if (stepped == a.steps) {  // leave the block selected, as a global step does
            if (mine && member) e.active[lo + base + row] = p0 + tid;
            if (tile == 0 && tid == 0) {
                cl->t_next = t_next;
                cl->n_act = n_act;
            }
            break;
        }
        if (wave == 0) z.row_base[lane] = ob;
        if ((lane & 3) == wave)  // the owners dealt to the waves
            for (int32_t i = 0; i < oc; ++i) z.row_tile[ob + i] = (uint8_t)lane;
        {  // predict the tile
            behind = behind || next < t_next;
            const double D = (double)(t_next - tick) * a.s.tick_len;
            double xp[3], vp[3];
#pragma unroll
            for (int d = 0; d < 3; ++d) predict_one(D, x[d], v[d], ac[d], k[d], xp[d], vp[d]);
            M::put(z.sm, tid, xp, vp, m);
        }
        __syncthreads();
        // force: 64 / S rows a wave
        const int32_t S = ens_split(n_act, e.smin), ls = 31 - __builtin_clz(S);
        const int32_t slice = lane & (S - 1);
        double *plane = part + tile * stride;
        for (int32_t q0 = wave << (6 - ls); q0 < n_act; q0 += 4 << (6 - ls)) {
            const int32_t q = q0 + (lane >> ls);
            int64_t to = 0;   // the row of the plane, or -1 - m for the tile's own member m
            double xi[3] = {0.0, 0.0, 0.0}, vi[3] = {0.0, 0.0, 0.0}, mi = 0.0;
            int32_t own = -1;  // the row's own slot in the tile (none on padding)
            if (q < n_act) {
                const int32_t rt = z.row_tile[q];
                const int32_t m = q - z.row_base[rt];
                const double *r = part + rt * (stride + TJ * ET_WORDS) + m * ET_WORDS;
                to = rt == tile ? -1 - m : rt * TJ + m;
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    xi[d] = agent_load(r + d);
                    vi[d] = agent_load(r + 3 + d);
                }
                mi = agent_load(r + 6);
                if (rt == tile) own = z.mem[m];
            }
            const typename M::I ii = M::make_i(xi, vi, mi);
            typename M::Sum F = M::sum_zero();
            tile_sums<M, 2, true, false>(ii, z.sm, slice, S, 1, own, eps2, F);
            lanes_add<M>(F, S);
            double *st = z.stage[wave];
            if (slice == 0) {
                const Out7 o = M::out(F);
#pragma unroll
                for (int d = 0; d < 7; ++d) st[(lane >> ls) * TL_WORDS + d] = o.v[d];
                st[(lane >> ls) * TL_WORDS + 7] = __longlong_as_double((long long)to);
            }
            __builtin_amdgcn_wave_barrier();
            for (int32_t w = lane; w < (64 >> ls) * TL_WORDS; w += 64) {
                const int32_t d = w & 7, at = (int32_t)__double_as_longlong(st[w | 7]);
                if (q0 + (w >> 3) >= n_act || d == 7) continue;
                if (at < 0) z.own[-1 - at][d] = st[w];
                else agent_store(plane + at * ET_WORDS + d, st[w]);
            }
            __builtin_amdgcn_wave_barrier();
        }
        stores_done();
        __syncthreads();
        if (tid == 0) agent_store(arrive + tile, epoch << TL_SHIFT);
        if (mine) {
            uint64_t w;
            if (tid < T && !wait_epoch(arrive + tid, epoch, w)) z.late = 1;
            __syncthreads();
            if (z.late) return false;
            // 64 rows at a time: lane 8 r + d of a unit of 8 rows takes sum d of row r, then the
            // row's own work-item corrects its particle
            const int32_t d = lane & 7;
            for (int32_t c0 = 0; c0 < n_own; c0 += 64) {
                for (int32_t r0 = wave * 8; r0 < 64 && c0 + r0 < n_own; r0 += 32) {
                    const int32_t r = r0 + (lane >> 3);
                    if (c0 + r < n_own && d < 7)
                        z.sums[r][d] = ens_planes_sum(part + (tile * TJ + c0 + r) * ET_WORDS + d, stride, T,
                                                      tile, z.own[c0 + r][d]);
                }
                __syncthreads();
                if (member && row >= c0 && row < c0 + 64) {
                    double o[7];
#pragma unroll
                    for (int j = 0; j < 7; ++j) o[j] = z.sums[row - c0][j];
                    // the corrector on this work-item's registers (a one-particle state)
                    StateRW one{x, v, ac, k, nullptr, &pot, &tick, &level, 1, a.s.tick_len};
                    const int32_t l0 = level;
                    ens_correct_one(e, one, 0, t_next, o, a.eta, bad, clamp);
                    next = tick + ((int64_t)1 << (lmax - level));
                    if (level != l0) {
                        atomicAdd(&z.hist[l0], -1);
                        atomicAdd(&z.hist[level], 1);
                    }
                }
                if (c0 + 64 < n_own) __syncthreads();  // the sums are written again
            }
        }
        t_cur = t_next;
        act_sum += n_act;
        stepped += 1;
        __syncthreads();  // corrected levels precede the next selection
    }
    // the team ends here with the same steps, or the state stays as it was
    {
        const uint64_t epoch = a.epoch + (uint64_t)a.steps + 1;
        uint64_t w;
        if (tid == 0) agent_store(arrive + tile, epoch << TL_SHIFT);
        if (tid < T && !wait_epoch(arrive + tid, epoch, w)) z.late = 1;
        __syncthreads();
        if (z.late) return false;
    }
    if (tile == 0 && tid == 0) {
        if (stepped > 0) {
            cl->t_cur = t_cur;
            cl->n_steps += stepped;
            cl->n_active_sum += act_sum;
            if (done) cl->t_next = t_cur;
        }
        if (done) {
            cl->done = 1;
            cl->n_act = 0;
        }
    }
    if (in && stepped > 0) {
        // the arguments and the place read again: addresses do not stay in registers through
        // the steps
        const StateRW s = ens_tiles_args().s;
        int32_t gw = g;
        asm volatile("" : "+v"(gw));
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const int64_t ix = d * (int64_t)s.n + gw;
            s.x[ix] = x[d]; s.v[ix] = v[d]; s.a[ix] = ac[d]; s.k[ix] = k[d];
        }
        s.pot[gw] = pot; s.tick[gw] = tick; s.level[gw] = level;
    }
    return true;
}

template <class M, int WAVES>
__global__ void __launch_bounds__(WG, WAVES) ens_tiles(EnsTilesArgs a) {
    __shared__ EnsTilesSmem<M> z;
    const int32_t tm = a.t.wg_team[blockIdx.x], tile = a.t.wg_tile[blockIdx.x];
    const EnsTeam team = a.t.team[tm];
    bool bad = false, clamp = false, behind = false, lost = false;
    int32_t place = team.first;
    if (threadIdx.x == 0) {
        const EnsTilesArgs r = ens_tiles_args();
        z.late = !roll_call(r.roll, r.epoch, roll_count(r.roll, r.present), r.polls);
    }
    __syncthreads();
    if (z.late) place = team.last;  // no cluster (a return here cost the loop 2 %: registers)
    for (uint64_t turn = a.turn; place < team.last;) {
        if (!ens_tiles_cluster<M>(a, z, a.t.queue[place], tile, team.tiles, bad, clamp, behind)) {
            lost = true;
            break;
        }
        // the team's next cluster: taken by its first workgroup, read by the others
        turn += 1;
        __syncthreads();
        if (threadIdx.x == 0) {
            uint64_t w = 0;
            if (tile == 0) {
                w = (uint64_t)atomicAdd(a.t.next + team.cls, 1);
                if (team.tiles > 1) agent_store(a.assign + tm, turn << TL_SHIFT | w);
            } else if (!wait_epoch(a.assign + tm, turn, w)) {
                z.late = 1;
            }
            z.place = (int32_t)(w & 0xffffff);
        }
        __syncthreads();
        if (tile != 0 && z.late) {
            lost = true;
            break;
        }
        place = z.place;
    }
    if (bad) a.e.flags[0] = 1;
    if (clamp) a.e.flags[1] = 1;
    if (behind) a.e.flags[2] = 1;
    if (lost) a.e.flags[3] = 1;
}

}  // namespace nbody
