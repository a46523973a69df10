// run_loop.hpp -- the order of nb_run's launches.  Host code without device calls: nb_run enqueues
// what it is told and reports what the scheduler record says.
#pragma once

#include <algorithm>
#include <cstdint>

namespace nbody {

constexpr int TL_SHIFT = 24;            // a published word: epoch << 24 | what it says
constexpr int32_t TL_STEPS = 1 << 20;   // most block steps of one launch

// The epochs (or turns) of launches whose workgroups meet through words that hold one above
// TL_SHIFT bits: each launch takes as many as it may use, so they are used up in time (a launch
// that ends early has taken them all the same).
struct Epochs {
    static constexpr uint64_t LAST = (1ull << (64 - TL_SHIFT)) - 1;
    uint64_t next = 1;
    // The first of n epochs for the next launch; again: they start over, and the words are to be
    // zeroed before it.
    uint64_t take(uint64_t n, bool &again) {
        again = n > LAST - next;
        if (again) next = 1;
        const uint64_t first = next;
        next += n;
        return first;
    }
};

struct RunLoop {
    enum Path {
        TILES,     // a launch of tile owners, cooperative or (`plain`) not
        RESIDENT,  // one resident workgroup
        CHAIN,     // launches per block step
        APART,     // the separate launches of a step, for particle times that fit no scheduler's
    };
    int32_t chunk;        // steps between two looks at the record
    int64_t max_steps;    // <= 0: no limit
    bool tiles;           // tiled launches are taken
    bool resident;        // what tiles do not take goes to the resident workgroup, else the chain
    // Cooperative launches follow each other whatever their streams, so a small set, which needs a
    // few compute units, starts plainly: launches of several contexts run side by side.  Where they
    // keep each other's workgroups from starting together they leave, and this run's next launches
    // are cooperative.
    bool plain = false;
    int64_t done_steps = 0;
    // a block too large for the tiled path ends its launch and takes the launch chain: for one
    // step, or for ever longer stretches while such blocks come within a few steps of each other
    int32_t chain_left = 0, stretch = 1;
    bool retimed = false, apart = false;

    // The next launches, of k steps: false when the step limit is reached.
    bool next(Path &p, int32_t &k) const {
        k = chunk;
        if (max_steps > 0) k = (int32_t)std::min<int64_t>(k, max_steps - done_steps);
        if (k <= 0) return false;
        p = apart ? APART : tiles && chain_left == 0 ? TILES : resident ? RESIDENT : CHAIN;
        if (p == TILES) k = std::min(k, TL_STEPS);
        else if (chain_left > 0) k = std::min(k, chain_left);
        return true;
    }

    // The device refused a tiled launch: there is none any more in this run.
    void refused() { tiles = false; }

    // The workgroups of a tiled launch did not start together.
    void missed() {
        tiles = plain;
        plain = false;
    }

    // k steps of a path are enqueued.  False: no need to look at the record, since a tiled launch
    // follows and sees for itself that the run is over.
    bool enqueued(Path p, int32_t k) {
        if (p == TILES) return true;
        chain_left = std::max(0, chain_left - k);
        done_steps += k;
        return !(tiles && k == 1 && chain_left == 0);
    }

    // A tiled launch of k steps took `steps` of them.
    void tiled(int32_t k, int32_t steps) {
        done_steps += steps;
        if (steps == k) return;
        stretch = steps < 8 ? std::min(stretch * 2, 1024) : 1;
        chain_left = stretch;
    }

    // A tiled launch found particle times that do not fit the scheduler's (nb_shared_step moves
    // them, a state may be bound in mid-run): the resident workgroup, whose blocks are the
    // smallest t_i + dt_i, takes a set that it holds; a larger one takes tiles again from the
    // state's own time (true: the caller sets it), or else steps apart.
    bool moved() {
        const bool again = !resident && !retimed;
        tiles = again;
        apart = !resident && retimed;
        retimed = again;
        return again;
    }
};

}  // namespace nbody
