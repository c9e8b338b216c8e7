// How the K ranges of a tile that each finish a share of it meet: which workgroup adds up which share.
//
// A range that has stored its sums of the other shares publishes that in one flag per other range, and looks for theirs a
// limited number of times.  Found, it finishes its own share.  Not found, it stores its sums of its own share as well and
// hands that share on to a range that has not come yet; that one finishes it, or hands it on in turn.  So no workgroup ever depends
// on one that is not running: with all ranges of a tile on the chip nothing is handed on, and with room for a single workgroup
// the last range of a tile finishes all of its shares.
//
// flags: [share][splits - 1: the other ranges in order], 0 between launches.  Flag (s, q) is the word in which range q meets the
// holder of share s, at first range s:
//   0         range q has not come
//   handed    it has not come, and takes the share over when it comes
//   epoch     its sums of share s are in memory
// Range q's exchange for `epoch` and the holder's compare-and-swap of 0 for `handed` are what decides: a share has one
// holder at any time, and a holder that finds all of the share's flags at `epoch` has all the sums.  It takes the flags down, which
// nobody looks at any more: a launch replayed from a captured graph carries the same epoch.
//
// A Wave is the first wave of a workgroup: the flag operations at device scope, a lane number, a ballot.  What a range has
// stored has to be acknowledged before it comes here, and loads of what it finds are to go past its caches: no fences.
#pragma once
#include <cstdint>

namespace axonn {

__device__ __forceinline__ uint32_t split_handed(uint32_t epoch) { return ~epoch; }   // epoch: neither 0 nor ~0

// Range `range` comes.  Returns the shares that it now holds, a bit each: those handed on to it, and its own unless that is complete, where
// it says so in `complete`.  The same on all lanes.
template <class Wave>
__device__ __forceinline__ uint32_t split_meet(const Wave& w, uint32_t* flags, int splits, int range, uint32_t epoch, uint32_t probes, bool* complete) {
    const int others = splits - 1, other = w.lane + (w.lane >= range ? 1 : 0);
    uint32_t* const ours = flags + range * others + w.lane;
    uint32_t before = 0;
    bool missing = false;
    if (w.lane < others) {
        before = w.exchange(flags + other * others + (range - (range > other ? 1 : 0)), epoch);
        missing = w.load(ours) != epoch;
        for (; missing && probes > 0; --probes) {
            w.pause();
            missing = w.load(ours) != epoch;
        }
    }
    *complete = w.ballot(missing) == 0;
    if (*complete && w.lane < others) w.store(ours, 0u);
    const uint32_t handed = (uint32_t)w.ballot(w.lane < others && before == split_handed(epoch));   // by lane; share `range` is not among them
    const uint32_t below = (1u << range) - 1;
    return (handed & below) | (handed & ~below) << 1 | (*complete ? 0u : 1u << range);
}

// The holder of `share`, whose own sums of it are in memory: true: all are, the holder finishes it; false: handed on.
template <class Wave>
__device__ __forceinline__ bool split_settle(const Wave& w, uint32_t* flags, int splits, int share, uint32_t epoch) {
    uint32_t* const flag = flags + share * (splits - 1) + w.lane;
    const bool mine = w.lane < splits - 1;
    for (;;) {   // splits times at most: a hand-over that fails has found one more range there
        const uint32_t seen = mine ? w.load(flag) : epoch;
        const uint64_t missing = w.ballot(seen != epoch);
        if (missing == 0) {
            if (mine) w.store(flag, 0u);
            return true;
        }
        const bool first = w.lane == __builtin_ctzll(missing);
        if (w.ballot(first && w.compare_exchange(flag, seen, split_handed(epoch))) != 0) return false;
    }
}

}  // namespace axonn
