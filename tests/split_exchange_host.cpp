// The exchange of split_exchange.hpp on the CPU: a workgroup's first wave is eight threads, `slots` workgroups run at a time, in the order of
// dispatch, as on a chip with room for that many.  Sums are replaced by marks: share s of a tile may be finished once, with every range's mark there.
#define __device__
#define __forceinline__ inline
#include "split_exchange.hpp"

#include <atomic>
#include <memory>
#include <thread>
#include <vector>

namespace {
constexpr int kLanes = 8;

struct Group {   // the threads of one slot
    std::atomic<uint32_t> arrived{0}, phase{0};
    std::atomic<uint64_t> votes{0};
    uint64_t last = 0;

    uint64_t ballot(int lane, bool b) {
        if (b) votes.fetch_or(1ull << lane);
        const uint32_t now = phase.load();
        if (arrived.fetch_add(1) + 1 == kLanes) {
            last = votes.exchange(0);
            arrived = 0;
            phase.fetch_add(1);
        } else {
            while (phase.load() == now) std::this_thread::yield();
        }
        return last;   // nobody writes it before all have voted again
    }
};

struct Wave {
    int lane;
    Group* group;
    uint32_t load(const uint32_t* p) const { return __atomic_load_n(p, __ATOMIC_SEQ_CST); }
    void store(uint32_t* p, uint32_t v) const { __atomic_store_n(p, v, __ATOMIC_SEQ_CST); }
    uint32_t exchange(uint32_t* p, uint32_t v) const { return __atomic_exchange_n(p, v, __ATOMIC_SEQ_CST); }
    bool compare_exchange(uint32_t* p, uint32_t seen, uint32_t v) const { return __atomic_compare_exchange_n(p, &seen, v, false, __ATOMIC_SEQ_CST, __ATOMIC_SEQ_CST); }
    uint64_t ballot(bool b) const { return group->ballot(lane, b); }
    void pause() const { std::this_thread::yield(); }
};
}  // namespace

// Returns the number of shares that another range than their own finished, or a negative number: -1 a share finished without all sums,
// -2 not once, -3 a flag left up.  flags: tiles * splits * (splits - 1) words, as the launch before left them.
extern "C" int split_exchange_run(int tiles, int splits, int slots, uint32_t epoch, uint32_t probes, uint32_t* flags) {
    const int workgroups = tiles * splits, pairs = splits * (splits - 1);
    std::vector<std::atomic<int>> marks(workgroups * splits), finished(workgroups);   // [tile][range][share], [tile][share]
    std::atomic<int> next{0}, early{0}, elsewhere{0};
    std::vector<std::unique_ptr<Group>> groups;
    std::vector<int> ids(slots);
    std::vector<std::thread> threads;
    for (int s = 0; s < slots; ++s) groups.emplace_back(new Group);
    auto lane_of_slot = [&](int slot, int lane) {
        Group& g = *groups[slot];
        const Wave w{lane, &g};
        for (;;) {
            if (lane == 0) ids[slot] = next.fetch_add(1);
            w.ballot(false);
            const int id = ids[slot];
            w.ballot(false);
            if (id >= workgroups) return;
            const int tile = id / splits, range = id % splits;
            auto mark = [&](int share) { marks[(tile * splits + range) * splits + share] = 1; };
            auto finish = [&](int share) {
                for (int q = 0; q < splits; ++q)
                    if (!(q == range && share == range) && !marks[(tile * splits + q) * splits + share]) ++early;
                ++finished[tile * splits + share];
                if (share != range) ++elsewhere;
            };
            if (lane == 0)
                for (int s = 0; s < splits; ++s)
                    if (s != range) mark(s);
            w.ballot(false);
            uint32_t* const f = flags + tile * pairs;
            bool complete;
            uint32_t held = axonn::split_meet(w, f, splits, range, epoch, probes, &complete);
            if (lane == 0) {
                if (complete) finish(range);
                else mark(range);
            }
            if (complete == (held >> range & 1)) ++early;
            w.ballot(false);
            for (int s = 0; s < splits; ++s)
                if (held >> s & 1)
                    if (axonn::split_settle(w, f, splits, s, epoch) && lane == 0) finish(s);
        }
    };
    for (int s = 0; s < slots; ++s)
        for (int l = 0; l < kLanes; ++l) threads.emplace_back(lane_of_slot, s, l);
    for (std::thread& t : threads) t.join();
    if (early) return -1;
    for (const auto& f : finished)
        if (f != 1) return -2;
    for (int i = 0; i < tiles * pairs; ++i)
        if (flags[i] != 0) return -3;
    return elsewhere;
}
