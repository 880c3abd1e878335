// Goes through the orders of events of the workgroups of one tile that meet (lords_meet.h), every one of them or `walks` drawn
// ones, and returns what went wrong first:
// 0 nothing, 1 a slice finished before all parts were there, 2 a slice finished twice or never, 3 the word not back at zero.
#include <cstdint>
#include <random>
#include <set>
#include <vector>
#include "../paper_2601_22716_amd/csrc/lords_meet.h"

using namespace lords;

namespace {
enum Phase : uint8_t { kWorking, kWaiting, kSeen, kFinishing, kLate, kLateFinishing, kGone };
struct State {
    uint32_t word = 0, answers[8] = {};                    // slices that this workgroup has taken
    uint8_t phase[8] = {}, finished[8] = {};
    bool operator<(const State &o) const
    {
        for (int w = 0; w < 8; ++w) {
            if (phase[w] != o.phase[w]) return phase[w] < o.phase[w];
            if (finished[w] != o.finished[w]) return finished[w] < o.finished[w];
            if (answers[w] != o.answers[w]) return answers[w] < o.answers[w];
        }
        return word < o.word;
    }
};
}  // namespace

extern "C" int meet_orders(int log, int may_give_up, int walks)
{
    const int W = 1 << log;
    std::set<State> seen;
    std::vector<State> todo{State{}};
    std::mt19937 rng(7);
    const bool all = walks == 0;
    while (!todo.empty()) {
        const State s = todo[all ? todo.size() - 1 : rng() % todo.size()];
        if (all) todo.pop_back();
        else todo.clear();                                 // (a walk: one of the next states, the others forgotten)
        if (all && !seen.insert(s).second) continue;
        bool end = true, arrived = true;
        for (int w = 0; w < W; ++w) {
            end &= s.phase[w] == kGone;
            arrived &= s.phase[w] != kWorking;
        }
        if (end) {
            for (int w = 0; w < W; ++w)
                if (s.finished[w] != 1) return 2;
            if (s.word != 0) return 3;
            if (--walks > 0) todo.push_back(State{});
            continue;
        }
        for (int w = 0; w < W; ++w) {
            State n = s;
            const uint8_t phase = s.phase[w];
            if (phase == kWorking) {                       // its parts are in memory
                n.word += meet_unit(log);
                n.phase[w] = kWaiting;
                todo.push_back(n);
            } else if (phase == kWaiting) {                // it looks, or has looked often enough
                if (s.word & kMeetAllThere) {
                    n.phase[w] = s.word & kMeetSlices ? kSeen : kFinishing;
                    todo.push_back(n);
                }
                if (may_give_up) {
                    n = s;
                    n.word += 1u << w;
                    n.phase[w] = s.word & kMeetAllThere ? kLate : kGone;
                    todo.push_back(n);
                }
            } else if (phase == kSeen || phase == kLate) { // it takes the slices that were left
                n.answers[w] = s.word & kMeetSlices;
                n.word &= ~kMeetSlices;
                n.phase[w] = phase == kSeen ? kFinishing : kLateFinishing;
                todo.push_back(n);
            } else if (phase != kGone) {
                if (!arrived) return 1;
                for (int t = 0; t < W; ++t) n.finished[t] += (s.answers[w] >> t & 1) + (phase == kFinishing && t == w);
                n.word += meet_leave(log, s.answers[w], phase == kFinishing);
                n.answers[w] = 0;
                n.phase[w] = kGone;
                todo.push_back(n);
            }
        }
    }
    return 0;
}

// Workgroups of a launch that are given no tile's part, one that is another's, or a tile's parts on two XCDs: 0 if every part has one.
extern "C" int meet_places_wrong(int xcd, int tiles, int log)
{
    std::vector<int> seen((size_t)tiles << log, 0), on(tiles, -1);
    int wrong = 0;
    for (int bx = 0; bx < (8 * ((tiles + 7) / 8)) << log; ++bx) {
        int tile, part;
        if (!lords::meet_place(bx, xcd, tiles, log, tile, part)) continue;
        if (tile < 0 || tile >= tiles || part < 0 || part >> log) { ++wrong; continue; }
        wrong += seen[((size_t)tile << log) + part]++ != 0;
        wrong += on[tile] >= 0 && on[tile] != (bx & 7);
        on[tile] = bx & 7;
    }
    for (int s : seen) wrong += s != 1;
    return wrong;
}
