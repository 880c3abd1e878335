// The count of an output tile that several workgroups finish together (lords_prefill_kernel.h), in plain C++ so that every order of
// events can be gone through on the host.
//
// One word per tile, zero before and after a launch.  Each of the tile's 2^log workgroups adds one unit (2^31 >> log) when its parts
// are in memory and one when it leaves: bit 31 says that all parts are there, and the last to leave brings the word back to zero.
// A workgroup that has waited long enough neither leaves its slice unfinished nor finishes it from parts that are not
// there: it writes what it holds of the slice, sets a bit of its own below the units, and goes.  Who finds all parts there takes such
// slices: it clears the bits with one atomic AND, finishes what bits that gave it, and counts for those who left them.  The
// last to arrive finds what was left before; one that gives up just as the last part has come finds bit 31 set in the
// word that it changes, and takes what there is.  So a slice is finished once, by a workgroup that knows all parts to be
// there, whichever workgroups run at the same time and however long any of them waits.
#pragma once
#include <stdint.h>

#ifdef __HIPCC__
#define LORDS_MEET_HD __host__ __device__ __forceinline__
#else
#define LORDS_MEET_HD inline
#endif

namespace lords {

constexpr uint32_t kMeetAllThere = 0x80000000u;
constexpr uint32_t kMeetSlices = 0xffu;                    // bits of the workgroups (eight at most) that have left their slices

LORDS_MEET_HD uint32_t meet_unit(int log) { return kMeetAllThere >> log; }
// What a workgroup adds to leave: a unit for itself (not if it gave up: who takes its slice counts for it) and for each slice taken.
LORDS_MEET_HD uint32_t meet_leave(int log, uint32_t taken, bool itself) { return meet_unit(log) * ((uint32_t)__builtin_popcount(taken) + (itself ? 1u : 0u)); }

// Where workgroup bx of 8 * (workgroups of a tile) * ceil(tiles / 8) works: a tile's workgroups are on one XCD (bx mod 8), and tiles go to
// the XCDs as evenly as they can, one more to the first ones from `xcd` on.  False: nowhere.
LORDS_MEET_HD bool meet_place(int bx, int xcd, int tiles, int log, int &tile, int &part)
{
    const int slot = bx >> 3, y = (bx - xcd) & 7, more = tiles & 7;
    tile = y * (tiles >> 3) + (y < more ? y : more) + (slot >> log);
    part = slot & ((1 << log) - 1);
    return slot >> log < (tiles >> 3) + (y < more ? 1 : 0);
}

}  // namespace lords
