// LDS of the walks that count their sets.
#pragma once

#include <stdint.h>

namespace surel {

constexpr int kWalkWavesPerBlock = 4;
constexpr int kWalkChains = 2;  // walks a lane moves at a time

// Ids that meet in a slot of a set (distinct.h) go on from it in steps of their own, a byte each: 67, 71, 73 or
// 79 by the id's lowest bits.  They are primes, so slots that are 64 times less than the smallest of them have
// no factor in common with one, and every slot is reached; and a step is less than the slots.
constexpr uint32_t kDistinctSteps = 0x4F494743u;
constexpr int kDistinctSlotsLeast = 128, kDistinctSlotsMost = 64 * 64;

// Slots for a set of at most n_max ids: a power of two, at least twice n_max, or a third more than
// n_max where twice were more than 8 KB and left a compute unit four waves of the walk (131,000 seeds
// of M = 150, m = 9: 4.2 -> 2.8 ms).  Any multiple of 64 above n_max from
// kDistinctSlotsLeast to kDistinctSlotsMost does.
constexpr int distinct_slots(int n_max) {
    int s = 128;
    while (s < 2048 ? s < 2 * n_max : 3 * s < 4 * n_max) s *= 2;
    return s;
}

// LDS for the set of a seed's nodes while walks are made from short records, whose second trip wants waves
// to hide behind: as many workgroups a compute unit as half as many slots again as nodes allow, or
// distinct_slots where those are fewer, and then as many slots as they have room for.  235,000 seeds of
// M = 150, m = 4 1,290 -> 880 us (12 -> 24 waves), of M = 200 1,380 -> 1,067 (20 waves), 120,000 of M = 200,
// m = 9 4,930 -> 2,635 (8 waves); 270,000 of M = 500, m = 3 with half as many again 2,244, with 2,048 (another
// workgroup) 1,892.  From packed records, where lines from memory are what bounds the walks, they are faster with
// fewer waves (1,000,000 seeds of M = 120, m = 5 5,790, with 20 waves 6,000; 400,000 of M = 200, m = 4 3,290 and
// 3,390).
// (At six workgroups free slots are worth more than waves: 235,000 seeds of M = 100, m = 4 with 832 slots
// 569 us, with 576, which eight have room for, 627.)
constexpr int kWalkMostGroups = 6;
struct WalkTable {
    int groups, slots;
};
inline WalkTable walk_table(int32_t M, int32_t m) {
    constexpr int kLds = 160 * 1024 / 4, kLdsPart = kLds / 128;  // words of a compute unit, given out in parts
    const int n = 1 + M * m;
    const int stage = kWalkChains * 64 * (m + 1);
    const int slots = distinct_slots(n) < n + n / 2 ? distinct_slots(n) : n + n / 2;
    WalkTable t{kLds / (kWalkWavesPerBlock * (stage + slots)), 0};
    t.groups = t.groups < 1 ? 1 : t.groups > kWalkMostGroups ? kWalkMostGroups : t.groups;
    const int room = kLds / t.groups / kLdsPart * kLdsPart / kWalkWavesPerBlock - stage;
    t.slots = (room < 5 * n / 2 ? room : 5 * n / 2) / 64 * 64;
    if (t.slots <= n) t.slots = (n + 64) / 64 * 64;
    if (t.slots < kDistinctSlotsLeast) t.slots = kDistinctSlotsLeast;
    if (t.slots > kDistinctSlotsMost) t.slots = kDistinctSlotsMost;  // (more than the 1,921 nodes at most)
    return t;
}

// Whether walks that count their sets have so few waves that the second trip of a step from short records shows,
// and no better a table with them than without.
inline bool walk_waves_are_few(int32_t M, int32_t m) {
    const WalkTable t = walk_table(M, m);
    return t.groups <= 2 && distinct_slots(1 + M * m) >= t.slots &&
           (kWalkChains * 64 * (m + 1) + distinct_slots(1 + M * m)) * kWalkWavesPerBlock * 4 * t.groups <= 160 * 1024;
}

}  // namespace surel
