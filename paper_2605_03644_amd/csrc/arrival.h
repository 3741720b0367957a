// How the workgroups of one unit (a row tile of one KV head) find out who merges their partials: the states of the arrival
// counter, without any HIP types, so that they can be checked on the CPU.
#pragma once

namespace adapshot {

// The counter holds three counts: the workgroups that have arrived, those among them that do not stay for the merge (they had
// less to do than the others and would wait too long), and those that stayed but gave up before all had arrived.
constexpr unsigned kArrivalPassed = 1u << 10;
constexpr unsigned kArrivalLeft = 1u << 20;
[[gnu::always_inline]] constexpr bool arrived_all(unsigned word, int n) { return (word & 0x3ffu) == (unsigned)n; }
// Of a workgroup that stays: how many that stay arrived before it (the counter held `before`); of a unit of n: how many stay.
[[gnu::always_inline]] constexpr int arrival_rank(unsigned before) { return (int)(before & 0x3ffu) - (int)((before >> 10) & 0x3ffu); }
[[gnu::always_inline]] constexpr int arrival_stayers(unsigned word, int n) { return n - (int)((word >> 10) & 0x3ffu); }

// What a workgroup merges that last saw `word` in the counter: after the last arrival nobody leaves any more (leaving is an
// exchange against a value with fewer arrivals), so all that see all n arrived see the same word.
enum MergeRole { kMergeNothing = 0, kMergeShare = 1, kMergeAll = 2 };
[[gnu::always_inline]] constexpr MergeRole merge_role(unsigned word, int n, bool arrived_last, bool stays) {
    if (!arrived_all(word, n)) return kMergeNothing;
    if (word < kArrivalLeft && arrival_stayers(word, n) > 0) return stays ? kMergeShare : kMergeNothing;
    return arrived_last ? kMergeAll : kMergeNothing;
}

}  // namespace adapshot
