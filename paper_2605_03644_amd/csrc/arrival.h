// How the workgroups of one unit (a row tile of one KV head) find out who merges their partials: the states of the arrival
// counter, without any HIP types, so that they can be checked on the CPU.
#pragma once

namespace adapshot {

// The counter holds the workgroups that have arrived in its lower half, those that left before all had in its upper half.
constexpr unsigned kArrivalLeft = 0x10000u;
constexpr bool arrived_all(unsigned word, int n) { return (word & 0xffffu) == (unsigned)n; }

// What a workgroup merges that last saw `word` in the counter: after the last arrival nobody leaves any more (leaving is an
// exchange against a value with fewer arrivals), so all that see all n arrived see the same word.
enum MergeRole { kMergeNothing = 0, kMergeShare = 1, kMergeAll = 2 };
constexpr MergeRole merge_role(unsigned word, int n, bool arrived_last, bool waits) {
    if (!arrived_all(word, n)) return kMergeNothing;
    if (waits && word < kArrivalLeft) return kMergeShare;
    return arrived_last ? kMergeAll : kMergeNothing;
}

}  // namespace adapshot
