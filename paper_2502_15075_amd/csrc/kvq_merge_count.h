// How a launch finds out which of the workgroups that write records for one (batch, kv head) finishes last.  The rules
// alone, without the memory operations between them, so that a program on the host can walk every order in which they can
// meet (tests/merge_count_check.cpp).
//
// One 64-bit word per (batch, kv head) lies behind the records: the launch's number, 48 bits, above a 16-bit count.  A word
// without this launch's number counts as zero, whatever it holds: the bytes of a fresh workspace, records of another
// shape, a count that calls overlapping on one workspace left wrong.  Nothing that went wrong before is taken over.
// A workgroup
//   1. raises the word to its launch's number with count 0 (an atomic maximum whose result nobody waits for), then stores
//      its records, and waits until all of that has been performed;
//   2. adds 1 to the word.  The one that brings the count to the number of records (merge_last) reads them all back,
//   3. and stores the number with count 0 again, for a replay from a graph, which carries the same number.
// Numbers grow from launch to launch and start above every pattern of a binary32 number, so that the maximum finds less in
// the word almost always.  Where it does not (a fresh workspace full of ones, a replay after launches with greater numbers),
// the addition returns a word without the number (merge_unmarked), and the workgroup counts itself in the long way: it swaps
// number and count 1 in for the very value it has seen last, or adds again once another has done so.
// All of it is device-scope and relaxed; the order is carried by the wait in 1.
#pragma once

namespace kvq {

using MergeWord = unsigned long long;
constexpr MergeWord kMergeCountBits = 0xFFFFull;
constexpr MergeWord kFirstLaunch = 0xFFF000000000ull, kLaunches = 1ull << 36;     // (then from the start: the long way, once)

constexpr MergeWord merge_tag(MergeWord launch) { return (kFirstLaunch + launch % kLaunches) << 16; }
constexpr bool merge_unmarked(MergeWord seen, MergeWord tag) { return (seen & ~kMergeCountBits) != tag; }
constexpr bool merge_last(MergeWord before, int records) { return (int)(before & kMergeCountBits) + 1 == records; }

}  // namespace kvq
