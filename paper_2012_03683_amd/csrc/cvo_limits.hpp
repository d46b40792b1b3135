// cvo_limits.hpp -- limits and integer rules of a view build and its work plan.
#pragma once
#include <limits>

namespace cvo {

// Output slots are named by ints (a piece's first slot, a query's slot), so a plan
// has fewer than 2^31 of them.  Its totals are counted in 64 bits and compared
// here before anything is sized or written by them: 1.5 million points against
// as many without a cutoff, in 16-point clusters, make 4.4e9 slots.  (A piece has
// at least one slot, so the pieces are within the same limit.)
constexpr unsigned long long kMaxSlots = 1ULL << 31;

constexpr bool plan_fits(unsigned long long pieces, unsigned long long slots)
{
    return slots < kMaxSlots && pieces <= slots;
}

// A call has fewer than 2^31 points on each side.  The passes of a large sort run
// their digit counts on from the reference side to the query side, so a place in
// them is a place among the points of both.
constexpr long long kMaxSidePoints = 1LL << 31;
using SortPlace = unsigned;
static_assert(2 * (kMaxSidePoints - 1) <= std::numeric_limits<SortPlace>::max(), "places of both sides' points");

// Several evaluations share one plan only while its partial moments stay within
// this: beyond, the pass takes tens of milliseconds, the launches saved do
// not count, and the handle would keep the memory of all of them.
constexpr unsigned long long kJointBytes = 4ULL << 30;

constexpr bool joint_fits(unsigned long long slots, unsigned long long bytes_per_slot)
{
    return slots < kMaxSlots && slots * bytes_per_slot <= kJointBytes;
}

// A piece's bucket in the dispatch order (heaviest bucket first), non-decreasing in
// its cost: steps of 96 up to 36,864 (every piece of the default plan: n <= 64
// queries x at most 576), then four buckets an octave, to the largest cost there is
// (64 queries x 2^30 candidates).
constexpr int kCostBuckets = 512;
constexpr unsigned long long kCostLinear = 384 * 96;

constexpr int cost_bucket(unsigned long long cost)
{
    if (cost <= kCostLinear) return (int)(cost / 96);
    const unsigned long long m = cost / (kCostLinear / 4);  // >= 4
    const int octave = 61 - __builtin_clzll(m);
    return 385 + 4 * octave + (int)((m >> octave) & 3);
}

}  // namespace cvo
