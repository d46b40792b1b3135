// cvo_limits.hpp -- limits of a view build and its work plan, in host arithmetic.
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

}  // namespace cvo
