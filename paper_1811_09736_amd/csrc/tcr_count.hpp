// The count by which the workgroups of a reduction that finishes in one launch find out which of them is done last.
// (No other header is needed here, so that the rule can be tried on the host.)
//
// Every launch adds kFinishCount to the count in total, however many workgroups it has: the first workgroup adds what is
// left, the others one each.  So the sum reaches a multiple of kFinishCount with the last workgroup and not before, no
// launch has to know where the count stands (a recorded launch repeats its arguments) or to set it back, and launches that
// overlap by a caller's mistake spoil their own results but not the count: it is a multiple again when they have ended.
#pragma once
#include <cstdint>

namespace tcr {

constexpr uint32_t kFinishCount = 256;        // a power of two: the count wraps at 2^32.  At least as many as workgroups
constexpr uint32_t finish_weight(uint32_t group, uint32_t groups) { return group == 0 ? kFinishCount + 1u - groups : 1u; }
constexpr bool finish_is_last(uint32_t before, uint32_t weight) { return ((before + weight) & (kFinishCount - 1u)) == 0u; }

}  // namespace tcr
