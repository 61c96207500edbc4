// kp_rules.hpp -- the arithmetic of the run's host-side decisions, without HIP, so
// that it can be checked on its own.
#pragma once
#include <stddef.h>
#include <stdint.h>

namespace kp {

// Bytes that a buffer of `have` elements must find free before it can hold
// `need`: nothing, or, as it is replaced, all of the new one.
constexpr size_t grow_bytes(size_t need, size_t have, size_t elem) { return need > have ? need * elem : 0; }

// Copies of the cells around the source (HOT_COPIES) that a run takes: those it
// wants, or none where the tally of `tally` doubles would fit but not with
// `per_copy` more for each.  have: doubles allocated; other: bytes that the
// run's other buffers still need.  The copies only save time: they must
// never be why a run is refused, nor why a tally that is held is replaced
// without room for its successor.
constexpr int copies_that_fit(int copies, size_t tally, size_t per_copy, size_t have, size_t other, size_t free_b) {
  return grow_bytes(tally + (size_t)copies * per_copy, have, sizeof(double)) + other <= free_b ? copies : 0;
}

}  // namespace kp
