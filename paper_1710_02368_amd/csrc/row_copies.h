// How much of a round's data is copied into aligned rows at a time (bf16
// contexts whose data rows fit no 16-byte load).  Host arithmetic, no HIP.
#pragma once

#include <stdint.h>

#include <algorithm>

namespace agn {

// A copy holds the mini-batches of as many local steps as fit in 256 MiB, so
// that one launch serves many steps, and of one step where that alone is
// larger; a step (or an evaluation's rows) of more than 2 GiB is not copied
// and its products read the rows where they lie.
constexpr int64_t kRowCopyElements = (int64_t)1 << 27;
constexpr int64_t kRowCopyMost = (int64_t)1 << 30;

// local steps of `step` elements each per copy, of a round of `lambda` steps
// (0: no copy)
inline int row_copy_steps(int64_t step, int lambda) {
  if (step > kRowCopyMost) return 0;
  return (int)std::min<int64_t>(lambda, std::max<int64_t>(1, kRowCopyElements / step));
}

}  // namespace agn
