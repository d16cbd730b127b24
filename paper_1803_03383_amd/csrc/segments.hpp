// Steps of a segment of an epoch, plain C++: host and device code, and its test, use the same text.
#pragma once

#include <stdint.h>

namespace halp {

// Steps that a chain ending after T steps takes in the segment [t0, t1): none where it ended
// before t0.  Formed in 64 bits: with option II, T may lie more than 2^31 below t0.  A segment's
// records fit the workspace, so its length is far below 2^31.
constexpr int segment_steps(int64_t t0, int64_t t1, int64_t T) {
  const int64_t end = t1 < T ? t1 : T;
  return end > t0 ? (int)(end - t0) : 0;
}

}  // namespace halp
