// The 8-bit softmax inner loop of one row per step (inner_softmax_b8.hip) for its launcher (inner_softmax.hip).
#pragma once

#include "softmax_ahead.hpp"

namespace halp {

using SoftmaxKernel = void (*)(InArgs, Ahead, int, int);

// upl: strips per lane, 1, 2, 4 or 8; expanded: records of 16-bit halves; dense (not both, not 16 classes): a wave less
SoftmaxKernel softmax_b8_kernel(int K, int upl, bool expanded, bool dense);
int softmax_b8_threads(int K, bool dense);

}  // namespace halp
