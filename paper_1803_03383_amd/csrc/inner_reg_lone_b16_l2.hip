// Instantiations of the register-resident inner loop with one chain wave and helper waves on
// the other SIMDs (16 bits, lambda > 0; see inner_reg_lone_impl.hpp).
#include "inner_reg_lone_impl.hpp"

namespace halp {
int launch_inner_reg_lone_b16_l2(const InArgs& a, int upl, int lanes, int R, bool pair, hipStream_t s) {
  return innerlone::launch_shape<16, true>(a, upl, lanes, R, pair, s);
}
}  // namespace halp
