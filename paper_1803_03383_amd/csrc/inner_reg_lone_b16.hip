// Instantiations of the register-resident inner loop with one chain wave and helper waves on
// the other SIMDs (16 bits; see inner_reg_lone_impl.hpp).
#include "inner_reg_lone_impl.hpp"

namespace halp {
int launch_inner_reg_lone_b16(const InArgs& a, int upl, int R, bool pair, hipStream_t s) {
  using innerlone::launch_one;
  if (upl == 1) return launch_one<16, 1, 64, true>(a, R, s);
  if (upl == 2) return pair ? launch_one<16, 2, 64, true>(a, R, s) : launch_one<16, 2, 64, false>(a, R, s);
  if (upl == 4) return pair ? launch_one<16, 4, 64, true>(a, R, s) : launch_one<16, 4, 64, false>(a, R, s);
  if (upl == 8) return launch_one<16, 8, 64, false>(a, R, s);
  return HALP_ERR_UNSUPPORTED;
}
}  // namespace halp
