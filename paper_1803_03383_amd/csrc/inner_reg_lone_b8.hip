// Instantiations of the register-resident inner loop with one chain wave and helper waves on
// the other SIMDs (8 bits; see inner_reg_lone_impl.hpp).
#include "inner_reg_lone_impl.hpp"

namespace halp {
int launch_inner_reg_lone_b8(const InArgs& a, int upl, int lanes, int R, bool pair, hipStream_t s) {
  using innerlone::launch_one;
  if (lanes == 16 && upl == 2) return launch_one<8, 2, 16, true>(a, R, s);
  if (upl == 2) return pair ? launch_one<8, 2, 64, true>(a, R, s) : launch_one<8, 2, 64, false>(a, R, s);
  if (upl == 4) return pair ? launch_one<8, 4, 64, true>(a, R, s) : launch_one<8, 4, 64, false>(a, R, s);
  if (upl == 8) return launch_one<8, 8, 64, false>(a, R, s);
  return HALP_ERR_UNSUPPORTED;
}
}  // namespace halp
