// What the minibatch inner loops share (inner_batch.hip, inner_batch_cut.hip).
#pragma once

#include "halp_device.hpp"
#include "inner_args.hpp"

namespace halp {

// the full-step form: one slice of 64 ndw dwords of a row per workgroup, P of them to a chain
constexpr int kCutMaxB = 128;              // rows per step at most
bool inner_batch_cut_takes(int B, int ndw);  // rows of a step in registers, at that fragment
size_t inner_batch_cut_workspace(const halp_params& p);  // exchange words, and z of wide minibatches
int launch_inner_batch_cut(const halp_handle& h, const InArgs& a, int ndw, int P, hipStream_t s);

typedef short short2v __attribute__((ext_vector_type(2)));

// Sums of 8 values over the 64 lanes of a wave at once: v[m] is this lane's share of sum m.
// Three exchange steps inside each group of 8 lanes (partner lane ^ 7, ^ 2, ^ 1) halve the
// number of values a lane carries while doubling the lanes each covers, leaving lane l with
// sum l % 8 over its group; three more (lane ^ 8, ^ 16, ^ 32) add the groups.  Every lane
// returns the complete sum number l % 8.  Integer sums: the order does not matter.
__device__ __forceinline__ int wave_sums8_i32(const int (&v)[8], int lane) {
  const bool f2 = (lane & 4) != 0, f1 = (lane & 2) != 0, f0 = (lane & 1) != 0;
  int w[4], u[2];
#pragma unroll
  for (int m = 0; m < 4; ++m) w[m] = (f2 ? v[m + 4] : v[m]) + dpp_half_mirror(f2 ? v[m] : v[m + 4]);
#pragma unroll
  for (int m = 0; m < 2; ++m) u[m] = (f1 ? w[m + 2] : w[m]) + dpp_quad_swap2(f1 ? w[m] : w[m + 2]);
  int r = (f0 ? u[1] : u[0]) + dpp_quad_swap1(f0 ? u[0] : u[1]);
  r += __builtin_amdgcn_update_dpp(0, r, 0x128, 0xF, 0xF, false);  // row_ror:8 = lane ^ 8
  r += __builtin_amdgcn_ds_swizzle(r, 0x401F);                      // lane ^ 16
  r += __shfl_xor(r, 32);
  return r;
}

// the same for M = 2 or 4 values: lane l returns sum number l % M; M = 8: as above
template <int M>
__device__ __forceinline__ int wave_sums_i32(const int (&v)[M], int lane) {
  static_assert(M == 2 || M == 4 || M == 8);
  if constexpr (M == 8) {
    return wave_sums8_i32(v, lane);
  } else {
    const bool f1 = (lane & 2) != 0, f0 = (lane & 1) != 0;
    int r;
    if constexpr (M == 4) {
      int u[2];
#pragma unroll
      for (int m = 0; m < 2; ++m) u[m] = (f1 ? v[m + 2] : v[m]) + dpp_quad_swap2(f1 ? v[m] : v[m + 2]);
      r = (f0 ? u[1] : u[0]) + dpp_quad_swap1(f0 ? u[0] : u[1]);
    } else {
      r = (f0 ? v[1] : v[0]) + dpp_quad_swap1(f0 ? v[0] : v[1]);
      r += dpp_quad_swap2(r);
    }
    r += __builtin_amdgcn_update_dpp(0, r, 0x124, 0xF, 0xF, false);  // row_ror:4: the four quads of a row
    r += __builtin_amdgcn_update_dpp(0, r, 0x128, 0xF, 0xF, false);  // row_ror:8
    r += __builtin_amdgcn_ds_swizzle(r, 0x401F);                     // lane ^ 16
    r += __shfl_xor(r, 32);
    return r;
  }
}

__device__ __forceinline__ double logistic_dl(double a, double y) {
  return __ddiv_rn(-y, __dadd_rn(1.0, halp_exp(__dmul_rn(y, a))));
}

}  // namespace halp
