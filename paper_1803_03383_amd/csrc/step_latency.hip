// Measurement aid: the dependent chain of one inner-loop step of Algorithm 4 at 8 bits,
// with nothing beside it.  One workgroup per CU, `waves` waves, each lane two coordinates;
// per step: two 24-bit multiply-adds, the DPP fold, the wave's sum through one LDS word and
// a barrier, the add of the waves' sums, the fp64 scalar path of gamma (conversion, three
// products, one sum, floor, conversion, clamp) and the update of the two coordinates
// (multiply-add, shift, add, clamp).  No row is fetched, no random bit drawn, nothing is
// counted: row values and rounding terms are lane constants.  The time per step of this
// kernel is the latency floor of the several-wave register kernels with one chain per CU
// (`waves` = 2 or 4; `waves` = 1 runs the chain of the one-chain-wave form, further down).
#include "halp_device.hpp"
#include "halp_internal.hpp"
#include "inner_reg_lone_impl.hpp"

namespace halp {
namespace {

template <int NW>
__global__ __launch_bounds__(64 * NW) void step_latency_kernel(int64_t steps, double dscale, double aB,
                                                              double inv_s, uint32_t* out) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  __shared__ __attribute__((aligned(16))) int s_part[2][16];
  __shared__ int s_dump[64 * NW];
  using Lds = __attribute__((address_space(3))) int;
  if (tid < 32) (&s_part[0][0])[tid] = 0;
  __syncthreads();
  Lds* const slot0 = (Lds*)((lane != 63) ? &s_dump[tid] : &s_part[0][wave]);
  Lds* const slot1 = (Lds*)((lane != 63) ? &s_dump[tid] : &s_part[1][wave]);
  int z0 = (lane * 7 + 1) & 7, z1 = -((lane * 3 + 1) & 3);
  int xs[8][2];
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    xs[s][0] = ((lane * 13 + s * 5 + 1) % 11) - 5;
    xs[s][1] = ((lane * 17 + s * 3 + 1) % 13) - 6;
  }
  const int hv0 = (lane * 29 + 1) & 1023, hv1 = (lane * 31 + 1) & 511;
  const double rho = 0.37;
  for (int64_t t = 0; t < steps; t += 8) {
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const int x0 = xs[s][0], x1 = xs[s][1];
      int D = wave_fold_i32(mad24(x0, z0, mad24(x1, z1, 0)));
      if (NW > 1) {
        *((s & 1) ? slot1 : slot0) = D;
        __syncthreads();
        int q[NW];
#pragma unroll
        for (int w = 0; w < NW; ++w) q[w] = s_part[s & 1][w];
#pragma unroll
        for (int w = NW / 2; w >= 1; w /= 2) {
#pragma unroll
          for (int k = 0; k < w; ++k) q[k] += q[k + w];
        }
        D = q[0];
      } else {
        D = __builtin_amdgcn_readlane(D, 63);
      }
      const double delta = __dmul_rn(dscale, (double)D);
      const double beta = __dmul_rn(aB, delta);
      const double f = floor(__dadd_rn(__dmul_rn(beta, inv_s), rho));
      int nf;
      asm("v_cvt_i32_f64 %0, -%1" : "=v"(nf) : "v"(f));
      const int ng = min(max(nf, -127), 128);
      const int v0 = mad24(ng, x0, hv0 + ((lane + s * 37) & 255));
      const int v1 = mad24(ng, x1, hv1 + ((lane * 3 + s * 11) & 255));
      z0 = min(max(z0 + (v0 >> 8), -128), 127);
      z1 = min(max(z1 + (v1 >> 8), -128), 127);
    }
  }
  out[blockIdx.x * 64 * NW + tid] = (uint32_t)(z0 * 131 + z1);
}

// The same for the form with ONE chain wave, at a row of 512 coordinates (four strips per lane, two
// coordinates per register): per step one packed dot per strip, the DPP fold over 16 lanes, the fp64
// matrix instruction that adds up the rows of lanes and does the multiply-add of gamma, the clamp of
// its high word and three instructions per strip for the update; gammas go to LDS two at a time and a window of
// 8 steps ends with the look at its fractions and a barrier.  A step's record (row values and
// rounding terms) and its rounding draw come from an LDS ring that nobody refills, two steps ahead.
__global__ __launch_bounds__(64) void step_latency_lone_kernel(int64_t steps, double dscale, double aB,
                                                              double inv_s, uint32_t* out) {
  using S = innerlone::Strip<8>;
  using innerlone::int2r;
  using innerlone::int4r;
  constexpr int UPL = 4;
  const int lane = threadIdx.x & 63;
  __shared__ __attribute__((aligned(16))) int4r s_rec[8][2][64];  // [step][values | rounding terms][lane]
  __shared__ double s_c[8];
  __shared__ __attribute__((aligned(16))) int s_hi[8];
  for (int s = 0; s < 8; ++s) {
    int4r xv, cv;
#pragma unroll
    for (int u = 0; u < UPL; ++u) {
      const int a = ((lane * 13 + s * 5 + u) % 11) - 5, b = ((lane * 17 + s * 3 + u) % 13) - 6;
      xv[u] = S::join(a, b);
      cv[u] = S::join((lane * 29 + s * 37 + u) & 511, (lane * 31 + s * 11 + u) & 511);
    }
    s_rec[s][0][lane] = xv;
    s_rec[s][1][lane] = cv;
  }
  if (lane < 8) s_c[lane] = innerlone::kDraw - 0.37;
  int zp[UPL];
#pragma unroll
  for (int u = 0; u < UPL; ++u) zp[u] = S::join(((lane * 7 + u) & 7) << 8, -((lane * 3 + u) & 3) * 256);
  const double scale_t = -dscale * aB * inv_s * 0x1p-8;
  struct Step {
    int4r x, r;
    double c;
  };
  Step ahead[2];
  __syncthreads();
  auto load_step = [&](Step& st, int s) __attribute__((always_inline)) {
    st.x = s_rec[s][0][lane];
    st.r = s_rec[s][1][lane];
    st.c = s_c[s];
  };
  load_step(ahead[0], 0);
  load_step(ahead[1], 1);
  for (int64_t t = 0; t < steps; t += 8) {
    int zsave[UPL];
#pragma unroll
    for (int u = 0; u < UPL; ++u) zsave[u] = zp[u];
    uint32_t nearest = 0xFFFFFFFFu;
    int hi_even = 0;
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const Step st = ahead[s % 2];
      int p0 = S::dot(st.x[0], zp[0]), p1 = S::dot(st.x[1], zp[1]);
      p0 = S::dot(st.x[2], zp[2], p0);
      p1 = S::dot(st.x[3], zp[3], p1);
      int v = p0 + p1;
      v += dpp_quad_swap1(v);
      v += dpp_quad_swap2(v);
      v += dpp_half_mirror(v);
      v += dpp_row_mirror(v);
      const uint64_t bits = __builtin_bit_cast(uint64_t, __builtin_amdgcn_mfma_f64_4x4x4f64((double)v, scale_t, st.c, 0, 0, 0));
      __builtin_amdgcn_sched_barrier(0);
      load_step(ahead[s % 2], (s + 2) % 8);
      __builtin_amdgcn_sched_barrier(0);
      const int hi = (int)(bits >> 32);
      nearest = (uint32_t)bits < nearest ? (uint32_t)bits : nearest;
      const int g = min(max(hi, innerlone::kMagicHi - 127), innerlone::kMagicHi + 128);
      if (s & 1) *reinterpret_cast<int2r*>(&s_hi[s - 1]) = int2r{hi_even, hi};
      else hi_even = hi;
#pragma unroll
      for (int u = 0; u < UPL; ++u) zp[u] = S::add_sat(zp[u], S::mad(st.x[u], g, st.r[u])) & S::kMask;
    }
    if (__builtin_expect(__ballot(nearest <= 2 * innerlone::kNear) != 0, 0)) {
#pragma unroll
      for (int u = 0; u < UPL; ++u) zp[u] = zsave[u];
    }
    asm volatile("s_barrier" ::: "memory");
  }
  uint32_t acc = (uint32_t)s_hi[7];
#pragma unroll
  for (int u = 0; u < UPL; ++u) acc = acc * 131u + (uint32_t)zp[u];
  out[blockIdx.x * 64 + threadIdx.x] = acc;
}

}  // namespace

int launch_debug_step_latency(int waves, int64_t steps, int blocks, uint32_t* out, hipStream_t s) {
  const double dscale = 1.0 / 512, aB = 0.3, inv_s = 8.0;
  const dim3 grid(blocks);
  switch (waves) {
    case 1: hipLaunchKernelGGL(step_latency_lone_kernel, grid, dim3(64), 0, s, steps, dscale, aB, inv_s, out); break;
    case 2: hipLaunchKernelGGL(step_latency_kernel<2>, grid, dim3(128), 0, s, steps, dscale, aB, inv_s, out); break;
    case 4: hipLaunchKernelGGL(step_latency_kernel<4>, grid, dim3(256), 0, s, steps, dscale, aB, inv_s, out); break;
    default: return HALP_ERR_INVALID;
  }
  return hip_ok(hipGetLastError());
}

}  // namespace halp
