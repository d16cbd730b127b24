// Records of the softmax inner loops, see softmax_ahead.hpp.
#include <algorithm>

#include "halp_device.hpp"
#include "softmax_ahead.hpp"

namespace halp {
namespace {

// One thread per (step, row, class), classes padded to KC = 2, 4, 8 or 16: the KC lanes of a row share its
// index and fold its softmax.  (With sixteen lanes whatever K, a step of 1024 chains of 64 x 2 took
// 0.98 us instead of 0.87.)  The arithmetic is that of the general kernel's "before" side, value by
// value; records of classes from KC on are left as they are, their readers drop them.
template <int BITS, int KC>
__global__ __launch_bounds__(256) void ahead_scalars(InArgs a, Ahead s, int chain0) {
  const int local = blockIdx.y, chain = chain0 + local;
  const int c = threadIdx.x & (KC - 1);
  const int64_t g = ((int64_t)blockIdx.x * 256 + threadIdx.x) / KC;  // (step, row)
  const int K = a.K, B = a.B;
  const int64_t steps = s.t1 - s.t0;
  const bool in = g < steps * B;
  const int64_t tl = in ? g / B : 0;
  const int m = in ? (int)(g - tl * B) : 0;
  const int64_t t = s.t0 + tl;
  const uint64_t seed = a.seed + (uint64_t)chain;
  const uint64_t row = (uint64_t)t * (uint64_t)B + (uint64_t)m;
  const uint32_t ri = pick(stream_block(seed, kIdx, a.epoch, row >> 2), (uint32_t)(row & 3));
  const int64_t i = (int64_t)__umulhi(ri, (uint32_t)a.N);
  const float* phi = a.phi + (int64_t)chain * a.N * K;
  const bool live = c < K;
  // Algorithm 4 with squared loss needs no margins, and a caller need not have bound any
  const bool need_phi = a.loss != HALP_LOSS_SQUARED || a.lp;
  AheadRec r;
  r.phi = live && need_phi ? phi[i * K + c] : 0.f;
  r.p0 = 0.0;
  if (a.loss == HALP_LOSS_SOFTMAX) {
    const double v = live ? (double)r.phi : -INFINITY;
    const double mx = row_max_f64<KC>(v);
    const double e = live ? halp_exp(__dadd_rn(v, -mx)) : 0.0;
    r.p0 = __ddiv_rn(e, row_sum_f64<KC>(e));
  } else if (a.loss == HALP_LOSS_LOGISTIC) {
    const float y = reinterpret_cast<const float*>(a.y)[(int64_t)chain * a.y_chain_stride + i];
    if (c == 0) r.p0 = __ddiv_rn(-(double)y, __dadd_rn(1.0, halp_exp(__dmul_rn((double)y, (double)r.phi))));
    if (c == 1) r.phi = y;
  }
  const uint64_t n = row * (uint64_t)K + (uint64_t)(live ? c : 0);
  r.rho = pick(stream_block(seed, kGamma, a.epoch, n >> 2), (uint32_t)(n & 3));
  if (!in) return;
  s.rec[(((int64_t)local * s.S + tl) * B + m) * kAheadK + c] = r;
  if (c == 0) s.idx[((int64_t)local * s.S + tl) * B + m] = (int32_t)i;
  if (m == 0 && c == 0) {
    int cl = 0;
    if (a.lambda > 0) {  // c_lambda = Q_(2^-b, b)(alpha lambda)
      const uint32_t w = pick(stream_block(seed, kReg, a.epoch, (uint64_t)t >> 2), (uint32_t)(t & 3));
      cl = (int)quantize_real(__dmul_rn(a.hyper[2 * chain], a.lambda), (double)(1 << BITS), w, 0.0,
                              (double)((1 << (BITS - 1)) - 1), nullptr);
    }
    s.cl[(int64_t)local * s.S + tl] = cl;
  }
}

// Two strips of a class and one window of 8 steps per thread: two Philox blocks, eight dwords, a
// wave's stores 256 contiguous bytes each.  Strips past the row are left as they are: whatever
// bits stand there, a coordinate with z = h~ = x = 0 stays 0.
__global__ __launch_bounds__(256) void ahead_zbits(InArgs a, Ahead s, int bits, int chain0) {
  const int local = blockIdx.z;
  const uint64_t seed = a.seed + (uint64_t)(chain0 + local);
  const int ct = 16 / bits, U = (a.d + ct - 1) / ct, per = (U + 1) / 2;
  const int v = (int)(blockIdx.x * 256 + threadIdx.x);
  if (v >= a.K * per) return;
  const int c = v / per, u = 2 * (v - c * per);
  const int64_t tw = s.t0 + 8 * (int64_t)blockIdx.y;
  const U4 r0 = zround_block(seed, a.epoch, (uint32_t)(c * U + u), (uint32_t)(tw >> 3));
  const U4 r1 = zround_block(seed, a.epoch, (uint32_t)(c * U + u + 1), (uint32_t)(tw >> 3));
  uint32_t* out = reinterpret_cast<uint32_t*>(s.zbits + (((int64_t)local * s.S + (tw - s.t0)) * a.K + c) * s.UP + u);
  const int64_t stride = (int64_t)a.K * s.UP / 2;  // dwords per step
#pragma unroll
  for (int k = 0; k < 8; ++k) out[k * stride] = zround_field(r0, (uint32_t)k) | (zround_field(r1, (uint32_t)k) << 16);
}

// The same at 8 bits, expanded: r - h~ modulo 2^16; strips of a class up to UP, those past the row 0.
__global__ __launch_bounds__(256) void ahead_halves(InArgs a, Ahead s, int chain0) {
  const int local = blockIdx.z, chain = chain0 + local;
  const uint64_t seed = a.seed + (uint64_t)chain;
  const int U = (a.d + 1) / 2;
  const int v = (int)(blockIdx.x * 256 + threadIdx.x);
  if (v >= a.K * s.UP) return;
  const int c = v / s.UP, u = v - c * s.UP;
  const int64_t tw = s.t0 + 8 * (int64_t)blockIdx.y;
  uint32_t* out = reinterpret_cast<uint32_t*>(s.zbits) + (((int64_t)local * s.S + (tw - s.t0)) * a.K + c) * s.UP + u;
  const int64_t stride = (int64_t)a.K * s.UP;  // dwords per step
  const bool in = u < U;
  const U4 r = zround_block(seed, a.epoch, (uint32_t)(c * U + u), (uint32_t)(tw >> 3));
  int h0 = 0, h1 = 0;
  if (in) {
    const int16_t* h = reinterpret_cast<const int16_t*>(a.h) + ((int64_t)chain * a.K + c) * a.d + 2 * u;
    h0 = h[0];
    h1 = 2 * u + 1 < a.d ? h[1] : 0;
  }
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const int f = (int)zround_field(r, (uint32_t)k);
    out[k * stride] = in ? (uint32_t)(((f & 0xFF) - h0) & 0xFFFF) | ((uint32_t)((f >> 8) - h1) << 16) : 0u;
  }
}

size_t round256(size_t n) { return (n + 255) / 256 * 256; }

}  // namespace

size_t ahead_bytes(const halp_params& p, int chains, int64_t S, int UP, bool expanded) {
  const size_t n = (size_t)chains * (size_t)S;
  return round256(n * p.B * kAheadK * sizeof(AheadRec)) + round256(n * p.B * 4) + round256(n * 4) +
         round256(n * p.K * (size_t)UP * (expanded ? 4 : 2));
}

int64_t ahead_steps(const halp_params& p, int chains, int UP, bool expanded, size_t bytes) {
  const size_t per8 = ahead_bytes(p, chains, 8, UP, expanded);
  int64_t S = (int64_t)(bytes / per8) * 8;  // each part is rounded up once per call, so this is on the safe side
  const int64_t most = (p.T + 7) / 8 * 8;
  return S < most ? S : (most > 8 ? most : 8);
}

size_t plan_ahead(halp_handle& h, int UP, int resident, bool expanded) {
  const halp_params& p = h.p;
  const size_t mb = (size_t)1 << 20;
  const size_t budget = std::min((size_t)1024 * mb, std::max((size_t)64 * mb, (size_t)p.R * 4 * mb));
  const int groups = (p.R + resident - 1) / resident;
  int chains = (p.R + groups - 1) / groups;
  int64_t S = ahead_steps(p, chains, UP, expanded, budget);
  for (; S < 8 && chains > 1; S = ahead_steps(p, chains, UP, expanded, budget)) chains = (chains + 1) / 2;
  h.ahead_chains = chains;
  h.ahead_steps = std::max((int64_t)8, S);
  return ahead_bytes(p, chains, h.ahead_steps, UP, expanded);
}

Ahead ahead_layout(const halp_params& p, int chains, int64_t S, int UP, bool expanded, void* ws) {
  const size_t n = (size_t)chains * (size_t)S;
  unsigned char* q = reinterpret_cast<unsigned char*>(ws);
  Ahead s;
  s.rec = reinterpret_cast<AheadRec*>(q);
  q += round256(n * p.B * kAheadK * sizeof(AheadRec));
  s.idx = reinterpret_cast<int32_t*>(q);
  q += round256(n * p.B * 4);
  s.cl = reinterpret_cast<int32_t*>(q);
  q += round256(n * 4);
  s.zbits = UP > 0 ? reinterpret_cast<uint16_t*>(q) : nullptr;
  s.expanded = expanded;
  s.S = S;
  s.UP = UP;
  s.t0 = s.t1 = 0;
  return s;
}

int launch_ahead(const InArgs& a, const Ahead& s, int bits, int chain0, int chains, hipStream_t stream) {
  const int64_t steps = s.t1 - s.t0;
  auto scalars = [&](auto kc) {
    constexpr int KC = decltype(kc)::value;
    const dim3 grid((unsigned)((steps * a.B * KC + 255) / 256), chains);
    if (bits == 8) hipLaunchKernelGGL((ahead_scalars<8, KC>), grid, dim3(256), 0, stream, a, s, chain0);
    else hipLaunchKernelGGL((ahead_scalars<16, KC>), grid, dim3(256), 0, stream, a, s, chain0);
  };
  if (a.K <= 2) scalars(std::integral_constant<int, 2>{});  // K = 1: the label takes the second record
  else if (a.K <= 4) scalars(std::integral_constant<int, 4>{});
  else if (a.K <= 8) scalars(std::integral_constant<int, 8>{});
  else scalars(std::integral_constant<int, 16>{});
  if (s.expanded) {
    const dim3 g2((unsigned)((a.K * s.UP + 255) / 256), (unsigned)((steps + 7) / 8), chains);
    hipLaunchKernelGGL(ahead_halves, g2, dim3(256), 0, stream, a, s, chain0);
  } else if (s.UP > 0) {
    const int U = (a.d + 16 / bits - 1) / (16 / bits);
    const dim3 g2((unsigned)((a.K * ((U + 1) / 2) + 255) / 256), (unsigned)((steps + 7) / 8), chains);
    hipLaunchKernelGGL(ahead_zbits, g2, dim3(256), 0, stream, a, s, bits, chain0);
  }
  return hip_ok(hipGetLastError());
}

}  // namespace halp
