// Inner loop of Algorithm 4 (LM-HALP) for softmax regression (K classes, one sampled row per step) at 8 bits,
// register-resident form with specialised waves: the 8-bit twin of inner_softmax.hip, which see for the roles of
// the waves and for the records made ahead.
//
// Class wave c owns row c of z (CPW = 2: two rows, for 16 classes): lane l holds the UPL consecutive strips (two
// coordinates each) from l UPL on, as 256 z in packed 16-bit halves.  There the rounding step is three
// packed instructions per strip,
//   n = -gamma x + (r - h~),   u = 256 z + n saturated to 16 bits,   256 z = u with its low byte cleared,
// since floor over 2^8 is clearing the low byte and the box [-128, 127] is what saturation keeps.  It needs
// |gamma x| + |r - h~| < 2^15: class waves with an |h~| past kWholeH take a second loop, in 32-bit arithmetic.
// What saturated is found by the sum without saturation and counted behind one branch.
//
// The row wave fetches the sampled rows and leaves them in LDS for all class waves, a coordinate in the high byte of
// its half: as such the dot with 256 z is one v_dot4 per strip, whatever the low bytes hold.  With few chains (EXP) the
// records hold r - h~ in 16-bit halves, with many, whose records' traffic counts, the bytes of r.
// (15 classes leave no room for a row wave, and more of many chains share a CU without one: kernel_for.)
//
// One step:
//   class waves   x_i^T z_c (v_dot4, DPP fold), one LDS word each                                            | barrier
//   service wave  softmax after the offset, one class per lane, -gamma_c into LDS; class waves meanwhile: what
//                 saturated at the last step, low bytes of 256 z cleared, the next row from LDS, r - h~      | barrier
//   class waves   update of row c of z: two packed instructions per strip; row wave: the row two steps on
//
// What bounds it: the dependent chain (~1000 cycles at 64 x 2), and from eight strips per lane and three class waves to a
// SIMD on the class waves' instructions, of which only multiply-add, saturated addition, dot and fold are on the chain.
// us per step of the loop, one chain, with the update in unsaturated halves (shift, two parts of h~, a test for clamps before
// the dot) and a row unpacked by every class wave -> now: 784 x 10 0.74 -> 0.62; 1024 x 15 0.88 -> 0.75; 784 x 5 0.55 -> 0.50; 300 x 4
// 0.451 -> 0.443; 64 x 2 0.413 -> 0.403; 256 chains of 784 x 10 1.36 -> 1.32; where the box binds (400 coordinates of 784 x 10
// clamped per step) 1.05 -> 0.72.
#include <algorithm>

#include "halp_device.hpp"
#include "softmax_ahead.hpp"
#include "softmax_fused.hpp"
#include "inner_softmax_b8.hpp"

namespace halp {
namespace {

constexpr int kWin = 8;   // steps per unrolled window
constexpr int kKC = 16;   // classes are padded to one DPP row

// Who fetches the rows: a wave of its own or the service wave, for all class waves, or every class wave for itself.
enum class Rows { kOwn, kService, kEach };

template <int UPL, int KT, int CPW, bool EXP, Rows ROWS>
__global__ __launch_bounds__(64 * KT) void inner_softmax_b8_kernel(InArgs a, Ahead ah, int chain0, int last) {
  constexpr int CPL = 2 * UPL;
  constexpr int NDW = (UPL + 1) / 2;          // dwords of a lane's fragment of a row
  constexpr int NZB = EXP ? UPL : NDW;        // dwords of its records of a step
  // steps a request runs ahead: four, or two where four sets of fragments do not fit the registers
  constexpr int kDep = CPW > 1 || (UPL == 8 && KT > 12 && EXP) ? 2 : 4;
  typedef short S2 __attribute__((ext_vector_type(2)));
  typedef unsigned short W2 __attribute__((ext_vector_type(2)));
  constexpr int QMAX = 127, QMIN = -128;
  const int local = blockIdx.x, chain = chain0 + local;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int d = a.d, K = a.K;
  const int U = (d + 1) / 2;
  // Waves w, w + 4, ... share a SIMD.  Wave 3's has the fewest waves, so the service wave goes
  // there (10 classes: beside one class wave, the other SIMDs have three), unless the class
  // waves alone fill whole rounds: then it comes last.
  const int ncw = K / CPW, svc = ncw % 4 == 0 ? ncw : min(3, ncw);
  const int64_t T = epoch_steps(a.seed + (uint64_t)chain, a.epoch, a.T, a.option2);
  const int steps = segment_steps(ah.t0, ah.t1, T);
  const double* sc = a.scales + (int64_t)chain * 8;
  unsigned long long* cnt_out = reinterpret_cast<unsigned long long*>(a.counters + (int64_t)chain * 4);
  const bool lp = a.lp != 0;  // Algorithm 2 (LP-SVRG): z is the model itself

  if (sc[7] != 0.0) {
    if (tid < 4) cnt_out[tid] = 0;
    return;
  }

  __shared__ __attribute__((aligned(16))) int s_D[2][kKC];  // x_i^T z_c
  __shared__ int s_ng[2][kKC];                              // -gamma_c
  __shared__ __attribute__((aligned(16))) uint32_t s_x[2][ROWS == Rows::kEach ? 1 : UPL * 64];  // the row in pairs, by step parity
  __shared__ int s_dumpD[64];  // partial folds of lanes 0..62 of every class wave (never read)
  __shared__ unsigned long long s_cnt[3];
  if (tid < 3) s_cnt[tid] = 0;
  if (tid < 2 * kKC) (&s_D[0][0])[tid] = 0;  // classes past K stay 0
  const bool use_reg = a.lambda > 0;
  const int32_t* __restrict__ clv = ah.cl + (int64_t)local * ah.S;
  const int tlast = steps > 0 ? steps - 1 : 0;  // requests past the segment's end repeat its last step
  const int s0 = lane * UPL, j0 = 2 * s0;
  const bool lane_ok = s0 < U;
  // a lane's dwords of a row in s_x: pieces of four dwords side by side over the lanes
  constexpr int XP = UPL < 4 ? UPL : 4;
  auto x_at = [&](int par, int u) { return &s_x[par][(u / XP) * 64 * XP + lane * XP + u % XP]; };

  const unsigned char* __restrict__ Xq = reinterpret_cast<const unsigned char*>(a.Xq) +
                                         (int64_t)chain * a.xq_chain_stride;
  const int32_t* __restrict__ idx = ah.idx + (int64_t)local * ah.S;
  // Rows are padded to whole 8-byte groups: a fragment is read in pieces of 8 bytes at most, and
  // a piece past the row repeats the row's last group.  What lies past d is masked to zero.
  const uint32_t last_group = (uint32_t)((((int64_t)d + 7) / 8 - 1) * 8);
  uint32_t fs[UPL];  // byte selectors of a pair, 0x0C (a zero byte) past d
#pragma unroll
  for (int u = 0; u < UPL; ++u) {
    const int nv = d - (j0 + 2 * u), b = 2 * (u & 1);
    fs[u] = ((nv >= 2 ? (uint32_t)(b + 1) : 0x0Cu) << 24) | 0x0C000Cu | ((nv >= 1 ? (uint32_t)b : 0x0Cu) << 8);
  }
  uint32_t foff[(UPL + 3) / 4];
#pragma unroll
  for (int q = 0; q < (UPL + 3) / 4; ++q)
    foff[q] = UPL >= 4 ? min((uint32_t)(s0 * 2 + 8 * q), last_group) : (lane_ok ? (uint32_t)(s0 * 2) : 0u);
  uint32_t fr[kDep][NDW];
  auto request_row = [&](int slot, int i) {
    const unsigned char* rp = Xq + (int64_t)i * a.ldxq;
    if constexpr (UPL == 1) {
      fr[slot][0] = *reinterpret_cast<const uint16_t*>(rp + lane_off(foff[0]));
    } else if constexpr (UPL == 2) {
      fr[slot][0] = *reinterpret_cast<const uint32_t*>(rp + lane_off(foff[0]));
    } else {
#pragma unroll
      for (int q = 0; q < UPL / 4; ++q) {
        const uint2 v = *reinterpret_cast<const uint2*>(rp + lane_off(foff[q]));
        fr[slot][2 * q] = v.x;
        fr[slot][2 * q + 1] = v.y;
      }
    }
  };
  auto hand_out_row = [&](int par, int slot) {
    uint32_t xv[UPL];
#pragma unroll
    for (int u = 0; u < UPL; ++u)
      xv[u] = __builtin_amdgcn_perm(0u, fr[slot][u / 2], fs[u]);
#pragma unroll
    for (int u = 0; u < UPL; u += XP) {
      if constexpr (XP == 4) *reinterpret_cast<uint4*>(x_at(par, u)) = make_uint4(xv[u], xv[u + 1], xv[u + 2], xv[u + 3]);
      else if constexpr (XP == 2) *reinterpret_cast<uint2*>(x_at(par, u)) = make_uint2(xv[u], xv[u + 1]);
      else *x_at(par, u) = xv[u];
    }
  };
  int iv = 0, ivn = 0, ivnn = 0;  // lane l: number of the row of step t0 + (l & 7), and of the next windows'
  auto start_rows = [&]() __attribute__((always_inline)) {
    if (steps == 0) return;
    iv = idx[min(lane & 7, tlast)];
    ivn = idx[min(kWin + (lane & 7), tlast)];
    request_row(0, __builtin_amdgcn_readlane(iv, 0));
    request_row(1, __builtin_amdgcn_readlane(iv, 1));
    hand_out_row(0, 0);
    hand_out_row(1, 1);
#pragma unroll
    for (int s = 2; s < 2 + kDep; ++s) request_row(s % kDep, __builtin_amdgcn_readlane(iv, s));
  };
  // behind the second barrier of step s of a window: the row of the step two steps on, and the next request
  auto next_row = [&](int s) __attribute__((always_inline)) {
    hand_out_row(s & 1, (s + 2) % kDep);
    request_row((s + 2) % kDep, __builtin_amdgcn_readlane(s + 2 + kDep < kWin ? iv : ivn, (s + 2 + kDep) % kWin));
  };
  auto window_rows = [&](int t0) __attribute__((always_inline)) { ivnn = idx[min(t0 + 2 * kWin + (lane & 7), tlast)]; };
  auto window_end = [&]() __attribute__((always_inline)) { iv = ivn; ivn = ivnn; };

  if (wave == svc) {
    // ===================================================================== service wave
    // every class wave waits for this one at the step's second barrier: it goes first
    // wherever it shares a SIMD with class waves
    __builtin_amdgcn_s_setprio(3);
    if constexpr (ROWS == Rows::kService) start_rows();
    __syncthreads();
    if (steps > 0) {
      const AheadRec* __restrict__ rec = ah.rec + (int64_t)local * ah.S * kAheadK;
      const double delta_m = sc[0], inv_s = sc[5];
      const double dscale = __dmul_rn(a.delta_d, delta_m);
      const double aB = a.hyper[2 * chain];  // alpha / B, B = 1
      unsigned int n_gclamp = 0, n_reg = 0;
      const int lc = lane & 15;
      // gammas of a step in the fixed order of roundings, one class per lane of a row of 16
      auto step_fixed = [&](int par, const AheadRec& r) __attribute__((always_inline)) {
        const bool live = lc < K;
        // Algorithm 4 moves the margins by x^T z; in Algorithm 2 (LP-SVRG) x^T w is the margin
        const double moved = __dmul_rn(dscale, (double)s_D[par][lc]);
        const double val = live ? (lp ? moved : __dadd_rn((double)r.phi, moved)) : -INFINITY;
        const double mx = row_max_f64(val);
        const double e = live ? halp_exp(__dadd_rn(val, -mx)) : 0.0;
        // normaliser: pairwise over adjacent classes, the order the DPP fold gives
        const double p = __ddiv_rn(e, row_sum_f64(e));
        // beta_c = alpha (p_c(phi + x^T z) - p_c(phi)), gamma_c = Q_(delta_s, b)(beta_c)
        const double beta = __dmul_rn(aB, __dadd_rn(p, -r.p0));
        const double f = floor(__dadd_rn(__dmul_rn(beta, inv_s), __dmul_rn((double)r.rho, 0x1p-32)));
        const double fc = fmin(fmax(f, (double)QMIN), (double)QMAX);
        if (lane < K) s_ng[par][lane] = (int)(-fc);
        n_gclamp += (lane < K && f != fc) ? 1u : 0u;
      };
      auto run = [&](auto fused_tag) __attribute__((always_inline)) {
        constexpr bool FUSED = decltype(fused_tag)::value;
        const int rc = FUSED ? soft_class(lane) : lc;  // class of the lane's records
        const bool live = rc < K;
        const double k2 = __dmul_rn(aB, inv_s);
        AheadRec rr[kDep];
#pragma unroll
        for (int s = 0; s < kDep; ++s) rr[s] = rec[(int64_t)min(s, tlast) * kAheadK + rc];
        int cln = use_reg ? clv[min(lane & 7, tlast)] : 0;
        SoftDraw dr{};
        double from = 0.0;  // what the new margins are measured from: phi in Algorithm 2
        auto draw = [&](const AheadRec& r) __attribute__((always_inline)) {
          if constexpr (FUSED) {
            dr = soft_draw<true>(live, r.p0, r.phi, r.rho, k2);
            from = lp && live ? (double)r.phi : 0.0;
          }
        };
        draw(rr[0]);
        for (int t0 = 0; t0 < steps; t0 += kWin) {
          if (use_reg) {
            n_reg += (lane < kWin && t0 + lane < steps && cln != 0) ? 1u : 0u;
            cln = clv[min(t0 + kWin + (lane & 7), tlast)];
          }
          if constexpr (ROWS == Rows::kService) window_rows(t0);
#pragma unroll
          for (int s = 0; s < kWin; ++s) {
            if (t0 + s < steps) {
              lds_barrier();  // the dot products of this step are in LDS
              if constexpr (FUSED) {
                int hi;
                if (__builtin_expect_with_probability(
                        soft_gamma<true>(dr, live, __fma_rn(dscale, (double)s_D[s & 1][rc], -from), &hi), 1, 1.0)) {
                  const int g = min(max(hi, kSoftMagicHi - QMAX), kSoftMagicHi - QMIN);
                  s_ng[s & 1][rc] = g - kSoftMagicHi;  // (four lanes store the same word)
                  n_gclamp += (live && soft_first_copy(lane) && g != hi) ? 1u : 0u;
                } else {
                  step_fixed(s & 1, rec[(int64_t)(t0 + s) * kAheadK + lc]);
                }
              } else {
                step_fixed(s & 1, rr[s % kDep]);
              }
              lds_barrier();  // gamma is out; the class waves update z
              rr[s % kDep] = rec[(int64_t)min(t0 + s + kDep, tlast) * kAheadK + rc];
              draw(rr[(s + 1) % kDep]);
              if constexpr (ROWS == Rows::kService) next_row(s);
            }
          }
          if constexpr (ROWS == Rows::kService) window_end();
        }
      };
      if (soft_covers(dscale, aB, inv_s)) run(std::true_type{});
      else run(std::false_type{});
      if (n_gclamp) atomicAdd(&s_cnt[1], (unsigned long long)n_gclamp);
      if (n_reg) atomicAdd(&s_cnt[2], (unsigned long long)n_reg);
    }
  } else if (ROWS == Rows::kOwn && wave == ncw + 1) {
    // ========================================================================= row wave
    start_rows();
    __syncthreads();
    for (int t0 = 0; t0 < steps; t0 += kWin) {
      window_rows(t0);
#pragma unroll
      for (int s = 0; s < kWin; ++s) {
        if (t0 + s < steps) {
          lds_barrier();
          lds_barrier();
          next_row(s);
        }
      }
      window_end();
    }
  } else {
    // ======================================================================= class wave
    // rows cls0 .. cls0 + CPW - 1 of z
    const int cls0 = (wave - (wave > svc ? 1 : 0)) * CPW;
    auto row0_of = [&](int cc) { return ((int64_t)chain * K + cls0 + cc) * d; };
    // 256 z before the step; what was added to it; their saturated sum, whose high bytes are z and whose low bytes are
    // cleared later, beside the softmax
    S2 zq[CPW][UPL], add[CPW][UPL], sum[CPW][UPL];
    uint32_t large = 0;  // not 0 where a coordinate of the wave's rows leaves no room for -gamma x + r - h~ in 16 bits
#pragma unroll
    for (int cc = 0; cc < CPW; ++cc) {
      const int8_t* __restrict__ zg = reinterpret_cast<const int8_t*>(a.z) + row0_of(cc);
      const int16_t* __restrict__ hg = reinterpret_cast<const int16_t*>(a.h) + row0_of(cc);
      int zv[CPL], hk[CPL];  // all loads in flight at once; those of h~ for the test alone: lane after lane
#pragma unroll
      for (int k = 0; k < CPL; ++k) hk[k] = (int)hg[min(64 * k + lane, d - 1)];
#pragma unroll
      for (int k = 0; k < CPL; ++k) zv[k] = (int)zg[min(j0 + k, d - 1)];
#pragma unroll
      for (int k = 0; k < CPL; ++k) asm volatile("" : "+v"(zv[k]), "+v"(hk[k]));
#pragma unroll
      for (int k = 0; k < CPL; ++k) {
        large |= hk[k] > kWholeH || hk[k] < -kWholeH ? 1u : 0u;
        sum[cc][k / 2][k % 2] = (short)(j0 + k < d ? zv[k] * 256 : 0);
      }
#pragma unroll
      for (int u = 0; u < UPL; ++u) {
        zq[cc][u] = sum[cc][u];
        add[cc][u] = (S2)(0);
      }
    }
    // lanes past the row read other coordinates' records: their z stays 0
    uint32_t keep = lane_ok ? 0xFF00FF00u : 0u;
    asm volatile("" : "+v"(keep));
    unsigned long long n_zclamp = 0;  // counted by the wave (steps with an L2 draw)
    W2 n_half = (W2)(0);              // counted by the lane, a window's and all of them
    uint32_t n_lane = 0;
    W2 ones = (W2)(1);
    asm volatile("" : "+v"(ones));  // a value the compiler does not see: one packed minimum per strip
    using LdsInt = __attribute__((address_space(3))) int;
    LdsInt* slotD[CPW][2];
#pragma unroll
    for (int cc = 0; cc < CPW; ++cc)
#pragma unroll
      for (int par = 0; par < 2; ++par)
        slotD[cc][par] = (LdsInt*)(lane == 63 ? &s_D[par][cls0 + cc] : &s_dumpD[lane]);
    __syncthreads();  // the first two rows are in LDS

    auto run = [&](auto whole_tag) __attribute__((always_inline)) {
      constexpr bool WHOLE = decltype(whole_tag)::value;
      constexpr bool kH = !EXP || !WHOLE;  // where the records do not hold h~
      S2 hp[CPW][kH ? UPL : 1];
      if constexpr (kH) {
#pragma unroll
        for (int cc = 0; cc < CPW; ++cc) {
          const int16_t* __restrict__ hg = reinterpret_cast<const int16_t*>(a.h) + row0_of(cc);
          int hk[CPL];
#pragma unroll
          for (int k = 0; k < CPL; ++k) hk[k] = (int)hg[min(j0 + k, d - 1)];
#pragma unroll
          for (int k = 0; k < CPL; ++k) asm volatile("" : "+v"(hk[k]));
#pragma unroll
          for (int k = 0; k < CPL; ++k) hp[cc][k / 2][k % 2] = (short)(j0 + k < d ? hk[k] : 0);
        }
      }
      // the step's records of this lane's strips
      uint32_t zb[kDep][CPW][NZB];
      constexpr uint32_t kStrip = EXP ? 4 : 2;  // bytes
      const unsigned char* __restrict__ zst =
          reinterpret_cast<const unsigned char*>(ah.zbits) + (int64_t)local * ah.S * K * ah.UP * kStrip;
      const uint32_t step_bytes = (uint32_t)(K * ah.UP) * kStrip;
      const uint32_t zoff = (uint32_t)((cls0 * ah.UP + (lane_ok ? s0 : 0)) * kStrip);
      auto request_bits = [&](int slot, int t) {
        const unsigned char* bp = zst + (uint32_t)t * step_bytes;  // a segment's records of a chain: 1 GB at most
#pragma unroll
        for (int cc = 0; cc < CPW; ++cc) {
          const unsigned char* p = bp + (cc * ah.UP * kStrip) + lane_off(zoff);
          if constexpr (UPL == 1 && !EXP) {
            zb[slot][cc][0] = *reinterpret_cast<const uint16_t*>(p);
          } else if constexpr (NZB == 1) {
            zb[slot][cc][0] = *reinterpret_cast<const uint32_t*>(p);
          } else if constexpr (NZB == 2) {
            const uint2 v = *reinterpret_cast<const uint2*>(p);
            zb[slot][cc][0] = v.x;
            zb[slot][cc][1] = v.y;
          } else {
#pragma unroll
            for (int q = 0; q < NZB / 4; ++q) {
              const uint4 v = reinterpret_cast<const uint4*>(p)[q];
              zb[slot][cc][4 * q] = v.x; zb[slot][cc][4 * q + 1] = v.y;
              zb[slot][cc][4 * q + 2] = v.z; zb[slot][cc][4 * q + 3] = v.w;
            }
          }
        }
      };
      int clw = use_reg ? clv[min(lane & 7, tlast)] : 0;
#pragma unroll
      for (int s = 0; s < kDep - (EXP ? 1 : 0); ++s) request_bits(s, min(s, tlast));
      uint32_t xs[2][UPL];  // the row, by step parity: pairs, a coordinate in the high byte of its half
      auto fetch_row = [&](int par) {
#pragma unroll
        for (int u = 0; u < UPL; u += XP) {
          if constexpr (XP == 4) {
            const uint4 v = *reinterpret_cast<const uint4*>(x_at(par, u));
            xs[par][u] = v.x; xs[par][u + 1] = v.y; xs[par][u + 2] = v.z; xs[par][u + 3] = v.w;
          } else if constexpr (XP == 2) {
            const uint2 v = *reinterpret_cast<const uint2*>(x_at(par, u));
            xs[par][u] = v.x; xs[par][u + 1] = v.y;
          } else {
            xs[par][u] = *x_at(par, u);
          }
        }
      };
      auto unpack = [&](int par, int slot) {
#pragma unroll
        for (int u = 0; u < UPL; ++u) xs[par][u] = __builtin_amdgcn_perm(0u, fr[slot][u / 2], fs[u]);
      };
      if constexpr (ROWS == Rows::kEach) {
        iv = idx[min(lane & 7, tlast)];
        ivn = idx[min(kWin + (lane & 7), tlast)];
#pragma unroll
        for (int s = 0; s < kDep; ++s) request_row(s, __builtin_amdgcn_readlane(iv, s));
        unpack(0, 0);
        request_row(0, __builtin_amdgcn_readlane(iv, kDep));
      } else {
        fetch_row(0);
      }

      for (int t0 = 0; t0 < steps; t0 += kWin) {
        const int clc = clw;
        if (use_reg) clw = clv[min(t0 + kWin + (lane & 7), tlast)];
        if constexpr (ROWS == Rows::kEach) window_rows(t0);
#pragma unroll
        for (int s = 0; s < kWin; ++s) {
          if (t0 + s < steps) {
            // the fold leaves the sum in lane 63, which stores it; the other lanes store their
            // partial folds into a dump row, so that no lane mask is set up and no lane is read
#pragma unroll
            for (int cc = 0; cc < CPW; ++cc) {
              int c0 = 0, c1 = 0;  // two chains
#pragma unroll
              for (int u = 0; u < UPL; ++u) {
                const int zu = __builtin_bit_cast(int, sum[cc][u]);
                if (u & 1) c1 = __builtin_amdgcn_sdot4((int)xs[s & 1][u], zu, c1, false);
                else c0 = __builtin_amdgcn_sdot4((int)xs[s & 1][u], zu, c0, false);
              }
              *slotD[cc][s & 1] = wave_fold_i32(UPL > 1 ? c0 + c1 : c0);
            }
            lds_barrier();
            __builtin_amdgcn_sched_barrier(0);
            // while the service wave evaluates the softmax
            S2 xp[UPL];
#pragma unroll
            for (int u = 0; u < UPL; ++u) xp[u] = __builtin_bit_cast(S2, xs[s & 1][u]) >> (S2)(8);
#pragma unroll
            for (int cc = 0; cc < CPW; ++cc) {  // the last step's sums: what saturated, low bytes cleared
              uint32_t off[UPL], hit = 0;  // not 0 in the halves that did
#pragma unroll
              for (int u = 0; u < UPL; ++u) {
                const uint32_t v = __builtin_bit_cast(uint32_t, sum[cc][u]);
                off[u] = v ^ __builtin_bit_cast(uint32_t, zq[cc][u] + add[cc][u]);
                hit |= off[u];
                zq[cc][u] = __builtin_bit_cast(S2, v & keep);
              }
              if (__ballot(hit != 0) != 0) {  // a coordinate left the box
#pragma unroll
                for (int u = 0; u < UPL; ++u) n_half += __builtin_elementwise_min(__builtin_bit_cast(W2, off[u]), ones);
              }
            }
            S2 crp[CPW][UPL];  // r - h~, or without WHOLE r alone (EXP: r - h~ modulo 2^16)
#pragma unroll
            for (int cc = 0; cc < CPW; ++cc)
#pragma unroll
              for (int u = 0; u < UPL; ++u) {
                if constexpr (EXP) {
                  crp[cc][u] = __builtin_bit_cast(S2, zb[s % kDep][cc][u]);
                } else {
                  const uint32_t rp = __builtin_amdgcn_perm(0u, zb[s % kDep][cc][u / 2], (u & 1) ? 0x0C030C02u : 0x0C010C00u);
                  crp[cc][u] = __builtin_bit_cast(S2, rp);
                  if constexpr (WHOLE) crp[cc][u] -= hp[cc][u];
                }
              }
            if constexpr (EXP) request_bits((s + kDep - 1) % kDep, min(t0 + s + kDep - 1, tlast));  // the last step's slot
            else request_bits(s % kDep, min(t0 + s + kDep, tlast));
            if constexpr (ROWS == Rows::kEach) {
              unpack((s + 1) & 1, (s + 1) % kDep);
              request_row((s + 1) % kDep, __builtin_amdgcn_readlane(s + 1 + kDep < kWin ? iv : ivn, (s + 1 + kDep) % kWin));
            } else {
              fetch_row((s + 1) & 1);
            }
            // all of it stays in front of the barrier
#pragma unroll
            for (int cc = 0; cc < CPW; ++cc)
#pragma unroll
              for (int u = 0; u < UPL; ++u) asm volatile("" : "+v"(crp[cc][u]), "+v"(zq[cc][u]));
#pragma unroll
            for (int u = 0; u < UPL; ++u) asm volatile("" : "+v"(xp[u]));
            __builtin_amdgcn_sched_barrier(0);
            lds_barrier();
            int ng[CPW];
#pragma unroll
            for (int cc = 0; cc < CPW; ++cc) ng[cc] = s_ng[s & 1][cls0 + cc];
            const int cl = __builtin_amdgcn_readlane(clc, s);  // 0 where there is no L2 term
            // u = z - gamma x - h~ (- c_lambda z), z = Q_(delta_m, b)(u)
#pragma unroll
            for (int cc = 0; cc < CPW; ++cc) {
              if constexpr (WHOLE) {
                const S2 ngp = S2{(short)ng[cc], (short)ng[cc]};
#pragma unroll
                for (int u = 0; u < UPL; ++u) {
                  add[cc][u] = xp[u] * ngp + crp[cc][u];
                  sum[cc][u] = __builtin_elementwise_add_sat(zq[cc][u], add[cc][u]);
                }
              }
              if (!WHOLE || __builtin_expect_with_probability(cl != 0, 0, 1.0)) {
                // a step with an L2 draw, or an h~ past kWholeH: 32-bit arithmetic
#pragma unroll
                for (int u = 0; u < UPL; ++u) {
                  int zc[2];
#pragma unroll
                  for (int e = 0; e < 2; ++e) {
                    const S2 xu = xp[u], zo = zq[cc][u], cu = crp[cc][u];
                    const int zk = (int)zo[e] >> 8;
                    int ad = EXP && !lane_ok ? 0 : (int)cu[e];
                    if constexpr (!WHOLE) {
                      const S2 hu = hp[cc][u];
                      ad = (EXP ? ((int)cu[e] + (int)hu[e]) & 0xFF : ad) - (int)hu[e];
                    }
                    const int zu = zk + (mad24(ng[cc], (int)xu[e], mad24(-cl, zk, ad)) >> 8);
                    zc[e] = min(max(zu, QMIN), QMAX);
                    n_zclamp += (unsigned long long)__builtin_popcountll(__ballot(zu != zc[e]));
                  }
                  sum[cc][u] = S2{(short)(zc[0] * 256), (short)(zc[1] * 256)};
                  add[cc][u] = sum[cc][u] - zq[cc][u];  // nothing left to count
                }
              }
            }
          }
          __builtin_amdgcn_sched_barrier(0);  // keep one step's temporaries from overlapping the next's
        }
        n_lane += (uint32_t)n_half[0] + (uint32_t)n_half[1];
        n_half = (W2)(0);
        if constexpr (ROWS == Rows::kEach) window_end();
      }
    };
    if (steps > 0) {
      // Two rows to a wave: said to be the rule, otherwise the compiler spills registers of this loop for the other's (1024 x 16 one
      // chain 0.91 instead of 0.99 us per step; one row to a wave, where the box binds, 0.723 instead of 0.718 at 784 x 10).
      const bool fits = __ballot(large != 0) == 0;
      if (CPW > 1 ? __builtin_expect_with_probability(fits, 1, 1.0) : fits) run(std::true_type{});
      else run(std::false_type{});
    }

#pragma unroll
    for (int cc = 0; cc < CPW; ++cc)  // the last step's
#pragma unroll
      for (int u = 0; u < UPL; ++u) {
        const uint32_t off = __builtin_bit_cast(uint32_t, sum[cc][u]) ^ __builtin_bit_cast(uint32_t, zq[cc][u] + add[cc][u]);
        n_lane += ((off & 0xFFFFu) != 0 ? 1u : 0u) + ((off >> 16) != 0 ? 1u : 0u);
      }

    // ---- hand z out; after the epoch's last segment w~ <- w~ + delta_m z (option I)
    const double delta_m = sc[0];
#pragma unroll
    for (int cc = 0; cc < CPW; ++cc) {
      int8_t* __restrict__ zg = reinterpret_cast<int8_t*>(a.z) + row0_of(cc);
      float* __restrict__ wg = a.w + row0_of(cc);
      int jl = j0;
      asm volatile("" : "+v"(jl));  // keeps the addresses below from being carried through the loop
      float wv[CPL];
#pragma unroll
      for (int k = 0; k < CPL; ++k) wv[k] = wg[min(jl + k, d - 1)];  // all loads in flight at once
#pragma unroll
      for (int k = 0; k < CPL; ++k) asm volatile("" : "+v"(wv[k]));
#pragma unroll
      for (int k = 0; k < CPL; ++k) {
        if (jl + k < d) {
          const int zk = (int)sum[cc][k / 2][k % 2] >> 8;
          zg[jl + k] = (int8_t)zk;
          if (last) {
            const double step = __dmul_rn(delta_m, (double)zk);
            wg[jl + k] = lp ? (float)step : (float)__dadd_rn((double)wv[k], step);  // Alg. 2: w~ = delta w
          }
        }
      }
    }
    if (lane == 0 && n_zclamp) atomicAdd(&s_cnt[0], n_zclamp);
    if (n_lane) atomicAdd(&s_cnt[0], (unsigned long long)n_lane);
  }
  __syncthreads();
  if (tid < 4) {  // the segments of an epoch follow each other on the stream
    const unsigned long long before = ah.t0 == 0 || tid == 3 ? 0ull : cnt_out[tid];
    cnt_out[tid] = before + (tid < 3 ? s_cnt[tid] : 0ull);
  }
}

// K / CPW class waves, the service wave, the row wave.  dense: without the row wave, for workgroups that share a CU
// (plan_inner_softmax): of up to two strips per lane every class wave fetches for itself, of more the service wave for all, as
// it does for 15 classes, which leave no room for a row wave.
template <int UPL, bool EXP>
SoftmaxKernel kernel_for(int K, bool dense) {
  if (K > 15) return inner_softmax_b8_kernel<UPL, 12, 2, EXP, Rows::kOwn>;  // two rows to a wave, 8 + 2 waves
  if constexpr (!EXP)
    if (dense) return inner_softmax_b8_kernel<UPL, 16, 1, EXP, (UPL <= 2 ? Rows::kEach : Rows::kService)>;
  if (K == 15) return inner_softmax_b8_kernel<UPL, 16, 1, EXP, Rows::kService>;
  if constexpr (EXP)  // fewer waves, more registers each (few chains: no matter that fewer share a CU)
    if (K + 2 <= 12) return inner_softmax_b8_kernel<UPL, 12, 1, EXP, Rows::kOwn>;
  return inner_softmax_b8_kernel<UPL, 16, 1, EXP, Rows::kOwn>;
}

}  // namespace

int softmax_b8_threads(int K, bool dense) { return 64 * (K > 15 ? K / 2 + 2 : K + (dense || K == 15 ? 1 : 2)); }

SoftmaxKernel softmax_b8_kernel(int K, int upl, bool expanded, bool dense) {
  if (expanded) return upl == 8 ? kernel_for<8, true>(K, false) : nullptr;
  switch (upl) {
    case 1: return kernel_for<1, false>(K, dense);
    case 2: return kernel_for<2, false>(K, dense);
    case 4: return kernel_for<4, false>(K, dense);
    default: return kernel_for<8, false>(K, dense);
  }
}

}  // namespace halp
