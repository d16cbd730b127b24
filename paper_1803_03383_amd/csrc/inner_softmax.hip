// Inner loop of Algorithm 4 (LM-HALP) for softmax regression (K classes, one sampled row per
// step), register-resident form with specialised waves, at 16 bits; and the launch of this form at
// either width (8 bits: inner_softmax_b8.hip).
//
// One workgroup per chain: K / CPW class waves and one service wave (CPW = 1 up to 15
// classes; CPW = 2, two rows of z per class wave, for the 16 classes that would need a
// seventeenth wave).
//
// Class wave c owns row c of z ([K][d]): lane l holds the UPL consecutive strips
// (a coordinate each, UPL up to 16) starting at l * UPL,
// with h~, in registers for the whole epoch.  Its fragment of the sampled row and the step's
// rounding bits come straight from memory, requested two or four steps ahead.
//
// The service wave evaluates the softmax.  It holds no part of z.
//
// Everything a step needs that does not follow from z -- sample index, margins of the row and
// their softmax, rounding words of gamma, L2 draws, rounding bits of z -- is made ahead by the
// whole chip, a segment of steps at a time (softmax_ahead.hpp).  A CU whose class waves drew
// their own Philox blocks spent 40 % of its issue slots on them.
//
// One step:
//   class waves   x_i^T z_c (packed dots, DPP fold), one LDS word each                 | barrier
//   service wave  softmax after the offset, one class per lane, gamma_c into LDS;      |
//   class waves   meanwhile: what of the update needs no gamma, the next row's         |
//                 fragment unpacked, the next requests                                 | barrier
//   class waves   integer update of row c of z
//
// What bounds it: the dependent chain dot, fold, LDS, softmax (the short chain of softmax_fused.hpp,
// ~350 cycles), LDS, update, with the issue slots of the SIMD that has most class waves next to
// it: three waves of 784 coordinates take 920 cycles for update and dot where one takes 630, and
// at ten classes of that width these slots are the longer part.
// So the class waves' instructions are kept few: z biased so that one test of the wave finds a clamp, requests
// with a scalar base, the rare paths (a clamp, an L2 draw) behind one branch each.
//
// Measured, us per step of one chain, before (class waves drawing their own blocks) and now (the loop and its records):
// 784 x 10 2.73 -> 1.29; 1000 x 15 29.8 -> 2.9; 64 x 2 0.75 -> 0.47.  With 256 chains, where making the records
// takes the whole chip's issue slots too: 784 x 10 3.2 -> 2.26.
#include <algorithm>

#include "halp_device.hpp"
#include "softmax_ahead.hpp"
#include "softmax_fused.hpp"
#include "inner_softmax_b8.hpp"

namespace halp {
namespace {

constexpr int kWin = 8;   // steps per unrolled window
constexpr int kKC = 16;   // classes are padded to one DPP row

// half k & 1 of x (16 bits, signed) times the low half of b, plus c
__device__ __forceinline__ int mad16(uint32_t x, int k, int b, int c) {
  int r;
  if (k & 1) asm("v_mad_i32_i16 %0, %1, %2, %3 op_sel:[1,0,0,0]" : "=v"(r) : "v"(x), "v"(b), "v"(c));
  else asm("v_mad_i32_i16 %0, %1, %2, %3" : "=v"(r) : "v"(x), "v"(b), "v"(c));
  return r;
}

template <int UPL, int KT, int CPW>
__global__ __launch_bounds__(64 * KT) void inner_softmax_kernel(InArgs a, Ahead ah, int chain0, int last) {
  using AccT = long long;
  constexpr int CPL = UPL;  // a strip is one coordinate
  constexpr int NDW = (UPL + 1) / 2;  // dwords of a lane's fragment of a row, and of its rounding bits
  // steps a request runs ahead: four, or two where four sets of fragments do not fit the registers
  constexpr int kDep = UPL > 8 ? 2 : 4;
  constexpr int NP = CPL == 1 ? 1 : CPL / 2;  // pairs of coordinates, two 16-bit halves of a register
  // z is kept in pairs, biased by 2^15: before clamping, a coordinate has left the box exactly
  // where bits from 16 upwards are set.
  // 16 values of c_k and as many of z - hh would not fit the 128 registers of 16 waves: there that
  // part of the update waits until gamma is known
  constexpr bool kLean = UPL > 8 && KT > 12;
  typedef short S2 __attribute__((ext_vector_type(2)));
  typedef unsigned short W2 __attribute__((ext_vector_type(2)));
  constexpr int QMAX = 32767, QMIN = -32768;
  const int local = blockIdx.x, chain = chain0 + local;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int d = a.d, K = a.K;
  const int U = d;
  // Waves w, w + 4, ... share a SIMD.  Wave 3's has the fewest waves, so the service wave goes
  // there (10 classes: beside one class wave, the other SIMDs have three), unless the class
  // waves alone fill whole rounds: then it comes last.
  const int ncw = K / CPW, svc = ncw % 4 == 0 ? ncw : min(3, ncw);
  const int64_t T = epoch_steps(a.seed + (uint64_t)chain, a.epoch, a.T, a.option2);
  const int steps = segment_steps(ah.t0, ah.t1, T);
  const int64_t row_bytes = a.ldxq * 2;
  const double* sc = a.scales + (int64_t)chain * 8;
  unsigned long long* cnt_out = reinterpret_cast<unsigned long long*>(a.counters + (int64_t)chain * 4);
  const bool lp = a.lp != 0;  // Algorithm 2 (LP-SVRG): z is the model itself

  if (sc[7] != 0.0) {
    if (tid < 4) cnt_out[tid] = 0;
    return;
  }

  __shared__ __attribute__((aligned(16))) AccT s_D[2][kKC];  // x_i^T z_c
  __shared__ int s_ng[2][kKC];                               // gamma_c
  __shared__ AccT s_dumpD[64];  // partial folds of lanes 0..62 of every class wave (never read)
  __shared__ unsigned long long s_cnt[3];
  if (tid < 3) s_cnt[tid] = 0;
  if (tid < 2 * kKC) (&s_D[0][0])[tid] = 0;  // classes past K stay 0
  const bool use_reg = a.lambda > 0;
  const int32_t* __restrict__ clv = ah.cl + (int64_t)local * ah.S;
  const int tlast = steps > 0 ? steps - 1 : 0;  // requests past the segment's end repeat its last step
  __syncthreads();

  if (wave == svc) {
    // ===================================================================== service wave
    // every class wave waits for this one at the step's second barrier: it goes first
    // wherever it shares a SIMD with class waves
    __builtin_amdgcn_s_setprio(3);
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
        if (lane < K) s_ng[par][lane] = (int)fc;
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
            dr = soft_draw<false>(live, r.p0, r.phi, r.rho, k2);
            from = lp && live ? (double)r.phi : 0.0;
          }
        };
        draw(rr[0]);
        for (int t0 = 0; t0 < steps; t0 += kWin) {
          if (use_reg) {
            n_reg += (lane < kWin && t0 + lane < steps && cln != 0) ? 1u : 0u;
            cln = clv[min(t0 + kWin + (lane & 7), tlast)];
          }
#pragma unroll
          for (int s = 0; s < kWin; ++s) {
            if (t0 + s < steps) {
              lds_barrier();  // the dot products of this step are in LDS
              if constexpr (FUSED) {
                int hi;
                if (__builtin_expect_with_probability(
                        soft_gamma<false>(dr, live, __fma_rn(dscale, (double)s_D[s & 1][rc], -from), &hi), 1, 1.0)) {
                  const int g = min(max(hi, kSoftMagicHi + QMIN), kSoftMagicHi + QMAX);
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
            }
          }
        }
      };
      if (soft_covers(dscale, aB, inv_s)) run(std::true_type{});
      else run(std::false_type{});
      if (n_gclamp) atomicAdd(&s_cnt[1], (unsigned long long)n_gclamp);
      if (n_reg) atomicAdd(&s_cnt[2], (unsigned long long)n_reg);
    }
  } else {
    // ======================================================================= class wave
    // rows cls0 .. cls0 + CPW - 1 of z
    const int cls0 = (wave - (wave > svc ? 1 : 0)) * CPW;
    auto row0_of = [&](int cc) { return ((int64_t)chain * K + cls0 + cc) * d; };
    const int s0 = lane * UPL;
    const int j0 = s0;
    const bool lane_ok = s0 < U;
    S2 zp[CPW][NP];
    int hv[CPW][CPL];
#pragma unroll
    for (int cc = 0; cc < CPW; ++cc) {
      const int32_t* __restrict__ hg = reinterpret_cast<const int32_t*>(a.h) + row0_of(cc);
      const int16_t* __restrict__ zg = reinterpret_cast<const int16_t*>(a.z) + row0_of(cc);
      int zv[CPL], hk[CPL];
#pragma unroll
      for (int k = 0; k < CPL; ++k) {  // unconditional: all loads in flight at once
        zv[k] = (int)zg[min(j0 + k, d - 1)];
        hk[k] = (int)hg[min(j0 + k, d - 1)];
      }
#pragma unroll
      for (int k = 0; k < CPL; ++k) asm volatile("" : "+v"(zv[k]), "+v"(hk[k]));
#pragma unroll
      for (int k = 0; k < CPL; ++k) {
        const bool ok = j0 + k < d;
        const int zz = ok ? zv[k] : 0, hh = ok ? hk[k] : 0;
        if (CPL == 1) zp[cc][0] = (S2)(short)(1 << 15);
        zp[cc][k / 2][k % 2] = (short)(zz + (1 << 15));
        hv[cc][k] = hh;
      }
    }
    uint32_t n_lane = 0;  // clamped coordinates, counted by the lane
    using LdsAcc = __attribute__((address_space(3))) AccT;
    LdsAcc* slotD[CPW][2];
#pragma unroll
    for (int cc = 0; cc < CPW; ++cc)
#pragma unroll
      for (int par = 0; par < 2; ++par)
        slotD[cc][par] = (LdsAcc*)(lane == 63 ? &s_D[par][cls0 + cc] : &s_dumpD[lane]);

    if (steps > 0) {
      const unsigned char* __restrict__ Xq = reinterpret_cast<const unsigned char*>(a.Xq) +
                                             (int64_t)chain * a.xq_chain_stride * 2;
      const int32_t* __restrict__ idx = ah.idx + (int64_t)local * ah.S;
      // Rows are padded to whole 8-byte groups: a fragment is read in pieces of 8 bytes at most, and
      // a piece past the row repeats the row's last group.  What lies past d is masked to zero.
      const uint32_t last_group = (uint32_t)((((int64_t)d * 2 + 7) / 8 - 1) * 8);
      uint32_t fm[NDW];
#pragma unroll
      for (int q = 0; q < NDW; ++q) {
        const int nv = d - (j0 + q * 2);
        fm[q] = nv >= 2 ? 0xFFFFFFFFu : (nv <= 0 ? 0u : 0xFFFFu);
      }
      uint32_t foff[(UPL + 3) / 4];
#pragma unroll
      for (int q = 0; q < (UPL + 3) / 4; ++q)
        foff[q] = UPL >= 4 ? min((uint32_t)(s0 * 2 + 8 * q), last_group) : (lane_ok ? (uint32_t)(s0 * 2) : 0u);
      uint32_t fr[kDep][NDW];
      auto request_row = [&](int slot, int i) {
        const unsigned char* rp = Xq + (int64_t)i * row_bytes;
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
      // the step's rounding bits of this lane's strips: halves of dwords, 2 UPL bytes
      uint32_t zb[kDep][CPW][NDW];
      const uint16_t* __restrict__ zst = ah.zbits + (int64_t)local * ah.S * K * ah.UP;
      const uint32_t zoff = (uint32_t)((cls0 * ah.UP + (lane_ok ? s0 : 0)) * 2);
      auto request_bits = [&](int slot, int t) {
        const unsigned char* bp = reinterpret_cast<const unsigned char*>(zst + (int64_t)t * K * ah.UP);
#pragma unroll
        for (int cc = 0; cc < CPW; ++cc) {
          const unsigned char* p = bp + (cc * ah.UP * 2) + lane_off(zoff);
          if constexpr (UPL == 1) {
            zb[slot][cc][0] = *reinterpret_cast<const uint16_t*>(p);
          } else if constexpr (UPL == 2) {
            zb[slot][cc][0] = *reinterpret_cast<const uint32_t*>(p);
          } else if constexpr (UPL == 4) {
            const uint2 v = *reinterpret_cast<const uint2*>(p);
            zb[slot][cc][0] = v.x;
            zb[slot][cc][1] = v.y;
          } else {
#pragma unroll
            for (int q = 0; q < UPL / 8; ++q) {
              const uint4 v = reinterpret_cast<const uint4*>(p)[q];
              zb[slot][cc][4 * q] = v.x; zb[slot][cc][4 * q + 1] = v.y;
              zb[slot][cc][4 * q + 2] = v.z; zb[slot][cc][4 * q + 3] = v.w;
            }
          }
        }
      };
      // lane l: number of the row of step t0 + (l & 7), and of the next window's
      int iv = idx[min(lane & 7, tlast)], ivn = idx[min(kWin + (lane & 7), tlast)];
      int clw = use_reg ? clv[min(lane & 7, tlast)] : 0;
#pragma unroll
      for (int s = 0; s < kDep; ++s) {
        request_row(s, __builtin_amdgcn_readlane(iv, s));
        request_bits(s, min(s, tlast));
      }
      // the row's fragment by step parity: this step's, and the next one's once it is unpacked
      S2 xp[2][NP];          // signed pairs
      int bias[2] = {0, 0};  // -128 sum x, for the bias of z in the dot product
      auto unpack = [&](int par, int slot) {
        bias[par] = 0;
#pragma unroll
        for (int q = 0; q < NDW; ++q) {
          xp[par][q] = __builtin_bit_cast(S2, fr[slot][q] & fm[q]);
          bias[par] = __builtin_amdgcn_sdot2(xp[par][q], (S2)(-128), bias[par], false);
        }
      };
      unpack(0, 0);
      request_row(0, __builtin_amdgcn_readlane(iv, kDep));

      for (int t0 = 0; t0 < steps; t0 += kWin) {
        const int ivnn = idx[min(t0 + 2 * kWin + (lane & 7), tlast)];
        const int clc = clw;
        if (use_reg) clw = clv[min(t0 + kWin + (lane & 7), tlast)];
#pragma unroll
        for (int s = 0; s < kWin; ++s) {
          if (t0 + s < steps) {
            AccT acc[CPW];
            // the high and the low bytes of z apart: 16 products of either fit 32 bits
#pragma unroll
            for (int cc = 0; cc < CPW; ++cc) {
              int ch = bias[s & 1], cl8 = 0;
#pragma unroll
              for (int q = 0; q < NP; ++q) {
                const uint32_t zq = __builtin_bit_cast(uint32_t, zp[cc][q]);
                ch = __builtin_amdgcn_sdot2(xp[s & 1][q], __builtin_bit_cast(S2, __builtin_bit_cast(W2, zp[cc][q]) >> (W2)(8)), ch, false);
                cl8 = __builtin_amdgcn_sdot2(xp[s & 1][q], __builtin_bit_cast(S2, zq & 0x00FF00FFu), cl8, false);
              }
              acc[cc] = ((AccT)ch << 8) + (AccT)cl8;
            }
            // the fold leaves the sum in lane 63, which stores it; the other lanes store their
            // partial folds into a dump row, so that no lane mask is set up and no lane is read
#pragma unroll
            for (int cc = 0; cc < CPW; ++cc) {
              *slotD[cc][s & 1] = (AccT)wave_fold_i64((long long)acc[cc]);
            }
            lds_barrier();
            __builtin_amdgcn_sched_barrier(0);
            // While the service wave evaluates the softmax: the part of the update that does not
            // need gamma, the next row's fragment, and the next requests.
            // h~ = 2^16 hh + hl, 0 <= hl < 2^16.  floor((-gamma x + r - h~) / 2^16) =
            // -hh - floor((gamma x + hl + 65535 - r) / 2^16), whose numerator fits 32 bits
            int hr[CPW][CPL], zr[CPW][CPL];
            auto before = [&](int cc) {
#pragma unroll
              for (int k = 0; k < CPL; ++k) {
                uint32_t rc = ~zb[s % kDep][cc][k / 2];
                asm("" : "+v"(rc));
                hr[cc][k] = (hv[cc][k] & 0xFFFF) + (int)((rc >> (16 * (k % 2))) & 0xFFFFu);
                zr[cc][k] = (int)(uint16_t)zp[cc][k / 2][k % 2] - (hv[cc][k] >> 16);
              }
            };
#pragma unroll
            for (int cc = 0; cc < CPW; ++cc) {
              if (!kLean) before(cc);
            }
            if (!kLean) request_bits(s % kDep, min(t0 + s + kDep, tlast));
            unpack((s + 1) & 1, (s + 1) % kDep);
            {
              const int sn = s + 1 + kDep;  // the slot just unpacked
              request_row((s + 1) % kDep, __builtin_amdgcn_readlane(sn < kWin ? iv : ivn, sn % kWin));
            }
            // all of it stays in front of the barrier
#pragma unroll
            for (int cc = 0; cc < CPW; ++cc)
#pragma unroll
              for (int k = 0; k < (kLean ? 0 : CPL); ++k) {
                asm volatile("" : "+v"(hr[cc][k]), "+v"(zr[cc][k]));
              }
#pragma unroll
            for (int q = 0; q < NP; ++q) asm volatile("" : "+v"(xp[(s + 1) & 1][q]));
            asm volatile("" : "+v"(bias[(s + 1) & 1]));
            __builtin_amdgcn_sched_barrier(0);
            lds_barrier();
            int ng[CPW];
#pragma unroll
            for (int cc = 0; cc < CPW; ++cc) ng[cc] = s_ng[s & 1][cls0 + cc];
            const int cl = __builtin_amdgcn_readlane(clc, s);  // 0 where there is no L2 term
            // u = z - gamma x - h~ (- c_lambda z), z = Q_(delta_m, b)(u)
#pragma unroll
            for (int cc = 0; cc < CPW; ++cc) {
              int v[CPL];
              uint32_t hit = 0;
              if (kLean) before(cc);
              if (__builtin_expect_with_probability(cl == 0, 1, 1.0)) {
#pragma unroll
                for (int k = 0; k < CPL; ++k)
                  v[k] = zr[cc][k] - (mad16(__builtin_bit_cast(uint32_t, xp[s & 1][k / 2]), k, ng[cc], hr[cc][k]) >> 16);
              } else {  // a step with an L2 draw
#pragma unroll
                for (int k = 0; k < CPL; ++k) {
                  uint32_t zq = __builtin_bit_cast(uint32_t, zp[cc][k / 2]);
                  asm volatile("" : "+v"(zq));  // unpacked here, not kept for every step
                  const int zk = (int)((zq >> (16 * (k % 2))) & 0xFFFFu) - 32768;
                  const long long n = (long long)ng[cc] * (int)xp[s & 1][k / 2][k % 2] + (long long)cl * zk + hr[cc][k];
                  v[k] = zr[cc][k] - (int)(n >> 16);
                }
              }
#pragma unroll
              for (int k = 0; k < CPL; ++k) hit |= (uint32_t)v[k];
              if (__builtin_expect_with_probability(__ballot((hit & 0xFFFF0000u) != 0) != 0, 0, 1.0)) {
#pragma unroll
                for (int k = 0; k < CPL; ++k) {
                  const int vc = min(max(v[k], 0), 65535);
                  n_lane += v[k] != vc ? 1u : 0u;
                  v[k] = vc;
                }
              }
#pragma unroll
              for (int q = 0; q < NP; ++q)
                zp[cc][q] = CPL == 1 ? S2{(short)v[0], (short)0x8000} : S2{(short)v[2 * q], (short)v[(2 * q + 1) % CPL]};
            }
            if (kLean) request_bits(s % kDep, min(t0 + s + kDep, tlast));
          }
          __builtin_amdgcn_sched_barrier(0);  // keep one step's temporaries from overlapping the next's
        }
        iv = ivn;
        ivn = ivnn;
      }
    }

    // ---- hand z out; after the epoch's last segment w~ <- w~ + delta_m z (option I)
    const double delta_m = sc[0];
#pragma unroll
    for (int cc = 0; cc < CPW; ++cc) {
      int16_t* __restrict__ zg = reinterpret_cast<int16_t*>(a.z) + row0_of(cc);
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
          const int zk = (int)(uint16_t)zp[cc][k / 2][k % 2] - (1 << 15);
          zg[jl + k] = (int16_t)zk;
          if (last) {
            const double step = __dmul_rn(delta_m, (double)zk);
            wg[jl + k] = lp ? (float)step : (float)__dadd_rn((double)wv[k], step);  // Alg. 2: w~ = delta w
          }
        }
      }
    }
    if (n_lane) atomicAdd(&s_cnt[0], (unsigned long long)n_lane);
  }
  __syncthreads();
  if (tid < 4) {  // the segments of an epoch follow each other on the stream
    const unsigned long long before = ah.t0 == 0 || tid == 3 ? 0ull : cnt_out[tid];
    cnt_out[tid] = before + (tid < 3 ? s_cnt[tid] : 0ull);
  }
}

using Kernel = SoftmaxKernel;

// one row of z per class wave up to 15 classes; 16 classes: two rows per wave, 8 + 1 waves
int classes_per_wave(int K) { return K > 15 ? 2 : 1; }
int block_threads(const halp_params& p, bool dense) {
  return p.b == 8 ? softmax_b8_threads(p.K, dense) : 64 * (p.K / classes_per_wave(p.K) + 1);
}

template <int UPL>
Kernel kernel_for(int K) {
  if (classes_per_wave(K) == 2) {
    if constexpr (UPL <= 8) return inner_softmax_kernel<UPL, 12, 2>;
    else return nullptr;
  } else if constexpr (UPL <= 4) {
    return inner_softmax_kernel<UPL, 16, 1>;
  } else {  // fewer waves, more registers each
    if (K + 1 <= 8) return inner_softmax_kernel<UPL, 8, 1>;
    if (K + 1 <= 12) return inner_softmax_kernel<UPL, 12, 1>;
    return inner_softmax_kernel<UPL, 16, 1>;
  }
}

Kernel kernel_for(int K, int upl) {
  switch (upl) {
    case 1: return kernel_for<1>(K);
    case 2: return kernel_for<2>(K);
    case 4: return kernel_for<4>(K);
    case 8: return kernel_for<8>(K);
    case 16: return kernel_for<16>(K);
    default: return nullptr;
  }
}

int strips_per_lane(const halp_params& p) {
  const int ct = 16 / p.b;
  const int U = (p.d + ct - 1) / ct;
  const int upl = (U + 63) / 64;
  int u2 = 1;
  while (u2 < upl) u2 *= 2;
  return u2;
}

// strips per class in the records: whole fragments, 16-byte multiples
int softmax_up(const halp_params& p) {
  const int ct = 16 / p.b, m = std::max(8, strips_per_lane(p));
  return ((p.d + ct - 1) / ct + m - 1) / m * m;
}

// Records of 16-bit halves: eight strips per lane, more than one class wave to a SIMD and few chains, whose records'
// traffic is nothing.  us per step, bytes / halves: 784 x 10 one chain 0.670 / 0.625, four 0.671 / 0.644, eight 0.698 / 0.695,
// sixteen 0.738 / 0.766, 256 1.31 / 2.18; 784 x 8 0.596 / 0.580, 784 x 7 0.516 / 0.545; 16 classes, 784 and 1024 coordinates: one chain
// 0.917 / 0.880 and 0.923 / 0.886, four 0.938 / 0.935 and 0.946 / 0.957, eight 0.994 / 1.017 and 1.032 / 1.107.
bool expanded(const halp_params& p) {
  return p.b == 8 && strips_per_lane(p) == 8 && p.K >= 8 && p.R <= (p.K > 15 ? 4 : 8);
}

Kernel kernel_for(const halp_params& p, bool dense) {
  return p.b == 8 ? softmax_b8_kernel(p.K, strips_per_lane(p), expanded(p), dense) : kernel_for(p.K, strips_per_lane(p));
}

}  // namespace

bool inner_softmax_takes(const halp_params& p) {
  if (p.algorithm == HALP_ALG_SVRG || p.loss != HALP_LOSS_SOFTMAX || p.B != 1 || p.K < 2 || p.K > 16) return false;
  return strips_per_lane(p) <= (p.b == 16 && p.K <= 15 ? 16 : 8);
}

// A launch takes as many chains as the device holds at once: a chain's step is mostly waiting, so
// several of them to a CU take little longer than one, and launches run one after the other.  us per
// step of all chains at 8 bits, 256 chains per launch and as many as fit: 64 x 2, 512 chains 0.98 and
// 0.57, 1024 chains 1.94 and 0.64; 64 x 10, 512 chains 1.13 and 0.69; 300 x 5, 1024 chains 2.33 and 1.81
// (two launches of 512: even shares, 768 and 256 took a third more); 784 x 5, 1024 chains 3.75 and 2.72.
size_t plan_inner_softmax(halp_handle& h) {
  const halp_params& p = h.p;
  if (!inner_softmax_takes(p)) return 0;
  auto resident = [&](bool dense, int threads) {
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void*>(kernel_for(p, dense)),
                                                     threads, 0) != hipSuccess)
      (void)hipGetLastError();
    return std::max(per_cu, 1);
  };
  int chains = resident(false, block_threads(p, false)) * h.num_cus;
  // 8 bits: the form without a row wave where it saves a launch.  A row wave makes the step of few chains shorter (784 x 3 0.485
  // instead of 0.502), but may be the fifth wave of a workgroup.  us per step, with a row wave / without: 64 x 3 2048 chains 1.84 /
  // 1.39, 64 x 7 768 1.33 / 0.79, 64 x 11 1024 2.58 / 1.62, 300 x 3 2048 1.85 / 1.76, 784 x 3 768 1.98 / 1.34, 784 x 7 1024 4.38 / 3.45.
  if (p.b == 8 && p.K < 15 && !expanded(p)) {
    auto launches = [&](int n) { return (p.R + n - 1) / n; };
    const int waves = block_threads(p, false) / 64;
    // what a CU holds whichever SIMDs their waves go to
    const int plain = std::max(resident(false, 256) / ((waves + 3) / 4), 1) * h.num_cus;
    const int dense = resident(true, block_threads(p, true)) * h.num_cus;
    h.softmax_dense = launches(dense) < launches(plain);
    chains = h.softmax_dense ? dense : plain;
  }
  return plan_ahead(h, softmax_up(p), chains, expanded(p));
}

// softmax, one row per step, up to 15 classes one wave each plus the service wave, 16 classes
// two to a wave (8 strips per lane at most then, for the registers of two rows of z), a
// class's row of z within one wave (8 strips per lane at most at 8 bits, 16 at 16 bits)
int inner_softmax_supported(const halp_handle& h) {
  if (!inner_softmax_takes(h.p)) return HALP_ERR_UNSUPPORTED;
  return (!h.bound || !h.buf.Xq || !h.ahead_ws) ? HALP_ERR_NOT_BOUND : HALP_OK;
}

int launch_inner_softmax(const halp_handle& h, uint32_t epoch, hipStream_t st) {
  const halp_params& p = h.p;
  const int rc = inner_softmax_supported(h);
  if (rc != HALP_OK) return rc;
  const InArgs a = make_inner_args(h, epoch);
  const Kernel kernel = kernel_for(p, h.softmax_dense);
  return for_segments(a, h, softmax_up(p), expanded(p), st, [&](const Ahead& s, int c0, int chains, int last) {
    hipLaunchKernelGGL(kernel, dim3(chains), dim3(block_threads(p, h.softmax_dense)), 0, st, a, s, c0, last);
    return hip_ok(hipGetLastError());
  });
}

}  // namespace halp
