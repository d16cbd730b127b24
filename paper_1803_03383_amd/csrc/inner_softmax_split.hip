// Inner loop of Algorithm 4 (LM-HALP) for softmax regression (K classes, one sampled row per
// step) on rows too wide for one workgroup: a chain is cut by columns across P workgroups.
//
// Workgroup p holds strips [p S, (p + 1) S) of every row of z ([K][d], strips of 16 rounding
// bits), S = 64 UPL: K / CPW class waves with UPL strips of CPW rows per lane in registers, and
// one service wave that evaluates the step's scalars.  z, h~ and the strips' Philox blocks stay
// in registers for the whole epoch; a class wave loads its fragment of the sampled row itself,
// eight steps ahead.
//
// The only thing the workgroups of a chain share is x_i^T z_c.  The class waves leave their parts
// in LDS, and the service wave adds them to the classes' 64-bit words in device memory with one
// device-scope atomic instruction: the part in the low 56 bits, a 1 in the top byte.  It then reads
// the K words until every top byte has moved by P since the word's last use (two sets of words, by
// step parity; words are never reset, both fields are taken as differences modulo 2^64), so
// arrival, sum and hand-over are one trip out and one trip back.  Integer sums: the order of
// arrival does not matter.  Every workgroup then evaluates the same K gammas.
//
// A wait has a limit: on a device whose CUs other work holds, some of a chain's workgroups may not
// get to run while the others wait.  z therefore goes to a workspace, and only a chain none of
// whose waits ran out hands it on; the others are run by the general kernel behind the launch,
// from the z they came with (one launch of workgroups that read a flag where there are none).
//
// One step:
//   class waves   x_i^T z_c over the slice, DPP fold, the part into LDS                    | barrier
//   service wave  adds the parts, makes part of the draws and of the softmax of the margins of
//                 a later step, polls, softmax after the offset, gamma_c into LDS
//   class waves   (the trip takes 0.5-0.7 us) a share of the next window's Philox blocks,
//                 what of the update needs no gamma                                        | barrier
//   class waves   integer update of their rows (8 bits: two packed instructions per strip, as in
//                 inner_softmax_b8.hip; what saturated is counted, and the next row unpacked, during the trip)
//
// What bounds it: latency, most of it the exchange.  One wave adds all classes at once because
// atomics of different waves queue up: with one atomic per class wave, words 256 bytes apart, a step of
// nothing but the exchange took 1.10 us at P = 4 and 1.57 at P = 20, this way 0.85 and 0.89 (K = 10,
// the parts on one XCD).  The atomics, and the first read behind them, are served by the memory
// a page of 4096 bytes is homed in: 0.23 us for the nearest, 0.36 for the farthest of the eight that
// alternate, so a chain's words lie in the page nearest to its XCD, which halp_create finds by timing
// (find_near): 1100 x 5 three chains 1.36 -> 1.12 us per step.  us per step of the loop (without the gradient pass; 2000 rows),
// one atomic per class wave -> the parts added by one wave, words in the nearest page -> at 8 bits the update in saturated
// halves too, clamps counted beside the exchange: 10000 x 10 8 bits one chain 2.73 -> 1.62 -> 1.44, five 2.76 -> 1.62 -> 1.45; 16
// bits five 3.15 -> 2.11; 4000 x 5 five chains 1.84 -> 1.28 -> 1.14; 2000 x 10 1.79 -> 1.45 -> 1.27; 1100 x 2 1.25 -> 1.16 ->
// 0.99; 256 chains of 1100 x 10 7.8 -> 7.0 -> 6.4.
#include <algorithm>

#include "halp_device.hpp"
#include "inner_args.hpp"
#include "softmax_ahead.hpp"
#include "softmax_fused.hpp"

namespace halp {
namespace {

constexpr int kWin = 8;          // steps per Philox window
constexpr int kIdxRing = 64;     // sample indices are drawn 64 steps at a time
constexpr int kKC = 16;          // classes are padded to one DPP row

// Exchange words: sixteen chains to eight pages of 4096 bytes, 256 bytes each in the page that lies nearest.
constexpr int kPage = 4096, kPages = 8, kChainsPerPage = 16, kPageWords = kPage / 8;

__host__ __device__ __forceinline__ size_t split_words(int chains) {
  return (size_t)((chains + kChainsPerPage - 1) / kChainsPerPage) * kPages * kPageWords;
}

__device__ __forceinline__ unsigned long long* words_of(unsigned long long* xbuf, int local, int page) {
  return xbuf + (int64_t)(local / kChainsPerPage * kPages + page) * kPageWords +
         (local % kChainsPerPage) * (kPageWords / kChainsPerPage);
}

// Workgroup x (on XCD x) finds the page of the first eight with the shortest atomics: near[x].
__global__ void find_near(unsigned long long* xbuf, int* near) {
  if (threadIdx.x != 0) return;
  long long best = INT64_MAX;
  int at = 0;
  for (int p = 0; p < kPages; ++p) {
    unsigned long long* w = xbuf + (int64_t)p * kPageWords + blockIdx.x * 16;
    long long least = INT64_MAX;
    for (int i = 0; i < 8; ++i) {
      const long long t0 = clock64();
      const unsigned long long v = __hip_atomic_fetch_add(w, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      asm volatile("" ::"v"((uint32_t)v) : "memory");
      const long long dt = clock64() - t0;
      least = dt < least ? dt : least;
    }
    if (least < best) {
      best = least;
      at = p;
    }
  }
  near[blockIdx.x] = blockIdx.x < 8 ? at : 0;
}

// LEAN: at most 128 registers, for chains that share a CU (plan_inner_softmax_split).
template <int BITS, int UPL, int CPW, int WAVES, bool LEAN>
__global__ __launch_bounds__(64 * WAVES) void inner_softmax_split_kernel(InArgs a, int P, int chain0, int nchains,
                                                                        int same_xcd, const int* near, unsigned long long* xbuf,
                                                                        int spin_limit) {
  using XT = typename std::conditional<BITS == 8, int8_t, int16_t>::type;
  using HT = typename std::conditional<BITS == 8, int16_t, int32_t>::type;
  using AccT = typename std::conditional<BITS == 8, int, long long>::type;
  constexpr int CT = 16 / BITS;     // coordinates per strip
  constexpr int CPL = UPL * CT;     // coordinates per lane and class
  constexpr int NDW = UPL / 2;      // dwords of a lane's row fragment
  constexpr bool PK = BITS == 8;    // 8 bits: the two coordinates of a strip as halves of one register
  typedef short S2 __attribute__((ext_vector_type(2)));
  typedef unsigned short W2 __attribute__((ext_vector_type(2)));
  constexpr int QMAX = (1 << (BITS - 1)) - 1, QMIN = -(1 << (BITS - 1));
  // Consecutive workgroups go to the eight XCDs in turn.  Where a chain's parts fit one XCD they
  // are placed there (the exchange is 0.15-0.3 us shorter); results do not depend on it.
  int local, part;
  if (same_xcd) {
    local = (int)(blockIdx.x & 7) + 8 * (int)(blockIdx.x / (8 * P));
    part = (int)(blockIdx.x >> 3) % P;
  } else {
    local = (int)blockIdx.x / P;
    part = (int)blockIdx.x - local * P;
  }
  if (local >= nchains) return;
  const int chain = chain0 + local;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int d = a.d, K = a.K;
  const int U = (d + CT - 1) / CT;
  const int NCW = K / CPW;
  const uint64_t seed = a.seed + (uint64_t)chain;
  const int64_t T = epoch_steps(seed, a.epoch, a.T, a.option2);
  const int64_t row_bytes = a.ldxq * (BITS / 8);
  const double* sc = a.scales + (int64_t)chain * 8;
  unsigned long long* cnt_out = reinterpret_cast<unsigned long long*>(a.counters + (int64_t)chain * 4);
  if (sc[7] != 0.0) return;  // converged or unusable gradient: no-op; the counters were cleared before the launch

  unsigned long long* words = words_of(xbuf, local, near[same_xcd ? blockIdx.x & 7 : 8]);  // [parity][class]: a 128-byte line per parity
  __shared__ long long s_part[kKC];  // this workgroup's x_i^T z_c
  __shared__ int s_idx[2][kIdxRing];
  __shared__ int s_ng[2][kKC];  // -gamma_c
  __shared__ int s_cl[2];       // c_lambda
  const bool use_reg = a.lambda > 0;
  const bool lp = a.lp != 0;
  const uint32_t N = (uint32_t)a.N;
  // sample index of step 64 blk + lane: any step number names a valid row
  auto draw_idx = [&](int64_t blk) {
    const uint64_t t = (uint64_t)blk * kIdxRing + (uint64_t)lane;
    const U4 r = stream_block(seed, kIdx, a.epoch, t >> 2);
    return (int)__umulhi(pick(r, (uint32_t)(t & 3)), N);
  };

  if (wave == NCW) {
    // ===================================================================== service wave
    __builtin_amdgcn_s_setprio(3);
    const float* __restrict__ phi = a.phi + (int64_t)chain * a.N * K;
    const double inv_s = sc[5];
    const double dscale = __dmul_rn(a.delta_d, sc[0]);
    const double aB = a.hyper[2 * chain];  // alpha / B, B = 1
    const double al = __dmul_rn(aB, a.lambda);
    unsigned int n_gclamp = 0, n_reg = 0, n_timeout = spin_limit < 0 ? 1u : 0u;
    const int c16 = lane & 15;
    const int lc = min(c16, K - 1);
    const bool live = lane < K;

    s_idx[0][lane] = draw_idx(0);
    __syncthreads();

    auto softmax = [&](double v) {  // this lane's class probability
      const double val = live ? v : -INFINITY;
      const double mx = row_max_f64(val);
      const double e = live ? halp_exp(__dadd_rn(val, -mx)) : 0.0;
      return __ddiv_rn(e, row_sum_f64(e));
    };
    // The step's gammas come from the short chain of softmax_fused.hpp, which has its classes in other lanes:
    // what is made one class per lane of a row of sixteen goes there through LDS's lane exchange, beside the
    // trip of the sums.  (16 bits with eight strips per lane, which kept the fixed order while this wave also drew
    // every step's words: 10000 x 10 five chains 2.88 us per step with the fixed order, 2.83 with the short chain.)
    const int rc = soft_class(lane);
    const bool live_f = rc < K;
    const bool fused = soft_covers(dscale, aB, inv_s);
    const double k2 = __dmul_rn(aB, inv_s);
    auto from_lane = [&](int src, int v) { return __builtin_amdgcn_ds_bpermute(src << 2, v); };
    auto from_lane64 = [&](int src, uint64_t v) {
      return (uint64_t)(uint32_t)from_lane(src, (int)(uint32_t)v) | ((uint64_t)(uint32_t)from_lane(src, (int)(v >> 32)) << 32);
    };
    // What a step needs and does not follow from z is made for four steps at a time, one to a row of 16 lanes: the
    // margins of the row, their softmax, the rounding words of gamma (class c of step t: word t K + c).  Half 0 are the first
    // four steps of a window, half 1 the others.
    float ph_req[2], ph[2];
    double p0q[2];
    uint32_t word[2];
    auto request_phi = [&](int half, int64_t win) {
      const int tn = (int)((win + 4 * half) & (2 * kIdxRing - 1)) + (lane >> 4);
      ph_req[half] = phi[(int64_t)s_idx[tn >> 6][tn & (kIdxRing - 1)] * K + lc];
    };
    // in three stages, so that none is longer than the trip that it runs beside
    U4 mk_word{};
    double mk_v = 0.0;
    auto make_half = [&](int half, int64_t win, int stage) __attribute__((always_inline)) {
      if (stage == 0) {
        const uint64_t n = (uint64_t)(win + 4 * half + (lane >> 4)) * (uint64_t)K + (uint64_t)lc;
        mk_word = philox_rounds<0, 4>(U4{(uint32_t)(n >> 2), (uint32_t)(n >> 34), a.epoch, (uint32_t)kGamma}, seed);
        const double val = c16 < K ? (double)ph_req[half] : -INFINITY;
        mk_v = __dadd_rn(val, -row_max_f64(val));
      } else if (stage == 1) {
        mk_word = philox_rounds<4, 7>(mk_word, seed);
        mk_v = c16 < K ? halp_exp(mk_v) : 0.0;
      } else {
        const uint32_t n3 = ((uint32_t)(win + 4 * half + (lane >> 4)) * (uint32_t)K + (uint32_t)lc) & 3;
        word[half] = pick(philox_rounds<7, 10>(mk_word, seed), n3);
        p0q[half] = __ddiv_rn(mk_v, row_sum_f64(mk_v));
        ph[half] = ph_req[half];
      }
    };
    request_phi(0, 0);
    request_phi(1, 0);
#pragma unroll
    for (int stage = 0; stage < 3; ++stage) make_half(0, 0, stage);
    request_phi(0, kWin);
    SoftDraw dr_n{};
    double from_n = 0.0;
    auto draw_fused = [&](int s) __attribute__((always_inline)) {  // step s of the window
      const int src = 16 * (s & 3) + rc, half = s >> 2;
      const float p = __builtin_bit_cast(float, from_lane(src, __builtin_bit_cast(int, ph[half])));
      const double q = __builtin_bit_cast(double, from_lane64(src, __builtin_bit_cast(uint64_t, p0q[half])));
      dr_n = soft_draw<true>(live_f, q, p, (uint32_t)from_lane(src, (int)word[half]), k2);
      from_n = lp && live_f ? (double)p : 0.0;  // Algorithm 2: x^T w is the whole margin
    };
    draw_fused(0);
    int cl64 = 0;  // lane l: the L2 draw of step 64 k + l
    unsigned long long old[2] = {0, 0};

    for (int64_t t0 = 0; t0 < T; t0 += kWin) {
      if ((t0 & (kIdxRing - 1)) == kIdxRing / 2) {  // the next 64 indices: first read three windows on
        const int64_t blk = (t0 / kIdxRing) + 1;
        s_idx[blk & 1][lane] = draw_idx(blk);
      }
      if (use_reg && (t0 & (kIdxRing - 1)) == 0) {
        const uint64_t n = (uint64_t)t0 + (uint64_t)lane;
        const uint32_t w = pick(stream_block(seed, kReg, a.epoch, n >> 2), (uint32_t)(n & 3));
        cl64 = (int)quantize_real(al, (double)(1 << BITS), w, 0.0, (double)QMAX, nullptr);
      }
#pragma unroll
      for (int s = 0; s < kWin; ++s) {
        const int64_t t = t0 + s;
        if (t < T) {
          const double from = from_n;
          const SoftDraw dr = dr_n;
          const int cl = use_reg ? __builtin_amdgcn_readlane(cl64, (int)(t & (kIdxRing - 1))) : 0;
          unsigned long long* w = words + (s & 1) * kKC + (live_f ? rc : 0);
          lds_barrier();  // the workgroup's parts are in LDS
          if (live_f && soft_first_copy(lane))
            __hip_atomic_fetch_add(w, (1ull << 56) + (unsigned long long)s_part[rc], __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
          // beside the trip of the sums: all that does not need them
          if (s < 3) make_half(1, t0, s);
          if (s >= 4 && s < 7) make_half(0, t0 + kWin, s - 4);
          draw_fused((s + 1) % kWin);
          unsigned long long v = old[s & 1];
          for (int spin = 0; n_timeout == 0; ++spin) {  // after one wait ran out, none is tried again
            if (live_f) v = __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            // arrivals so far: a signed part below 2^55 in magnitude may borrow from the top byte
            const bool missing = live_f && (uint32_t)((v - old[s & 1] + (1ull << 55)) >> 56) != (uint32_t)P;
            if (__ballot(missing) == 0) break;
            if (spin >= spin_limit) n_timeout = 1;  // only if a workgroup of the chain never ran: give up
          }
          const long long D = (long long)(v - old[s & 1] - ((unsigned long long)P << 56));
          old[s & 1] = v;
          // a window ahead, and behind the polls, which would wait for them
          if (s == 2) request_phi(1, t0 + kWin);
          if (s == 6) request_phi(0, t0 + 2 * kWin);
          double f = 0.0, fc = 0.0;  // gamma in the fixed order of roundings, classes in the first lanes
          auto fixed = [&](double moved) __attribute__((always_inline)) {
            const int src = 16 * (s & 3) + lc, half = s >> 2;
            const double a0 = (double)__builtin_bit_cast(float, from_lane(src, __builtin_bit_cast(int, ph[half])));
            const double p0 = __builtin_bit_cast(double, from_lane64(src, __builtin_bit_cast(uint64_t, p0q[half])));
            const double rho = __dmul_rn((double)(uint32_t)from_lane(src, (int)word[half]), 0x1p-32);
            const double p1 = softmax(lp ? moved : __dadd_rn(a0, moved));
            // beta_c = alpha (p_c(phi + x^T z) - p_c(phi)), gamma_c = Q_(delta_s, b)(beta_c)
            const double beta = __dmul_rn(aB, __dadd_rn(p1, -p0));
            f = floor(__dadd_rn(__dmul_rn(beta, inv_s), rho));
            fc = fmin(fmax(f, (double)QMIN), (double)QMAX);
            if (live) s_ng[s & 1][lane] = (int)(-fc);
          };
          int g, hi = 0;
          if (__builtin_expect_with_probability(
                  fused && soft_gamma<true>(dr, live_f, live_f ? __fma_rn(dscale, (double)D, -from) : 0.0, &hi), 1, 1.0)) {
            g = min(max(hi, kSoftMagicHi - QMAX), kSoftMagicHi - QMIN);
            s_ng[s & 1][rc] = g - kSoftMagicHi;  // (four lanes store the same word)
          } else {
            g = hi;
            fixed(__dmul_rn(dscale, (double)(long long)from_lane64((lc & 3) + 16 * (lc >> 2), (uint64_t)D)));
          }
          if (lane == 0) s_cl[s & 1] = cl;
          lds_barrier();  // gamma is out; the class waves update z
          n_gclamp += (live_f && soft_first_copy(lane) && g != hi) ? 1u : 0u;
          n_gclamp += (live && f != fc) ? 1u : 0u;
          n_reg += (lane == 0 && cl != 0) ? 1u : 0u;
        }
      }
    }
    if (part == 0) {  // the scalars are the same in every part
      if (n_gclamp) atomicAdd(&cnt_out[1], (unsigned long long)n_gclamp);
      if (n_reg) atomicAdd(&cnt_out[2], (unsigned long long)n_reg);
    }
    if (lane == 0 && n_timeout) atomicMax(&cnt_out[3], 1ull);
  } else {
    // ======================================================================= class wave
    const int cls0 = wave * CPW;
    const int s0 = (part * 64 + lane) * UPL;  // first strip of this lane in every row
    const int j0 = s0 * CT;
    const unsigned char* __restrict__ Xq = reinterpret_cast<const unsigned char*>(a.Xq) +
                                           (int64_t)chain * a.xq_chain_stride * (BITS / 8);
    // Rows are padded to whole 8-byte groups.  A lane past the row reads the row's start;
    // whatever lies past d is masked to zero, so that z stays zero there.
    const int64_t off0 = s0 < U ? (int64_t)s0 * 2 : 0;
    const int64_t off1 = UPL == 8 && s0 + 4 < U ? off0 + 8 : off0;
    uint32_t fm[PK ? 1 : NDW], fs[PK ? UPL : 1];  // 8 bits: byte selectors of a pair, 0x0C (a zero byte) past d
#pragma unroll
    for (int q = 0; q < NDW; ++q) {
      const int nv = d - (j0 + q * (32 / BITS));
      if (!PK) fm[q] = nv >= 32 / BITS ? 0xFFFFFFFFu : (nv <= 0 ? 0u : (1u << (nv * BITS)) - 1u);
    }
    if constexpr (PK) {
#pragma unroll
      for (int u = 0; u < UPL; ++u) {
        const int nv = d - (j0 + 2 * u), b = 2 * (u & 1);
        fs[u] = ((nv >= 2 ? (uint32_t)(b + 1) : 0x0Cu) << 24) | 0x0C000Cu | ((nv >= 1 ? (uint32_t)b : 0x0Cu) << 8);
      }
    }
    uint32_t fr[kWin][NDW];
    auto request = [&](int s, int i) {
      const unsigned char* rp = Xq + (int64_t)i * row_bytes;
      if constexpr (NDW == 1) {
        fr[s][0] = *reinterpret_cast<const uint32_t*>(rp + off0);
      } else {
        const uint2 v = *reinterpret_cast<const uint2*>(rp + off0);
        fr[s][0] = v.x; fr[s][1] = v.y;
        if constexpr (NDW == 4) {
          const uint2 u = *reinterpret_cast<const uint2*>(rp + off1);
          fr[s][2] = u.x; fr[s][3] = u.y;
        }
      }
    };
    // z and h~, 16 bits plain.  8 bits: packed, h~ and 256 z before the step, what was added to it, and their
    // saturated sum, whose high bytes are z and whose low bytes are cleared beside the exchange (inner_softmax_b8.hip)
    S2 hp[CPW][PK ? UPL : 1], zq[CPW][PK ? UPL : 1], add[CPW][PK ? UPL : 1], sum[CPW][PK ? UPL : 1];
    bool whole = true;  // |h~| of this wave's coordinates leaves room for -gamma x + r - h~ in 16 bits
    int z[CPW][PK ? 1 : CPL], hv[CPW][PK ? 1 : CPL];
    auto row_of = [&](int cc) { return ((int64_t)chain * K + cls0 + cc) * d; };
#pragma unroll
    for (int cc = 0; cc < CPW; ++cc) {
      const HT* __restrict__ hg = reinterpret_cast<const HT*>(a.h) + row_of(cc);
      const XT* __restrict__ zg = reinterpret_cast<const XT*>(a.z) + row_of(cc);
#pragma unroll
      for (int k = 0; k < CPL; ++k) {
        const int j = min(j0 + k, d - 1);
        const int zk = j0 + k < d ? (int)zg[j] : 0, hk = j0 + k < d ? (int)hg[j] : 0;
        if constexpr (PK) {
          sum[cc][k / 2][k % 2] = (short)(zk * 256);
          zq[cc][k / 2] = sum[cc][k / 2];
          add[cc][k / 2] = (S2)(0);
          hp[cc][k / 2][k % 2] = (short)hk;
          whole = whole && hk <= kWholeH && hk >= -kWholeH;
        } else {
          z[cc][k] = zk;
          hv[cc][k] = hk;
        }
      }
    }
    uint32_t zrw[CPW][UPL][4], zrn[CPW][UPL][4];  // this window's rounding words and the next one's
    // LEAN: a strip's number is opaque at the place of use.  The products of a block's first two rounds do not change from
    // window to window, and are carried through the loop otherwise, in 20 registers of the 154; made anew they cost 2 % of a step.
    auto strip = [&](int cc, int u) {
      uint32_t n = (uint32_t)((cls0 + cc) * U + s0 + u);
      if constexpr (LEAN) asm volatile("" : "+v"(n));
      return n;
    };
    auto draw_block = [&](uint32_t (&dst)[4], int cc, int u, uint32_t win) {
      const U4 r = zround_block(seed, a.epoch, strip(cc, u), win);
      dst[0] = r.x; dst[1] = r.y; dst[2] = r.z; dst[3] = r.w;
    };
#pragma unroll
    for (int cc = 0; cc < CPW; ++cc)
#pragma unroll
      for (int u = 0; u < UPL; ++u) draw_block(zrn[cc][u], cc, u, 0u);
    constexpr int kBlocks = CPW * UPL;  // a window's blocks
    static_assert(kBlocks == 4 || kBlocks % 8 == 0);
    U4 half_block{};
    unsigned long long n_zclamp = 0;  // counted by the wave (8 bits: by the lane)
    W2 n_half = (W2)(0), ones = (W2)(1);
    asm volatile("" : "+v"(ones));  // a value the compiler does not see: one packed minimum per strip
    __syncthreads();  // the first 64 indices are in LDS
    {
      const int iv = s_idx[0][lane & 7];
#pragma unroll
      for (int s = 0; s < kWin; ++s) request(s, __builtin_amdgcn_readlane(iv, s));
    }

    uint32_t xs[PK ? UPL : 1];  // 8 bits: the row in pairs, a coordinate in the high byte of its half
    auto unpack = [&](int slot) __attribute__((always_inline)) {
#pragma unroll
      for (int u = 0; u < (PK ? UPL : 1); ++u) xs[u] = PK ? __builtin_amdgcn_perm(0u, fr[slot][u / 2], fs[PK ? u : 0]) : 0u;
    };
    auto run = [&](auto whole_tag) __attribute__((always_inline)) {
      constexpr bool WHOLE = decltype(whole_tag)::value;
      for (int64_t t0 = 0; t0 < T; t0 += kWin) {
#pragma unroll
        for (int cc = 0; cc < CPW; ++cc)
#pragma unroll
          for (int u = 0; u < UPL; ++u)
#pragma unroll
            for (int w = 0; w < 4; ++w) zrw[cc][u][w] = zrn[cc][u][w];
        const int tn = (int)((t0 + kWin) & (2 * kIdxRing - 1)) + (lane & 7);
        const int idxn = s_idx[tn >> 6][tn & (kIdxRing - 1)];  // rows of the next window
#pragma unroll
        for (int s = 0; s < kWin; ++s) {
          if (t0 + s < T) {
            uint32_t xw[PK ? 1 : NDW];
            if constexpr (!PK) {
#pragma unroll
              for (int q = 0; q < NDW; ++q) xw[q] = fr[s][q] & fm[q];
            }
            S2 xp[PK ? UPL : 1];
            AccT acc[CPW];
#pragma unroll
            for (int cc = 0; cc < CPW; ++cc) acc[cc] = 0;
            auto x_of = [&](int k) { return (int)(int16_t)(xw[k / 2] >> (16 * (k % 2))); };  // 16 bits
            if constexpr (PK) {
#pragma unroll
              for (int cc = 0; cc < CPW; ++cc)
#pragma unroll
                for (int u = 0; u < UPL; ++u)
                  acc[cc] = (AccT)__builtin_amdgcn_sdot4((int)xs[u], __builtin_bit_cast(int, sum[cc][u]), (int)acc[cc], false);
            } else {  // two products of 16-bit factors fit 32 bits; their sums are added in 64
#pragma unroll
              for (int cc = 0; cc < CPW; ++cc)
#pragma unroll
                for (int k = 0; k + 1 < CPL; k += 2)
                  acc[cc] += (AccT)mad24(x_of(k), z[cc][k], mad24(x_of(k + 1), z[cc][k + 1], 0));
            }
#pragma unroll
            for (int cc = 0; cc < CPW; ++cc) {
              const long long D = BITS == 8 ? (long long)wave_fold_i32((int)acc[cc]) : wave_fold_i64((long long)acc[cc]);
              if (lane == 63) s_part[cls0 + cc] = D;
            }
            lds_barrier();
            // while the sums travel: blocks of the next window, and what of the update needs no gamma
#pragma unroll
            for (int q = 0; q < kBlocks / 8; ++q) {
              const int ub = s * (kBlocks / 8) + q;
              draw_block(zrn[ub / UPL][ub % UPL], ub / UPL, ub % UPL, (uint32_t)(t0 >> 3) + 1u);
            }
            if constexpr (kBlocks % 8 != 0) {  // four blocks to eight steps: half of one each
              const int ub = s / 2;
              if (s % 2 == 0) {
                half_block = philox_rounds<0, 5>(U4{strip(ub / UPL, ub % UPL), (uint32_t)(t0 >> 3) + 1u, a.epoch,
                                                    (uint32_t)kZround}, seed);
              } else {
                const U4 r = philox_rounds<5, 10>(half_block, seed);
                zrn[ub / UPL][ub % UPL][0] = r.x; zrn[ub / UPL][ub % UPL][1] = r.y;
                zrn[ub / UPL][ub % UPL][2] = r.z; zrn[ub / UPL][ub % UPL][3] = r.w;
              }
            }
            S2 crp[CPW][PK ? UPL : 1];
            if constexpr (PK) {
#pragma unroll
              for (int u = 0; u < UPL; ++u) xp[u] = __builtin_bit_cast(S2, xs[u]) >> (S2)(8);
              unpack((s + 1) % kWin);  // the next row
              request(s, __builtin_amdgcn_readlane(idxn, s));  // step t + 8
            }
            int hr[CPW][PK ? 1 : CPL];
#pragma unroll
            for (int cc = 0; cc < CPW; ++cc) {
              if constexpr (PK) {
                uint32_t off[UPL], hit = 0;  // not 0 in the halves that saturated at the last step
#pragma unroll
                for (int u = 0; u < UPL; ++u) {
                  const uint32_t v = __builtin_bit_cast(uint32_t, sum[cc][u]);
                  off[u] = v ^ __builtin_bit_cast(uint32_t, zq[cc][u] + add[cc][u]);
                  hit |= off[u];
                  zq[cc][u] = __builtin_bit_cast(S2, v & 0xFF00FF00u);
                  const uint32_t rp = __builtin_amdgcn_perm(0u, zrw[cc][u][s >> 1], (s & 1) ? 0x0C030C02u : 0x0C010C00u);
                  crp[cc][u] = __builtin_bit_cast(S2, rp) - hp[cc][u];  // r - h~
                }
                if (__ballot(hit != 0) != 0) {
#pragma unroll
                  for (int u = 0; u < UPL; ++u) n_half += __builtin_elementwise_min(__builtin_bit_cast(W2, off[u]), ones);
                }
              } else {
                // h~ = 2^16 hh + hl, 0 <= hl < 2^16: floor((-gamma x + r - h~) / 2^16) =
                // floor((-gamma x + r - hl) / 2^16) - hh, and that numerator fits 32 bits
#pragma unroll
                for (int k = 0; k < CPL; ++k)
                  hr[cc][k] = (int)((zrw[cc][k][s >> 1] >> (16 * (s & 1))) & 0xFFFFu) - (hv[cc][k] & 0xFFFF);
              }
            }
            lds_barrier();
            const int cl = use_reg ? __builtin_amdgcn_readfirstlane(s_cl[s & 1]) : 0;
#pragma unroll
            for (int cc = 0; cc < CPW; ++cc) {
              const int ng = s_ng[s & 1][cls0 + cc];
              if constexpr (PK) {
                if constexpr (WHOLE) {
                  const S2 ngp = S2{(short)ng, (short)ng};
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
                      const S2 xu = xp[u], zo = zq[cc][u], hu = hp[cc][u];
                      const int zk = (int)zo[e] >> 8;
                      int ad = 0;  // r - h~
                      if constexpr (WHOLE) {
                        const S2 cu = crp[cc][u];
                        ad = (int)cu[e];
                      } else {
                        ad = (int)((zrw[cc][u][s >> 1] >> (16 * (s & 1) + 8 * e)) & 0xFFu) - (int)hu[e];
                      }
                      const int zu = zk + (mad24(ng, (int)xu[e], mad24(-cl, zk, ad)) >> 8);
                      zc[e] = min(max(zu, QMIN), QMAX);
                      n_zclamp += zu != zc[e] ? 1 : 0;
                    }
                    sum[cc][u] = S2{(short)(zc[0] * 256), (short)(zc[1] * 256)};
                    add[cc][u] = sum[cc][u] - zq[cc][u];  // nothing left to count
                  }
                }
              } else {
#pragma unroll
                for (int k = 0; k < CPL; ++k) {
                  int num = mad24(ng, x_of(k), hr[cc][k]);
                  if (cl != 0) num = mad24(-cl, z[cc][k], num);
                  const int zu = z[cc][k] + (num >> 16) - (hv[cc][k] >> 16);
                  const int zc = min(max(zu, QMIN), QMAX);
                  n_zclamp += (unsigned long long)__builtin_popcountll(__ballot(zu != zc));
                  z[cc][k] = zc;
                }
              }
            }
            if constexpr (!PK) request(s, __builtin_amdgcn_readlane(idxn, s));  // step t + 8
          }
          __builtin_amdgcn_sched_barrier(0);  // keep one step's temporaries from overlapping the next's
        }
        if constexpr (PK) {
          n_zclamp += (unsigned long long)n_half[0] + (unsigned long long)n_half[1];
          n_half = (W2)(0);
        }
      }
    };
    if constexpr (PK) {
      unpack(0);
      if (__ballot(!whole) == 0) run(std::true_type{});
      else run(std::false_type{});
#pragma unroll
      for (int cc = 0; cc < CPW; ++cc)  // the last step's
#pragma unroll
        for (int u = 0; u < UPL; ++u) {
          const uint32_t off = __builtin_bit_cast(uint32_t, sum[cc][u]) ^ __builtin_bit_cast(uint32_t, zq[cc][u] + add[cc][u]);
          n_zclamp += ((off & 0xFFFFu) != 0 ? 1 : 0) + ((off >> 16) != 0 ? 1 : 0);
        }
    } else {
      run(std::true_type{});
    }

    // ---- hand z out (on to a.z, and w~ <- w~ + delta_m z: split_finish)
#pragma unroll
    for (int cc = 0; cc < CPW; ++cc) {
      XT* __restrict__ zg =
          reinterpret_cast<XT*>(xbuf + split_words(nchains)) + ((int64_t)local * K + cls0 + cc) * d;
#pragma unroll
      for (int k = 0; k < CPL; ++k) {
        int zk;
        if constexpr (PK) zk = (int)sum[cc][k / 2][k % 2] >> 8;
        else zk = z[cc][k];
        if (j0 + k < d) zg[j0 + k] = (XT)zk;
      }
    }
    if ((PK || lane == 0) && n_zclamp) atomicAdd(&cnt_out[0], n_zclamp);
  }
}

using Kernel = void (*)(InArgs, int, int, int, int, const int*, unsigned long long*, int);

int classes_per_wave(int K) { return K > 15 ? 2 : 1; }
int block_threads(int K) { return 64 * (K / classes_per_wave(K) + 1); }

template <int BITS, int UPL, int CPW>
Kernel kernel_for(int waves) {
  if (waves <= 8) return inner_softmax_split_kernel<BITS, UPL, CPW, 8, false>;
  if (waves <= 12) return inner_softmax_split_kernel<BITS, UPL, CPW, 12, false>;
  if constexpr (UPL * CPW <= 4) return inner_softmax_split_kernel<BITS, UPL, CPW, 16, false>;
  else return nullptr;
}

template <int BITS>
Kernel kernel_for(int K, int upl) {
  const int cpw = classes_per_wave(K), waves = block_threads(K) / 64;
  if (upl == 4) return cpw == 1 ? kernel_for<BITS, 4, 1>(waves) : kernel_for<BITS, 4, 2>(waves);
  return cpw == 1 ? kernel_for<BITS, 8, 1>(waves) : nullptr;
}

constexpr int kMaxWorkgroups = 127;  // of a chain: its additions are counted in the top byte of an exchange word

struct SplitShape {
  int upl, P;  // strips per lane, workgroups per chain
};

// Four strips per lane; eight where four would need more workgroups than an XCD has CUs (32) and a wave has the
// registers, or where beyond 24 the chains would no longer fit the device one workgroup to a CU.
// us per step of the loop, 4 / 8 strips: 16 bits 6500 x 10 (26 workgroups with four strips) three chains 1.71 / 1.99, 8000 x 10 (32)
// 1.80 / 2.04, 6500 x 5 1.53 / 1.64; 8 bits 15000 x 10 (30) 1.59 / 2.17; past 32 workgroups (40) 10000 x 8 16 bits 1.93 / 1.85,
// 10000 x 3 1.81 / 1.54, 20000 x 4 8 bits 1.68 / 1.32.  At 8 bits eight strips spill 28 registers with up to seven class waves and 204
// from eight on: 20000 x 10 1.92 / 2.30.
// Past kMaxWorkgroups four strips have no launch at all, so the row goes to eight while these fit.
SplitShape pick_shape(const halp_params& p, int num_cus) {
  const int ct = 16 / p.b, U = (p.d + ct - 1) / ct;
  const int P4 = (U + 255) / 256;
  const bool four = p.K >= 12 || P4 <= 24 ||
                    ((P4 <= 32 || (p.b == 8 && p.K >= 8 && P4 <= kMaxWorkgroups)) && (int64_t)p.R * P4 <= num_cus);
  const int upl = four ? 4 : 8;
  const int P = (U + 64 * upl - 1) / (64 * upl);
  return SplitShape{upl, P};
}

Kernel kernel_for(const halp_params& p, int upl, bool lean) {
  if (lean) return inner_softmax_split_kernel<8, 4, 1, 16, true>;
  return p.b == 8 ? kernel_for<8>(p.K, upl) : kernel_for<16>(p.K, upl);
}

// A workspace: the nearest pages [9], from its first whole page; the exchange words, from the next; z.
int* near_at(void* ws) {
  return reinterpret_cast<int*>((reinterpret_cast<uintptr_t>(ws) + kPage - 1) / kPage * kPage);
}
unsigned long long* words_at(void* ws) { return reinterpret_cast<unsigned long long*>(near_at(ws)) + kPageWords; }

}  // namespace

// A launch takes as many chains as the device holds workgroups for (a wait that other work makes run
// out all the same only costs time).  us per step of all chains, one workgroup to a CU and as many as
// fit (the general kernel): 1100 x 2 at 8 bits, 256 chains 5.3 and 1.25 (7.9), 1024 chains 18.1 and 4.9 (31.7);
// 1100 x 5, 256 chains 5.8 and 3.0 (9.8); 1100 x 2 at 16 bits, 256 chains 8.7 and 1.63 (7.7).  Where one fits:
// 1100 x 10, 256 chains 6.2 (18.3).
size_t plan_inner_softmax_split(halp_handle& h) {
  const halp_params& p = h.p;
  if (p.algorithm == HALP_ALG_SVRG || p.loss != HALP_LOSS_SOFTMAX || p.B != 1 || p.K < 2 || p.K > 16) return 0;
  if (inner_softmax_takes(p)) return 0;          // the register kernel has the shape
  if (p.b == 8 && p.d > 131071) return 0;        // int32 dot products stay exact
  const SplitShape shape = pick_shape(p, h.num_cus);
  const int P = shape.P;
  if (P > kMaxWorkgroups || P > h.num_cus) return 0;  // all workgroups of a chain resident
  const int waves = block_threads(p.K) / 64;
  auto per_cu = [&](bool lean, int threads) {
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, reinterpret_cast<const void*>(kernel_for(p, shape.upl, lean)),
                                                     threads, 0) != hipSuccess)
      (void)hipGetLastError();
    return std::max(n, 1);
  };
  auto launches = [&](int workgroups) { return (p.R + workgroups / P - 1) / (workgroups / P); };
  h.split_workgroups = per_cu(false, 64 * waves) * h.num_cus;
  // 8 bits, four strips, up to seven classes: the form with 128 registers, of which a CU holds more workgroups than of the one
  // with 154, where it saves a launch.  us per step, 154 registers / 128: 256 chains of 1100 x 4 4.8 / 2.4, x 5 5.2 / 3.0,
  // x 7 5.8 / 3.1, 128 of 3000 x 4 5.9 / 2.5; with as many launches either way 154 are 2 - 3 % faster.
  if (p.b == 8 && shape.upl == 4 && waves <= 8) {
    // What a CU holds whichever SIMDs their waves go to.  (Going by the occupancy of workgroups of 5 to 7 waves, two to a
    // CU, 256 chains of 1100 x 5 took 5.3 in two launches: the second workgroup waited for the first.)
    const int plain = std::max(per_cu(false, 256) / ((waves + 3) / 4), 1) * h.num_cus;
    const int lean = per_cu(true, 64 * waves) * h.num_cus;
    h.split_lean = launches(lean) < launches(plain);
    h.split_workgroups = h.split_lean ? lean : plain;
  }
  h.split_chains = std::min(p.R, h.split_workgroups / P);
  return 2 * kPage + split_words(h.split_chains) * sizeof(long long) + (size_t)h.split_chains * p.K * p.d * (p.b / 8);
}

int prepare_inner_softmax_split(const halp_handle& h) {
  hipLaunchKernelGGL(find_near, dim3(9), dim3(64), 0, 0, words_at(h.batch_xbuf), near_at(h.batch_xbuf));
  const int rc = hip_ok(hipGetLastError());
  return rc != HALP_OK ? rc : hip_ok(hipStreamSynchronize(0));  // a loop on any stream indexes with what it wrote
}

int inner_softmax_split_supported(const halp_handle& h) {
  if (h.split_chains == 0) return HALP_ERR_UNSUPPORTED;
  return !h.bound || !h.buf.Xq || !h.batch_xbuf ? HALP_ERR_NOT_BOUND : HALP_OK;
}

int launch_inner_softmax_split(const halp_handle& h, uint32_t epoch, hipStream_t s) {
  const halp_params& p = h.p;
  const int rc = inner_softmax_split_supported(h);
  if (rc != HALP_OK) return rc;
  const InArgs a = make_inner_args(h, epoch);
  const auto [upl, P] = pick_shape(p, h.num_cus);
  const Kernel kernel = kernel_for(p, upl, h.split_lean);
  unsigned long long* xbuf = words_at(h.batch_xbuf);
  const int* near = near_at(h.batch_xbuf);
  const bool report = h.spin_limit < 0;  // waits switched off: their outcome is what is asked for
  for (int c0 = 0; c0 < p.R; c0 += h.split_chains) {
    const int nc = std::min(h.split_chains, p.R - c0);
    const int same = P * ((nc + 7) / 8) <= h.split_workgroups / 8 && h.num_cus % 8 == 0;
    launch_split_prepare(reinterpret_cast<long long*>(xbuf), (int)split_words(nc), h.buf.counters + 4 * (int64_t)c0, 4 * nc, s);
    hipLaunchKernelGGL(kernel, dim3(same ? 8 * ((nc + 7) / 8) * P : nc * P), dim3(block_threads(p.K)), 0, s, a, P, c0,
                       nc, same, near, xbuf, h.spin_limit);
    int r = hip_ok(hipGetLastError());
    if (r == HALP_OK) r = launch_split_finish(a, h.buf.scales, xbuf + split_words(nc), c0, nc, report, p.b, s);
    if (r != HALP_OK) return r;
  }
  return report ? HALP_OK : launch_inner_generic(h, epoch, TraceBufs{}, s, true);
}

}  // namespace halp
