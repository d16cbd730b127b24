// Inner loop of Algorithm 4 (LM-HALP), register-resident form for few chains per CU: one sampled
// row per step (B = 1), one class, ONE "chain" wave that carries the whole of z, and helper waves
// on the other SIMDs of the CU.
//
// With a chain to itself a CU is bound by the step's dependent chain; a dependent vector
// instruction of a lone wave takes 8 cycles, an LDS round trip 66, so the chain wave is written
// for the fewest dependent instructions:
//   dot     one packed dot per strip (8 bits: two coordinates; at 16 bits one, multiplied and cut into
//           low 16 bits and the rest), DPP fold over 16 lanes.  Rows that
//           16 lanes hold (LANES = 16: the four rows of a wave do the same work) are done there;
//           wider rows are added up across the four rows of 16 lanes by one fp64 4x4x4 matrix
//           instruction (28 cycles; two row broadcasts and a lane read take 45), which multiplies
//           by the step's scale and adds the rounding draw in the same breath
//   scalar  gamma = floor(t), t = beta / delta_s + rho, out of ONE fused multiply-add: the draw
//           comes as C = 1.5 2^20 + 1 - rho, so that the high word of C - t' is a constant plus -gamma
//           and the low word is the fraction in units of 2^-32 (no floor, no conversion).  The method
//           fixes the order of roundings on the way to t, which differs from the fused form by
//           less than 2^-28 there: a step whose fraction lies within 2^-24 of an integer makes its
//           window (8 steps) be run again in that order from the z it began with.  Everything
//           else is the same integer in both, so results are those of the other kernels bit for bit
//   update  z is kept as 2^b z: n = -gamma x + r - h~, z <- saturating (z + n) with the low b bits
//           cleared -- the saturation of the 16-bit (b = 8) or 32-bit add is the box.  Three
//           instructions per strip.  An L2 draw cl takes -cl z along in the addend, r - h~ - cl z, made
//           while the dot is under way: two more instructions per strip in every step of an epoch that has draws
// Whatever does not depend on z is made by the helpers, up to two windows of 8 steps ahead, and
// handed over through LDS as one record per lane and step: per strip the sign-extended row
// values and r - h~.  A helper serves one or two of the strips of every lane: it draws their Philox
// blocks, requests the row fragments kSets - 1 windows ahead and writes its dwords of the records.
// Where -h~ / 2^b is not small in every coordinate, n leaves its word: the records then carry only
// the low b bits of -h~, z is kept as it is and the chain wave adds the rest behind the shift (FOLD = false;
// five instructions per strip, the sum of z and that rest being made beforehand).  A service wave refills the
// 256-step batches of step-indexed draws (sample indices, rounding draws of gamma and of the L2 term, margins and
// labels of the sampled rows), counts the steps with an L2 draw and the clamped coordinates: the chain wave stores
// the gammas of a window in LDS and the service wave, which holds a z of its own, takes it through the same steps with and
// without saturation.  One barrier per window orders every hand-over: in period w the chain wave
// consumes window w out of a ring of four and requests the first records of window w + 1 before the
// barrier, the helpers make window w + 2, and the service wave takes the records of window w - 1 out
// of the ring and goes through window w - 2.
//
// The chain wave is wave 0; the helpers and the service wave are placed on the other three
// SIMDs (waves w and w + 4 of a workgroup share a SIMD: wave 4 only keeps the barriers).
//
// This header holds the kernel template, inner_reg_lone_b8.hip and inner_reg_lone_b16.hip instantiate it, and the
// same with _l2 the builds for lambda > 0.
#pragma once

#include "inner_reg_impl.hpp"

namespace halp {
namespace innerlone {

using innerreg::kBatch;
using innerreg::kLossSquaredWithMargins;
using innerreg::kWin;
using innerreg::logistic_dl;
using innerreg::short2r;

typedef int int4r __attribute__((ext_vector_type(4)));
typedef int int2r __attribute__((ext_vector_type(2)));
typedef unsigned short ushort2r __attribute__((ext_vector_type(2)));

template <int LOSS>
constexpr bool logistic_c = LOSS == HALP_LOSS_LOGISTIC;

// waves of a workgroup: chain, helpers, the service wave, and wave 4 kept idle when there is one
constexpr int waves_of(int upl, int lanes) { return lanes == 16 || upl == 1 ? 3 : (upl == 2 ? 4 : 7); }

constexpr int kSlots = 4;  // windows of records in the ring
constexpr int kSets = 4;   // windows of row fragments a helper has in flight
constexpr int kHis = 3;    // windows of gammas that the chain wave leaves for the service wave

// C = kMagic + 1 - rho + kNear / 2^32: at this magnitude a double's last place is 2^-32 and its high
// word counts whole numbers.  Fractions within kNear / 2^32 of an integer are told by a low word of at most 2 kNear.
constexpr double kMagic = 0x1.8p20;
constexpr int kMagicHi = 0x41380000;
constexpr uint32_t kNear = 256;
constexpr double kDraw = kMagic + 1.0 + kNear * 0x1p-32;  // C + rho

// strip u of a lane; the strips a helper reads as one fragment are adjacent, those of its lanes too
template <int UPL, int LANES>
__device__ __forceinline__ int strip_of(int u, int lane) {
  if (LANES == 16) return 16 * u + (lane & 15);
  if (UPL == 8) return 128 * (u / 2) + 2 * lane + (u & 1);
  return 64 * u + lane;
}

// What a strip is: two coordinates as the halves of a word (8 bits) or one (16 bits), values times 2^b.
template <int BITS>
struct Strip;
template <>
struct Strip<8> {
  static constexpr int CT = 2;
  using Z = int8_t;
  using H = int16_t;
  static constexpr int kMask = (int)0xFF00FF00;
  // high parts of -h~ that may ride in the records: n stays inside its word; with L2 draws of up to kMaxDraw
  static constexpr int kSmallLow = -64, kSmallHigh = 62;
  static constexpr int kMaxDraw = 32, kSmallLowReg = -48, kSmallHighReg = 46;
  // n = -gamma x + c; g: kMagicHi - gamma, whose low half is -gamma
  static __device__ __forceinline__ int mad(int x, int g, int c) {
    const short2r gp = short2r{(short)g, (short)g};
    return __builtin_bit_cast(int, __builtin_bit_cast(short2r, x) * gp + __builtin_bit_cast(short2r, c));
  }
  static __device__ __forceinline__ int add_sat(int z, int n) {
    return __builtin_bit_cast(int, __builtin_elementwise_add_sat(__builtin_bit_cast(short2r, z), __builtin_bit_cast(short2r, n)));
  }
  static __device__ __forceinline__ int add(int z, int n) {
    return __builtin_bit_cast(int, __builtin_bit_cast(short2r, z) + __builtin_bit_cast(short2r, n));
  }
  // (n >> b) + k, before the clamp
  static __device__ __forceinline__ int shifted(int n, int k) {
    return __builtin_bit_cast(int, (__builtin_bit_cast(short2r, n) >> (short2r)(8)) + __builtin_bit_cast(short2r, k));
  }
  static __device__ __forceinline__ int high(int z) { return __builtin_bit_cast(int, __builtin_bit_cast(short2r, z) >> (short2r)(8)); }
  static __device__ __forceinline__ int clamp(int v) {  // to the box
    return __builtin_bit_cast(int, __builtin_elementwise_min(__builtin_elementwise_max(__builtin_bit_cast(short2r, v), (short2r)(-128)), (short2r)(127)));
  }
  // coordinates in which a and b differ (a minimum with a 1 that the compiler knows becomes a comparison per half)
  static __device__ __forceinline__ int differ(int a, int b) {
    int ones = 0x00010001;
    asm("" : "+s"(ones));
    return __builtin_bit_cast(int, __builtin_elementwise_min(__builtin_bit_cast(ushort2r, a ^ b), __builtin_bit_cast(ushort2r, ones)));
  }
  // coordinates in which the sum of z and n leaves its word: its sign there is not that of the saturated sum
  static __device__ __forceinline__ int clamped(int sat, int wrapped) {
    return __builtin_bit_cast(int, __builtin_bit_cast(ushort2r, sat ^ wrapped) >> (ushort2r)(15));
  }
  static __device__ __forceinline__ unsigned int counted(int acc) { return (unsigned int)(acc & 0xFFFF) + ((unsigned int)acc >> 16); }
  // x^T z of a strip, times 2^b, added to acc.  The saturating form, in which a zero to start from needs no register;
  // a lane's sum is at most 2^26.  (The instruction is the compiler's to place: a dot's result wants three wait states
  // before another kind of dot reads it, which the compiler keeps only between dots that it knows of)
  static __device__ __forceinline__ int dot(int x, int z, int acc) {
    return __builtin_amdgcn_sdot2(__builtin_bit_cast(short2r, x), __builtin_bit_cast(short2r, z), acc, true);
  }
  static __device__ __forceinline__ int dot(int x, int z) { return dot(x, z, 0); }
  // what takes the strip's bytes (strip `at` of a fragment) out of it and leaves zeros for coordinates that do not exist
  static __device__ __forceinline__ uint32_t take(int at, bool ok0, bool ok1) {
    return (ok0 ? (at ? 0x0200u : 0x0000u) : 0x0C00u) | (ok1 ? (at ? 0x03000000u : 0x01000000u) : 0x0C000000u) | 0x000C000Cu;
  }
  // the row value and the addend of a record from the fragment and the 16 rounding bits of step s; add: what the
  // record adds to them
  static __device__ __forceinline__ void record(uint32_t frag, int /*at*/, uint32_t take, uint32_t word, int s, int add, int* x, int* c) {
    // the bytes go to the high bytes of the halves and come back down with their signs
    const uint32_t up = __builtin_amdgcn_perm(0u, frag, take);
    const uint32_t rp = __builtin_amdgcn_perm(0u, word, (s & 1) ? 0x0C030C02u : 0x0C010C00u);
    *x = __builtin_bit_cast(int, __builtin_bit_cast(short2r, up) >> (short2r)(8));
    *c = __builtin_bit_cast(int, __builtin_bit_cast(short2r, rp) + __builtin_bit_cast(short2r, add));
  }
  static __device__ __forceinline__ int addend(int c, int /*x*/) { return c; }  // r - h~ (r + hl) of a record
  static __device__ __forceinline__ int value(int v, int e) { return e ? v >> 16 : (int)(short)v; }
  static __device__ __forceinline__ int join(int a, int b) { return (a & 0xFFFF) | (b << 16); }
};

template <>
struct Strip<16> {
  static constexpr int CT = 1;
  using Z = int16_t;
  using H = int32_t;
  static constexpr int kMask = (int)0xFFFF0000;
  static constexpr int kSmallLow = -16000, kSmallHigh = 16000;
  static constexpr int kMaxDraw = 4096, kSmallLowReg = -14000, kSmallHighReg = 14000;
  // The 24-bit multiplier takes g = kMagicHi - gamma as it is, i.e. kOffset - gamma; the records carry
  // c - kOffset x, and everything is exact modulo 2^32, where n lies.
  static constexpr int kOffset = kMagicHi & 0xFFFFFF;
  static __device__ __forceinline__ int mad(int x, int g, int c) { return mad24(g, x, c); }
  static __device__ __forceinline__ int add_sat(int z, int n) { return __builtin_elementwise_add_sat(z, n); }
  static __device__ __forceinline__ int add(int z, int n) { return (int)((uint32_t)z + (uint32_t)n); }
  static __device__ __forceinline__ int shifted(int n, int k) { return (n >> 16) + k; }
  static __device__ __forceinline__ int high(int z) { return z >> 16; }
  static __device__ __forceinline__ int clamp(int v) { return min(max(v, -32768), 32767); }
  static __device__ __forceinline__ int differ(int a, int b) {
    uint32_t one = 1;
    asm("" : "+s"(one));
    return (int)min((uint32_t)(a ^ b), one);
  }
  static __device__ __forceinline__ int clamped(int sat, int wrapped) { return (int)((uint32_t)(sat ^ wrapped) >> 31); }
  static __device__ __forceinline__ unsigned int counted(int acc) { return (unsigned int)acc; }
  static __device__ __forceinline__ uint32_t take(int /*at*/, bool ok0, bool /*ok1*/) { return ok0 ? 16 : 0; }  // bits
  static __device__ __forceinline__ void record(uint32_t frag, int at, uint32_t take, uint32_t word, int s, int add, int* x, int* c) {
    *x = __builtin_amdgcn_sbfe((int)frag, (uint32_t)(16 * at), take);
    *c = mad24(*x, -kOffset, (int)((s & 1) ? word >> 16 : word & 0xFFFFu) + add);
  }
  static __device__ __forceinline__ int addend(int c, int x) { return mad24(x, kOffset, c); }
  static __device__ __forceinline__ int value(int v, int) { return v; }
  static __device__ __forceinline__ int join(int a, int) { return a; }
};

// LANES: lanes that share a row of z, 64 or 16 (four copies of the same work in a wave).
// PAIR: built for several workgroups per CU (more chains than CUs), at most 128 registers per lane.
// REG: lambda > 0, steps may have L2 draws.
template <int BITS, int LOSS, int UPL, int LANES, bool PAIR, bool REG>
__global__ __launch_bounds__(64 * waves_of(UPL, LANES), PAIR ? 4 : 2) void inner_reg_lone_kernel(InArgs a) {
  static_assert((UPL == 2 && (LANES == 64 || BITS == 8)) || (LANES == 64 && (UPL == 4 || UPL == 8 || (UPL == 1 && BITS == 16))), "the forms that are launched");
  using S = Strip<BITS>;
  constexpr int CT = S::CT;
  constexpr int NQ = UPL > 1 ? UPL / 2 : 1;  // vectors of a record: UPL row values, then UPL of r - h~
  constexpr int QW = UPL > 1 ? 4 : 2;        // dwords of one
  using RecV = typename std::conditional<UPL == 1, int2r, int4r>::type;
  using ZT = typename S::Z;
  using HT = typename S::H;
  constexpr int QMAX = (1 << (BITS - 1)) - 1, QMIN = -(1 << (BITS - 1));
  constexpr int kMask = 2 * kBatch - 1;
  const int chain = blockIdx.x;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // Roles by wave.  Waves w and w + 4 share a SIMD and wave 0 is the chain wave, so wave 4 only
  // keeps the barriers.  The service wave has a SIMD to itself where the row is wide (counting
  // the clamps of a strip takes about as long as serving it): 16 lanes: wave 1 serves every strip,
  // wave 2 is the service wave, and so with one strip per lane.  2: waves 1, 2 one strip each, service wave 3.  4 and 8: waves
  // 1, 2, 5, 6 one or two strips each, service wave 3.
  constexpr int kStripsHere = UPL == 8 ? 2 : 1;  // of a lane, served by a helper
  int first_strip = -1;
  if (LANES == 16 || UPL == 1) first_strip = wave == 1 ? 0 : -1;
  else if (wave == 1 || wave == 2) first_strip = kStripsHere * (wave - 1);
  else if (UPL >= 4 && (wave == 5 || wave == 6)) first_strip = kStripsHere * (wave - 3);
  const bool is_service = wave == (LANES == 16 || UPL == 1 ? 2 : 3);
  const int d = a.d;
  const int U = (d + CT - 1) / CT;  // strips in a row
  const uint32_t N = (uint32_t)a.N;
  const int64_t row_bytes = a.ldxq * (BITS / 8);
  const unsigned char* __restrict__ Xq =
      reinterpret_cast<const unsigned char*>(a.Xq) + (int64_t)chain * a.xq_chain_stride * (BITS / 8);
  const float* __restrict__ phi = a.phi + (int64_t)chain * a.N;
  const float* __restrict__ y =
      reinterpret_cast<const float*>(a.y) + (int64_t)chain * a.y_chain_stride;
  const HT* __restrict__ hg = reinterpret_cast<const HT*>(a.h) + (int64_t)chain * d;
  ZT* __restrict__ zg = reinterpret_cast<ZT*>(a.z) + (int64_t)chain * d;
  float* __restrict__ wg = a.w + (int64_t)chain * d;
  const double* sc = a.scales + (int64_t)chain * 8;
  uint64_t* cnt_out = a.counters + (int64_t)chain * 4;
  const uint64_t seed = a.seed + (uint64_t)chain;
  const int64_t T = epoch_steps(seed, a.epoch, a.T, a.option2);
  const int64_t nwin = (T + kWin - 1) / kWin;

  if (sc[7] != 0.0) {  // converged or unusable gradient: the epoch is a no-op
    if (tid < 4) cnt_out[tid] = 0;
    return;
  }

  __shared__ __attribute__((aligned(16))) int s_idx[2 * kBatch];
  __shared__ __attribute__((aligned(16))) double s_c[2 * kBatch];  // kDraw - rho
  __shared__ __attribute__((aligned(16))) short s_ncl[REG ? 2 * kBatch : 8];  // L2 draws, negated
  constexpr bool kMargins = LOSS != HALP_LOSS_SQUARED;
  __shared__ __attribute__((aligned(16))) float s_phi[kMargins ? 2 * kBatch : 4];
  __shared__ __attribute__((aligned(16))) float s_y[logistic_c<LOSS> ? 2 * kBatch : 4];
  // logistic loss: l'(phi_i) of the sampled rows, which no step has to evaluate itself
  __shared__ __attribute__((aligned(16))) double s_dl0[logistic_c<LOSS> ? 2 * kBatch : 2];
  __shared__ __attribute__((aligned(16))) int s_hi[kHis][kWin];  // kMagicHi - gamma of the steps, before the clamp
  __shared__ unsigned long long s_cnt[4];
  __shared__ int s_fold;  // 1: the whole of -h~ rides in the records (set by the chain wave before the first barrier)
  // records: [slot of the ring][step of the window][vector][lane]
  extern __shared__ __attribute__((aligned(16))) int s_rec[];
  auto rec_at = [&](int slot, int s, int q) -> const RecV* {
    return reinterpret_cast<const RecV*>(s_rec) + ((slot * kWin + s) * NQ + q) * LANES + (lane & (LANES - 1));
  };
  auto split_record = [&](const RecV (&r)[NQ], int (&x)[UPL], int (&cr)[UPL]) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < UPL; ++u) {
      x[u] = r[u / QW][u % QW];
      cr[u] = r[(UPL + u) / QW][(UPL + u) % QW];
    }
  };

  const double delta_m = sc[0], inv_s = sc[5];
  const double dscale = __dmul_rn(a.delta_d, delta_m);
  const double aB = a.hyper[2 * chain];  // B = 1: alpha / 1
  constexpr bool logistic = LOSS == HALP_LOSS_LOGISTIC;
  constexpr bool need_phi = LOSS != HALP_LOSS_SQUARED;
  const bool lp = a.lp != 0;
  const double al = __dmul_rn(aB, a.lambda);
  // a draw is at most floor(al 2^b) + 1 (larger ones: every step in the fixed order, in wide arithmetic)
  const bool reg_small = REG && al * (double)(1 << BITS) < (double)S::kMaxDraw;

  if (tid < 4) s_cnt[tid] = 0;

  // z of a lane's strips (zeros past the row, where no record changes them) and the high part of -h~; true where every
  // high part is small.  With -h~ = 2^b hh + hl, 0 <= hl < 2^b, and every hh in [-64, 62] (16 bits: [-16000, 16000]),
  // n = -gamma x + r - h~ fits its word of 2 b bits (|gamma x| <= 2^(2b-2), 0 <= r < 2^b); with an L2 draw
  // cl <= 32 (4096) n has another cl z, |cl z| <= 2^12 (2^27), and hh lies in [-48, 46] ([-14000, 14000]).
  auto load_z = [&](int (&zp)[UPL], int (&hh)[UPL]) -> bool {
    bool small = true;
#pragma unroll
    for (int u = 0; u < UPL; ++u) {
      int zv[2] = {0, 0}, hv[2] = {0, 0};
#pragma unroll
      for (int e = 0; e < CT; ++e) {
        const int j = CT * strip_of<UPL, LANES>(u, lane) + e;
        const bool ok = j < d;
        zv[e] = ok ? (int)zg[ok ? j : 0] : 0;
        hv[e] = ok ? (int)((-(int64_t)hg[ok ? j : 0]) >> BITS) : 0;
        small = small && hv[e] >= (REG ? S::kSmallLowReg : S::kSmallLow) && hv[e] <= (REG ? S::kSmallHighReg : S::kSmallHigh);
      }
      zp[u] = S::join(zv[0], zv[1]);
      hh[u] = S::join(hv[0], hv[1]);
    }
    return small;
  };
  // z <- Q(z - gamma x - h~) of a strip; g: kMagicHi - gamma.  fold: c holds r - h~ and z is kept times 2^b, else c
  // holds r + hl and hh goes to z beforehand (left to itself the compiler adds the two one after the other behind
  // the shift, which waits for gamma)
  auto begin_strip = [&](int z, int hh, auto fold_tag) __attribute__((always_inline)) -> int {
    if constexpr (decltype(fold_tag)::value) return z;
    int zb = S::add(hh, z);
    if constexpr (BITS == 8) asm("" : "+v"(zb));  // (at 16 bits the registers are worth more)
    return zb;
  };
  auto step_strip = [&](int zb, int x, int g, int c, auto fold_tag) __attribute__((always_inline)) -> int {
    const int n = S::mad(x, g, c);
    if constexpr (decltype(fold_tag)::value) return S::add_sat(zb, n) & S::kMask;
    else return S::clamp(S::shifted(n, zb));
  };
  // the addend of a step with an L2 draw; ncl: -cl
  auto with_draw = [&](int z, int ncl, int c, auto fold_tag) __attribute__((always_inline)) -> int {
    return S::mad(decltype(fold_tag)::value ? S::high(z) : z, ncl, c);
  };
  // z <- Q(z - gamma x - h~ - cl z) in wide arithmetic on the coordinates, for draws of any size (steps in the
  // fixed order); g here is -gamma itself
  using Wide = typename std::conditional<BITS == 8, int, int64_t>::type;
  auto step_strip_reg = [&](int z, int x, int g, int ncl, int c, int hh, auto fold_tag, int* clamped) __attribute__((always_inline)) -> int {
    constexpr int kShift = decltype(fold_tag)::value ? BITS : 0;
    int zn[2] = {0, 0};
    const int cc = S::addend(c, x);
#pragma unroll
    for (int e = 0; e < CT; ++e) {
      const Wide zk = S::value(z, e) >> kShift, xk = S::value(x, e);
      const Wide hr = (decltype(fold_tag)::value ? 0 : (Wide)S::value(hh, e) << BITS) + S::value(cc, e);
      const Wide zuk = zk + ((g * xk + ncl * zk + hr) >> BITS);
      const Wide zc = zuk < QMIN ? QMIN : (zuk > QMAX ? QMAX : zuk);
      if (clamped) *clamped += zuk != zc ? 1 : 0;
      zn[e] = (int)zc << kShift;
    }
    return S::join(zn[0], zn[1]);
  };
  // z as it is <-> as the steps keep it
  auto keep_z = [&](int (&zp)[UPL], auto fold_tag) __attribute__((always_inline)) {
    if constexpr (decltype(fold_tag)::value) {
#pragma unroll
      for (int u = 0; u < UPL; ++u) zp[u] = S::join(S::value(zp[u], 0) << BITS, S::value(zp[u], 1) << BITS);
    }
  };

  if (is_service) {
    // ============================ service wave ============================
    int zs[UPL], hh[UPL];
    (void)load_z(zs, hh);
    // draws that depend on the step number only, 256 steps per batch
    auto fill_batch = [&](int64_t bb) {
      const int half = (int)(bb & 1) * kBatch;
      const uint64_t blk = (uint64_t)bb * 64 + (uint64_t)lane;
      const U4 ri = stream_block(seed, kIdx, a.epoch, blk);
      const U4 rg = stream_block(seed, kGamma, a.epoch, blk);
      int4 iv;
      iv.x = (int)__umulhi(ri.x, N); iv.y = (int)__umulhi(ri.y, N);
      iv.z = (int)__umulhi(ri.z, N); iv.w = (int)__umulhi(ri.w, N);
      *reinterpret_cast<int4*>(&s_idx[half + 4 * lane]) = iv;
      if constexpr (need_phi) {
        float4 pv;
        pv.x = phi[iv.x]; pv.y = phi[iv.y]; pv.z = phi[iv.z]; pv.w = phi[iv.w];
        *reinterpret_cast<float4*>(&s_phi[half + 4 * lane]) = pv;
        if constexpr (logistic) {
          float4 yv;
          yv.x = y[iv.x]; yv.y = y[iv.y]; yv.z = y[iv.z]; yv.w = y[iv.w];
          *reinterpret_cast<float4*>(&s_y[half + 4 * lane]) = yv;
          s_dl0[half + 4 * lane + 0] = logistic_dl((double)pv.x, (double)yv.x);
          s_dl0[half + 4 * lane + 1] = logistic_dl((double)pv.y, (double)yv.y);
          s_dl0[half + 4 * lane + 2] = logistic_dl((double)pv.z, (double)yv.z);
          s_dl0[half + 4 * lane + 3] = logistic_dl((double)pv.w, (double)yv.w);
        }
      }
      auto magic = [](uint32_t r) { return __dadd_rn(kDraw, -__dmul_rn((double)r, 0x1p-32)); };  // exact
      s_c[half + 4 * lane + 0] = magic(rg.x);
      s_c[half + 4 * lane + 1] = magic(rg.y);
      s_c[half + 4 * lane + 2] = magic(rg.z);
      s_c[half + 4 * lane + 3] = magic(rg.w);
      if constexpr (REG) {
        const U4 rr = stream_block(seed, kReg, a.epoch, blk);
        const double two_b = (double)(1 << BITS);
        short4 cv;
        cv.x = (short)-quantize_real(al, two_b, rr.x, 0.0, (double)QMAX, nullptr);
        cv.y = (short)-quantize_real(al, two_b, rr.y, 0.0, (double)QMAX, nullptr);
        cv.z = (short)-quantize_real(al, two_b, rr.z, 0.0, (double)QMAX, nullptr);
        cv.w = (short)-quantize_real(al, two_b, rr.w, 0.0, (double)QMAX, nullptr);
        *reinterpret_cast<short4*>(&s_ncl[half + 4 * lane]) = cv;
      }
    };
    // Clamped coordinates: this wave holds a z of its own and takes it through the steps once more, with
    // the gammas that the chain wave leaves in s_hi; a coordinate was clamped where the sums with and
    // without saturation differ.  The records of window w are taken out of the ring in period w + 1
    // and gone through in period w + 2, when the chain wave's stores have landed for certain.
    unsigned long long n_lane = 0;  // this lane's count of clamped coordinates: up to 16 of a step, of up to 2^32 steps
    unsigned int n_gclamp = 0;      // clamped gammas
    unsigned int n_reg = 0;         // steps with an L2 draw
    RecV r[kWin][NQ];
    auto take = [&](int64_t w) __attribute__((always_inline)) {
#pragma unroll
      for (int s = 0; s < kWin; ++s)
#pragma unroll
        for (int q = 0; q < NQ; ++q) r[s][q] = *rec_at((int)(w & (kSlots - 1)), s, q);
    };
    int part = 0;  // of s_hi, the next to be counted
    // kind_tag: 0 no L2 draws, 1 draws of up to kMaxDraw, in eight steps; 2 whatever there is, in `steps` of them
    auto count_steps = [&](int64_t w, int steps, auto kind_tag, auto fold_tag) __attribute__((always_inline)) {
      constexpr int KIND = decltype(kind_tag)::value;
      const int base = (int)((w * kWin) & kMask);
      const int4r h0 = *reinterpret_cast<const int4r*>(&s_hi[part][0]), h1 = *reinterpret_cast<const int4r*>(&s_hi[part][4]);
      const int hi[kWin] = {h0[0], h0[1], h0[2], h0[3], h1[0], h1[1], h1[2], h1[3]};
      int4r nc = int4r{0, 0, 0, 0};
      if constexpr (KIND == 1) nc = *reinterpret_cast<const int4r*>(&s_ncl[base]);
      int acc = 0;  // at most 8 UPL per half and window
      int wide = 0;
#pragma unroll
      for (int s = 0; s < kWin; ++s) {
        if (KIND < 2 || s < steps) {
          const int pair = nc[s / 2];
          int ncl = (s & 1) ? pair >> 16 : (int)(short)pair;
          if constexpr (KIND == 2) ncl = REG ? __builtin_amdgcn_readfirstlane((int)s_ncl[REG ? base + s : 0]) : 0;
          const int g = min(max(hi[s], kMagicHi - QMAX), kMagicHi - QMIN);
          int x[UPL], cr[UPL];
          split_record(r[s], x, cr);
          // (all strips go through one instruction before the next: one strip after the other, each would wait for
          // its own results; at 16 bits there are not the registers for it)
          constexpr int G = BITS == 8 ? UPL : 1;
          auto next = [&]() __attribute__((always_inline)) { if constexpr (BITS == 8) __builtin_amdgcn_sched_barrier(0); };
#pragma unroll
          for (int u = 0; u < UPL; u += G) {
            int n[G], v[G];
            if (KIND == 2 && ncl != 0) {
#pragma unroll
              for (int k = 0; k < G; ++k)
                zs[u + k] = step_strip_reg(zs[u + k], x[u + k], g - kMagicHi, ncl, cr[u + k], hh[u + k], fold_tag, &wide);
              continue;
            }
#pragma unroll
            for (int k = 0; k < G; ++k)
              n[k] = S::mad(x[u + k], g, KIND == 1 ? with_draw(zs[u + k], ncl, cr[u + k], fold_tag) : cr[u + k]);
            if constexpr (decltype(fold_tag)::value) {
#pragma unroll
              for (int k = 0; k < G; ++k) {
                v[k] = S::add_sat(zs[u + k], n[k]);
                acc = S::add(acc, S::clamped(v[k], S::add(zs[u + k], n[k])));
                zs[u + k] = v[k] & S::kMask;
              }
            } else {
#pragma unroll
              for (int k = 0; k < G; ++k) zs[u + k] = begin_strip(zs[u + k], hh[u + k], fold_tag);
              next();
#pragma unroll
              for (int k = 0; k < G; ++k) v[k] = S::shifted(n[k], zs[u + k]);
              next();
#pragma unroll
              for (int k = 0; k < G; ++k) zs[u + k] = S::clamp(v[k]);
              next();
#pragma unroll
              for (int k = 0; k < G; ++k) acc = S::add(acc, S::differ(v[k], zs[u + k]));
            }
          }
        }
      }
      n_lane += S::counted(acc) + (unsigned int)wide;
    };
    auto count_window = [&](int64_t w, auto fold_tag) __attribute__((always_inline)) {
      const int64_t left = T - w * kWin;
      const int steps = (int)(left < kWin ? left : kWin);
      if (left >= kWin && (!REG || reg_small)) count_steps(w, kWin, std::integral_constant<int, REG ? 1 : 0>{}, fold_tag);
      else count_steps(w, steps, std::integral_constant<int, 2>{}, fold_tag);
      const int hi = s_hi[part][lane & (kWin - 1)];
      n_gclamp += (unsigned int)__builtin_popcountll(__ballot(lane < steps && (hi < kMagicHi - QMAX || hi > kMagicHi - QMIN)));
      if constexpr (REG)
        n_reg += (unsigned int)__builtin_popcountll(__ballot(lane < steps && s_ncl[(int)((w * kWin) & kMask) + (lane & (kWin - 1))] != 0));
      part = part == kHis - 1 ? 0 : part + 1;
    };
    fill_batch(0);
    __syncthreads();  // P0: the first batch is in place
    __syncthreads();  // P1: the records of windows 0 and 1 are in place
    auto run = [&](auto fold_tag) __attribute__((always_inline)) {
      keep_z(zs, fold_tag);
      for (int64_t w = 0; w < nwin + 2; ++w) {
        if (w >= 2) count_window(w - 2, fold_tag);
        if (w >= 1 && w <= nwin) take(w - 1);
        // window w = 32 m + 1: every reader has left batch m - 1, whose half takes batch m + 1 (the first to read indices
        // out of it are the helpers in period 32 m + 27; an epoch that ends before then has nobody who does)
        if ((w & (kBatch / kWin - 1)) == 1 && w < nwin) fill_batch(w / (kBatch / kWin) + 1);
        if (w <= nwin) __syncthreads();  // w = nwin: P2, the last gammas are in place
      }
    };
    if (s_fold) run(std::true_type{});
    else run(std::false_type{});
    if (lane < LANES) atomicAdd(&s_cnt[0], n_lane);  // (it stood at 0 behind P0)
    if (lane == 0) {
      s_cnt[1] = n_gclamp;
      s_cnt[2] = n_reg;
    }
    __syncthreads();  // the counters
    return;
  }

  if (first_strip >= 0) {
    // ============================ helper wave =============================
      constexpr int SPH = kStripsHere;
      // 16 lanes: lane h of the helper serves strip h mod 16 UPL, i.e. strip h / 16 of lane h mod 16
      const int g0 = LANES == 16 ? lane & (16 * UPL - 1) : 64 * first_strip + SPH * lane;  // the first of them in the row
      const int owner = LANES == 16 ? g0 & 15 : lane;
      const int u0 = LANES == 16 ? g0 >> 4 : first_strip;
      int hlp[SPH];  // what a record adds to the rounding bits: the low b bits of -h~, or the whole of it
      int hfp[SPH];  // where every -h~ / 2^b is small
      uint32_t take[SPH];
#pragma unroll
      for (int i = 0; i < SPH; ++i) {
        int hl[2] = {0, 0}, hf[2] = {0, 0};
#pragma unroll
        for (int e = 0; e < CT; ++e) {
          const int j = CT * (g0 + i) + e;
          const bool ok = j < d;
          const int64_t hneg = ok ? -(int64_t)hg[ok ? j : 0] : 0;
          hl[e] = (int)(hneg & ((1 << BITS) - 1));
          hf[e] = (int)hneg;
        }
        hlp[i] = S::join(hl[0], hl[1]);
        hfp[i] = S::join(hf[0], hf[1]);
        take[i] = S::take(i, CT * (g0 + i) < d, CT * (g0 + i) + 1 < d);
      }
      // The rows of a window: its eight sample indices in two LDS reads (every entry that is read is a valid row, also
      // for windows past the end of the epoch, whose rows are never used),
      // then one multiply-add for the address and one load per step.
      const unsigned char* const frag = Xq + (g0 < U ? 2 * g0 : 0);  // lanes past the row re-read its first bytes
      auto request = [&](uint32_t (&dst)[kWin], int64_t win) {
        const int base = (int)((win * kWin) & kMask);
        const int4 i0 = *reinterpret_cast<const int4*>(&s_idx[base]);
        const int4 i1 = *reinterpret_cast<const int4*>(&s_idx[base + 4]);
        const int iv[kWin] = {i0.x, i0.y, i0.z, i0.w, i1.x, i1.y, i1.z, i1.w};
#pragma unroll
        for (int s = 0; s < kWin; ++s) {
          const unsigned char* at = frag + (uint64_t)(uint32_t)iv[s] * (uint32_t)row_bytes;
          if (row_bytes >> 32) at += (uint64_t)(uint32_t)iv[s] * (uint32_t)(row_bytes >> 32) << 32;  // uniform
          if (SPH == 1) dst[s] = (uint32_t) * reinterpret_cast<const uint16_t*>(at);
          else dst[s] = *reinterpret_cast<const uint32_t*>(at);
        }
      };
      uint32_t f[kSets][kWin];  // row fragments in flight: window v in set v % kSets
      U4 zn[SPH];  // rounding blocks of the window whose records are made next
      auto blocks = [&](int64_t win) {
#pragma unroll
        for (int i = 0; i < SPH; ++i) zn[i] = zround_block(seed, a.epoch, (uint32_t)(g0 + i), (uint32_t)win);
      };
      int* const rec = s_rec + QW * owner;
      constexpr int kStep = NQ * LANES * QW;  // dwords of a step's records
      // the records of a window into a slot of the ring
      auto make_window = [&](const uint32_t (&fr)[kWin], int slot) {
        int* const at = rec + slot * (kWin * kStep);
        int* const xw = at + (u0 / QW) * (QW * LANES) + u0 % QW;
        int* const cw = at + ((UPL + u0) / QW) * (QW * LANES) + (UPL + u0) % QW;
#pragma unroll
        for (int s = 0; s < kWin; ++s) {
#pragma unroll
          for (int i = 0; i < SPH; ++i)
            S::record(fr[s], i, take[i], pick(zn[i], (uint32_t)(s >> 1)), s, hlp[i], &xw[s * kStep + i], &cw[s * kStep + i]);
        }
      };
      __syncthreads();  // P0: the first batch is in place
      if (s_fold) {
#pragma unroll
        for (int i = 0; i < SPH; ++i) hlp[i] = hfp[i];
      }
#pragma unroll
      for (int v = 0; v < kSets; ++v) request(f[v], v);
      blocks(0);
      make_window(f[0], 0);
      request(f[0], kSets);
      blocks(1);
      make_window(f[1], 1);
      blocks(2);
      __syncthreads();  // P1: the records of windows 0 and 1 are in place
      // Period w: the rows of window w + 1 + kSets are requested into the set window w + 1 left, the
      // records of window w + 2 are made, then the blocks of window w + 3.  kSets periods per
      // trip, so that the fragment sets rotate by name.
      // (nothing may be scheduled across the borders of a period: left to itself the compiler
      // masks the fragments of all sets at the top of the loop, i.e. waits for every load)
      int slot = 2;
      auto period = [&](int64_t w, uint32_t (&freq)[kWin], const uint32_t (&fuse)[kWin]) {
        __builtin_amdgcn_sched_barrier(0);
        request(freq, w + 1 + kSets);
        __builtin_amdgcn_sched_barrier(0);
        make_window(fuse, slot);
        slot = (slot + 1) & (kSlots - 1);
        blocks(w + 3);
        __syncthreads();
        __builtin_amdgcn_sched_barrier(0);
      };
      int64_t w = 0;
      for (; w + kSets <= nwin; w += kSets) {
#pragma unroll
        for (int k = 0; k < kSets; ++k) period(w + k, f[(k + 1) % kSets], f[(k + 2) % kSets]);
      }
#pragma unroll
      for (int k = 0; k < kSets - 1; ++k)
        if (w + k < nwin) period(w + k, f[(k + 1) % kSets], f[(k + 2) % kSets]);
      __syncthreads();  // P2
      __syncthreads();  // the counters
    return;
  }

  if (wave != 0) {
    // ============================== idle wave ==============================
    __syncthreads();
    __syncthreads();
    for (int64_t w = 0; w < nwin; ++w) __syncthreads();
    __syncthreads();
    __syncthreads();
    return;
  }

  // ============================== chain wave ==============================
  int zp[UPL], hh[UPL];
  const bool hh_small = load_z(zp, hh);
  // The fused form stands for the fixed order of roundings while nothing underflows on the way.  `direct`: and
  // no partial sum of the matrix instruction is so large that its last place matters (|t| <= 2^22), so that it
  // may do the multiply-add too; else it adds up the whole number x^T z, and the multiply-add follows.
  const double k2 = __dmul_rn(aB, inv_s), k1 = __dmul_rn(dscale, k2);
  auto normal = [](double v) { return v > 1e-200 && v < 1e200; };
  const bool fused_ok = normal(dscale) && normal(aB) && normal(__dmul_rn(dscale, aB)) && normal(inv_s) && normal(k2) && normal(k1);
  const bool direct = LANES == 16 || k1 * (double)d * (double)(1 << (2 * BITS - 2)) < 0x1p22;
  const bool fold = __ballot(!hh_small) == 0;  // uniform
  if (lane == 0) s_fold = fold ? 1 : 0;
  __syncthreads();  // P0
  __syncthreads();  // P1: the records of windows 0 and 1 are in place
  __builtin_amdgcn_s_setprio(3);

  // what a step needs from LDS, requested kAhead steps ahead: its record and its step-indexed draws
  struct Step {
    RecV rec[NQ];
    double c, dl0;
    float phi, y;
    int ncl;
  };
  auto load_step = [&](Step& st, int slot, int base, int s) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < NQ; ++q) st.rec[q] = *rec_at(slot, s, q);
    st.c = s_c[base + s];
    if constexpr (REG) st.ncl = s_ncl[base + s];
    if constexpr (need_phi) st.phi = s_phi[base + s];
    if constexpr (logistic) {
      st.y = s_y[base + s];
      st.dl0 = s_dl0[base + s];
    }
  };
  constexpr int kAhead = logistic ? 1 : 2;  // (a step with exp in it is long enough for one, and needs the registers)
  Step ahead[kAhead];

  // x^T z of a step's row: the sum over the 16 lanes of a row of lanes; at 8 bits with fold x^T (2^8 z)
  auto fold16 = [](int v) {
    v += dpp_quad_swap1(v);
    v += dpp_quad_swap2(v);
    v += dpp_half_mirror(v);
    v += dpp_row_mirror(v);
    return v;
  };
  auto row_dot = [&](const int (&x)[UPL], auto fold_tag) __attribute__((always_inline)) -> double {
    if constexpr (BITS == 8) {
      int v;
      if constexpr (UPL == 2) {
        v = S::dot(x[1], zp[1], S::dot(x[0], zp[0]));
      } else {
        int p0 = S::dot(x[0], zp[0]), p1 = S::dot(x[1], zp[1]);
#pragma unroll
        for (int u = 2; u < UPL; u += 2) {
          p0 = S::dot(x[u], zp[u], p0);
          p1 = S::dot(x[u + 1], zp[u + 1], p1);
        }
        v = p0 + p1;
      }
      return (double)fold16(v);
    } else {
      // products, or sums of two less 2^16, fit 32 bits; each is cut into its low 16 bits and the rest, and the
      // two kinds are folded apart (the instructions of one fill the wait states of the other)
      int lo = 0, hi = 0;
      int z[UPL];
#pragma unroll
      for (int u = 0; u < UPL; ++u) z[u] = decltype(fold_tag)::value ? zp[u] >> 16 : zp[u];
      if constexpr (UPL == 1) {
        const int p = mad24(x[0], z[0], 0);
        lo = p & 0xFFFF;
        hi = p >> 16;
      } else {
        hi = UPL / 2;
#pragma unroll
        for (int u = 0; u < UPL; u += 2) {
          const int p = mad24(x[u], z[u], mad24(x[u + 1], z[u + 1], -65536));
          lo += p & 0xFFFF;
          hi += p >> 16;
        }
      }
      lo = fold16(lo);
      hi = fold16(hi);
      return __fma_rn((double)hi, 65536.0, (double)lo);
    }
  };
  auto scale_one = [](auto fold_tag) { return BITS == 8 && decltype(fold_tag)::value ? 0x1p-8 : 1.0; };
  // scale * (the sum of row_dot) + add
  auto whole_dot = [&](double row, double scale, double add) -> double {
    if (LANES == 16) return __fma_rn(row, scale, add);
    return __builtin_amdgcn_mfma_f64_4x4x4f64(row, scale, add, 0, 0, 0);
  };
  // l'(phi_i + x^T z) - l'(phi_i), in the fixed order
  auto moved = [&](double D, float phi_s, float y_s, double dl0_s) -> double {
    const double delta = __dmul_rn(dscale, D);
    if constexpr (logistic) {
      const double a1 = lp ? delta : __dadd_rn((double)phi_s, delta);
      return __dadd_rn(logistic_dl(a1, (double)y_s), -dl0_s);  // l'(phi_i) comes with the draws
    } else if constexpr (need_phi) {
      return __dadd_rn(delta, -(double)phi_s);
    } else {
      return delta;
    }
  };
  // A window in the fixed order of roundings, whatever it holds: `steps` of them, L2 draws among
  // them or not.  For windows in which a fused step came too close to an integer, the last, partial
  // window, and epochs whose scales the fused form does not cover.
  auto window_fixed = [&](int64_t t0, int slot, int part, int steps, auto fold_tag) __attribute__((always_inline)) {
    const int base = (int)(t0 & kMask);
#pragma unroll 1
    for (int s = 0; s < steps; ++s) {
      RecV r[NQ];
#pragma unroll
      for (int q = 0; q < NQ; ++q) r[q] = *rec_at(slot, s, q);
      int x[UPL], cr[UPL];
      split_record(r, x, cr);
      const double D = whole_dot(row_dot(x, fold_tag), scale_one(fold_tag), 0.0);
      const int k = base + s;
      const double diff = moved(D, kMargins ? s_phi[kMargins ? k : 0] : 0.f, logistic ? s_y[logistic ? k : 0] : 0.f,
                                logistic ? s_dl0[logistic ? k : 0] : 0.0);
      const double beta = __dmul_rn(aB, diff);
      const double rho = __dadd_rn(kDraw, -s_c[k]);  // exact
      const double fl = floor(__dadd_rn(__dmul_rn(beta, inv_s), rho));
      int nf;
      asm("v_cvt_i32_f64 %0, -%1" : "=v"(nf) : "v"(fl));  // saturates
      const int ng = min(max(nf, -QMAX), -QMIN);
      s_hi[part][s] = kMagicHi + min(max(nf, -(1 << 20)), 1 << 20);
      const int ncl = REG ? __builtin_amdgcn_readfirstlane((int)s_ncl[REG ? k : 0]) : 0;
#pragma unroll
      for (int u = 0; u < UPL; ++u)
        zp[u] = ncl == 0 ? step_strip(begin_strip(zp[u], hh[u], fold_tag), x[u], kMagicHi + ng, cr[u], fold_tag)
                         : step_strip_reg(zp[u], x[u], ng, ncl, cr[u], hh[u], fold_tag, nullptr);
    }
  };

  // A whole window of fused steps; false (and z as it was) where one of them came too close to an integer.
  auto window = [&](int64_t t0, int slot, int part, auto fold_tag, auto direct_tag) __attribute__((always_inline)) -> bool {
    const int base = (int)(t0 & kMask);
    const int next_base = (base + kWin) & kMask;  // (any window has its place in the ring, also past the end of the epoch)
    int zsave[UPL];
#pragma unroll
    for (int u = 0; u < UPL; ++u) zsave[u] = zp[u];
    uint32_t nearest = 0xFFFFFFFFu;  // the least of the window's low words
    int hi_even = 0;
    const int next_slot = (slot + 1) & (kSlots - 1);
#pragma unroll
    for (int s = 0; s < kWin; ++s) {
      const Step st = ahead[s % kAhead];
      int x[UPL], cr[UPL];
      split_record(st.rec, x, cr);
      constexpr bool DIRECT = decltype(direct_tag)::value && !need_phi;
      double t = DIRECT ? whole_dot(row_dot(x, fold_tag), -k1 * scale_one(fold_tag), st.c)
                        : whole_dot(row_dot(x, fold_tag), scale_one(fold_tag), 0.0);
      // (held in place: the scheduler would sink the reads to where their latency is not covered)
      __builtin_amdgcn_sched_barrier(0);
      if (s + kAhead < kWin) load_step(ahead[s % kAhead], slot, base, s + kAhead);
      else load_step(ahead[s % kAhead], next_slot, next_base, s + kAhead - kWin);
      if constexpr (REG) {
#pragma unroll
        for (int u = 0; u < UPL; ++u) cr[u] = with_draw(zp[u], st.ncl, cr[u], fold_tag);
      }
#pragma unroll
      for (int u = 0; u < UPL; ++u) zp[u] = begin_strip(zp[u], hh[u], fold_tag);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (need_phi) t = __fma_rn(moved(t, st.phi, st.y, st.dl0), -k2, st.c);
      else if constexpr (!DIRECT) t = __fma_rn(t, -k1, st.c);
      const uint64_t bits = __builtin_bit_cast(uint64_t, t);
      const int hi = (int)(bits >> 32);
      const uint32_t fr = (uint32_t)bits;
      nearest = fr < nearest ? fr : nearest;
      // monotone in t over the whole range of doubles, so the clamp of the word is the clamp of gamma
      const int g = min(max(hi, kMagicHi - QMAX), kMagicHi - QMIN);
      if (s & 1) *reinterpret_cast<int2r*>(&s_hi[part][s - 1]) = int2r{hi_even, hi};
      else hi_even = hi;
#pragma unroll
      for (int u = 0; u < UPL; ++u) zp[u] = step_strip(zp[u], x[u], g, cr[u], fold_tag);
    }
    if (__builtin_expect(__ballot(nearest <= 2 * kNear) != 0, 0)) {
#pragma unroll
      for (int u = 0; u < UPL; ++u) zp[u] = zsave[u];
      return false;
    }
    return true;
  };
  auto run = [&](auto fold_tag, auto direct_tag) __attribute__((always_inline)) {
    keep_z(zp, fold_tag);
    int slot = 0, part = 0;
    int64_t t0 = 0;
    auto next_window = [&]() {
      // window t0 / 8 is consumed, the records of the one after the next are in place; nothing of this wave
      // is waited for (what the service wave reads of it was stored a window ago: LDS answers in order, and
      // reads behind those stores have been used by now)
      asm volatile("s_barrier" ::: "memory");
      slot = (slot + 1) & (kSlots - 1);
      part = part == kHis - 1 ? 0 : part + 1;
      t0 += kWin;
    };
    const bool fused = fused_ok && (!REG || reg_small);
    while (t0 < T) {
      // Windows of fused steps, in a loop of their own: the registers that the steps' records arrive in are
      // carried round it, and a copy anywhere would wait for them
      if (fused) {
#pragma unroll
        for (int k = 0; k < kAhead; ++k) load_step(ahead[k], slot, (int)(t0 & kMask), k);
        while (t0 + kWin <= T && __builtin_expect(window(t0, slot, part, fold_tag, direct_tag), 1)) next_window();
        if (t0 >= T) break;
      }
      window_fixed(t0, slot, part, (int)(T - t0 < kWin ? T - t0 : kWin), fold_tag);
      next_window();
    }
    __syncthreads();  // P2: the last gammas are in place
    if constexpr (decltype(fold_tag)::value) {
#pragma unroll
      for (int u = 0; u < UPL; ++u) zp[u] = S::high(zp[u]);
    }
  };
  using Direct = std::bool_constant<!need_phi>;
  if (need_phi || direct) {
    if (fold) run(std::true_type{}, Direct{});
    else run(std::false_type{}, Direct{});
  } else {
    if (fold) run(std::true_type{}, std::false_type{});
    else run(std::false_type{}, std::false_type{});
  }

  // ---- w~ <- w~ + delta_m z (option I); hand z out
#pragma unroll
  for (int u = 0; u < UPL; ++u)
#pragma unroll
    for (int e = 0; e < CT; ++e) {
      const int j = CT * strip_of<UPL, LANES>(u, lane) + e;
      if (lane < LANES && j < d) {
        const int zk = S::value(zp[u], e);
        zg[j] = (ZT)zk;
        const double step = __dmul_rn(delta_m, (double)zk);
        wg[j] = lp ? (float)step : (float)__dadd_rn((double)wg[j], step);  // Alg. 2: w~ = delta w
      }
    }
  __syncthreads();  // the counters
  if (tid < 4) cnt_out[tid] = tid < 3 ? s_cnt[tid] : 0ull;
}

// the record ring: windows of 8 steps, 8 UPL bytes per lane and step
constexpr size_t ring_bytes(int upl, int lanes) { return (size_t)kSlots * kWin * upl * 8 * lanes; }

template <int BITS, int UPL, int LANES, bool PAIR, bool REG>
int launch_one(const InArgs& a, int R, hipStream_t s) {
  const dim3 grid(R), block(64 * waves_of(UPL, LANES));
#define HALP_LONE(LOSS_)                                                                          \
  do {                                                                                            \
    auto kern = inner_reg_lone_kernel<BITS, LOSS_, UPL, LANES, PAIR, REG>;                        \
    const size_t smem = ring_bytes(UPL, LANES);                                     \
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern),                                  \
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem) != hipSuccess) \
      return HALP_ERR_HIP;                                                                        \
    hipLaunchKernelGGL(kern, grid, block, smem, s, a);                                            \
  } while (0)
  if (a.loss == HALP_LOSS_SQUARED && a.lp) HALP_LONE(kLossSquaredWithMargins);
  else if (a.loss == HALP_LOSS_SQUARED) HALP_LONE(HALP_LOSS_SQUARED);
  else HALP_LONE(HALP_LOSS_LOGISTIC);
#undef HALP_LONE
  return hip_ok(hipGetLastError());
}

template <int BITS, bool REG>
int launch_shape(const InArgs& a, int upl, int lanes, int R, bool pair, hipStream_t s) {
  if constexpr (BITS == 8) {
    if (upl == 2 && lanes == 16) return launch_one<8, 2, 16, true, REG>(a, R, s);
  } else {
    if (upl == 1) return launch_one<16, 1, 64, true, REG>(a, R, s);
  }
  if (upl == 2) return pair ? launch_one<BITS, 2, 64, true, REG>(a, R, s) : launch_one<BITS, 2, 64, false, REG>(a, R, s);
  if (upl == 4) return pair ? launch_one<BITS, 4, 64, true, REG>(a, R, s) : launch_one<BITS, 4, 64, false, REG>(a, R, s);
  if (upl == 8) return launch_one<BITS, 8, 64, false, REG>(a, R, s);
  return HALP_ERR_UNSUPPORTED;
}

}  // namespace innerlone
}  // namespace halp
