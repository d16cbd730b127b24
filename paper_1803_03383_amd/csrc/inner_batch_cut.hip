// Inner loop of Algorithm 4 (LM-HALP) with a minibatch of B rows per step (K = 1, 2 <= B <= 128), full-step form:
// the rows of a step are dealt to waves and stay in registers.
//
// A workgroup holds one slice of S = 64 CPT coordinates, a chain P of them on P CUs.  Row wave w takes kRows
// consecutive rows of every step (2, 4, 8 or 16 by B, so that up to 8 waves share them): their fragments (NDW dwords per
// lane) are requested two steps ahead, in three register sets that trade places, and serve both passes.  One more
// wave, the service wave, takes the step's scalars, one row (two) per lane.  z, h~ and the rounding words of z live in LDS,
// one coordinate per thread in the update.  A step:
//   row waves     z from LDS, packed dots of the wave's rows with it (v_dot4 at 8 bits; at 16 bits v_dot2 against
//                 a low and a high part of z, so that 32-bit sums stay exact), all wave sums at once      | barrier
//   service wave  adds the workgroup's B partial dots to the rows' 64-bit words in device memory, one device-scope
//                 atomic instruction, waits (bounded) until every word has counted P additions, gammas into LDS
//   row waves     meanwhile request the rows two steps on, and draw: sample indices and rounding words of gamma,
//                 256 of either at a time, rounding words of z for the next eight steps                   | barrier
//   row waves     sum_m gamma_m x_m over the wave's rows into LDS                                         | barrier
//                 sums over the waves, rounding of z, one coordinate per thread                           | barrier
//
// The P partial dots of a row meet in one word per row, double-buffered by step parity: the share in the low 56 bits,
// a 1 in the top byte per addition; both fields are differences modulo 2^64, so nothing is reset.  A word is used
// again only after every workgroup of the chain has read it: its next addition follows this step's gamma, hence
// everyone's share of the step after.
//
// What bounds it: latency.  At 4096 x 16 bits, B = 64 a step takes 2.5 us: the exchange ~1.0, the scalars
// ~0.35, the passes over 8 rows per wave, four barriers.  Rows requested behind gamma instead of beside the exchange: 0.3 us
// more; requested three to five steps ahead: the same.  All parts of a chain on one XCD: 4096 x 8 bits 0.13 us less, 4096 x
// 16 bits at 8 GB of rows 0.7 us more, the others the same: not done.
// The form before had four waves of 16 rows with a copy of z each, all draws and updates repeated in every wave.  us per
// step of the loop (without the gradient pass; logistic), that form -> this one: 4096 x 16 bits B = 64 N = 10^6 4.55 -> 2.60, N = 200 000
// 4.20 -> 2.53, 4096 x 8 bits 3.54 -> 1.99, 1024 x 16 bits 4.25 -> 2.18, 512 x 8 bits B = 16 3.14 -> 1.36, 128 x 8 bits B = 4 3.57
// -> 0.98; small steps of several slices, on one workgroup before, 1024 x 8 bits B = 4 3.70 -> 1.36; 128 rows, on the kernels of the
// matrix cores and of class waves or on the general kernel before: 1000 x 8 bits 6.5 -> 2.4, 1024 x 16 bits 95 -> 3.2, 4096 x
// 8 bits 207 -> 2.6.
#include <algorithm>

#include "inner_batch.hpp"

namespace halp {
namespace {

constexpr int kRowWaves = 8;    // row waves at most
constexpr int kLeastWaves = 4;  // beside the service wave: fewer would take the update and the draws in turn
constexpr int kRing = 1024;     // words drawn ahead: sample indices, rounding words of gamma
constexpr int kDraw = 256;      // words of one wave's Philox evaluation

template <int BITS, int NDW, int kRows>
__global__ __launch_bounds__(64 * (kRowWaves + 1)) void inner_batch_cut_kernel(InArgs a, void* zout, int nrw, int P,
                                                                               unsigned long long* xbuf,
                                                                               int spin_limit, int poll_delay) {
  using XT = typename std::conditional<BITS == 8, int8_t, int16_t>::type;
  using HT = typename std::conditional<BITS == 8, int16_t, int32_t>::type;
  constexpr int EPD = 32 / BITS;       // elements per dword
  constexpr int CPT = NDW * EPD;       // coordinates per lane of a fragment
  constexpr int S = 64 * CPT;          // coordinates of the slice
  constexpr int CT = 16 / BITS;        // coordinates per strip of 16 rounding bits
  constexpr int kStrips = S / CT;
  constexpr int HB = kRows == 16 ? 2 : 1;  // rows of a step per lane of the service wave: lane, lane + 64
  constexpr int NV = BITS == 16 ? 2 : 1;  // partial sums of gamma x: low and high byte of gamma apart at 16 bits
  constexpr int QMAX = (1 << (BITS - 1)) - 1, QMIN = -(1 << (BITS - 1));
  constexpr int kGroups = kRows == 2 ? kLeastWaves : kRowWaves;  // waves that may hold rows
  constexpr int kSets = 3;  // register sets: the rows of a step are requested kSets - 1 steps ahead
  static_assert(kStrips <= 8 * 64);    // one draw per step fills the next window
  const int chain = (int)blockIdx.x / P;
  const int part = (int)blockIdx.x - chain * P;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int d = a.d, B = a.B;
  const uint64_t seed = a.seed + (uint64_t)chain;
  const int64_t T = epoch_steps(seed, a.epoch, a.T, a.option2);
  const double* sc = a.scales + (int64_t)chain * 8;
  uint64_t* cnt_out = a.counters + (int64_t)chain * 4;
  if (sc[7] != 0.0) {
    if (tid < 4) cnt_out[tid] = 0;
    return;
  }

  __shared__ __attribute__((aligned(16))) int s_idx[kRing];
  __shared__ __attribute__((aligned(16))) uint32_t s_rw[kRing];
  __shared__ int s_part[NV][64 * HB];                                 // partial dots with the parts of z
  __shared__ __attribute__((aligned(16))) uint32_t s_gam[NV][32 * HB];  // gammas: pairs (low, high bytes), or four bytes
  __shared__ __attribute__((aligned(16))) int s_acc[kGroups][NV][S];
  __shared__ int s_z[S], s_h[S];
  __shared__ __attribute__((aligned(16))) uint32_t s_zp[NV][S / EPD];  // z packed for the dots
  __shared__ uint32_t s_zr[2][4][kStrips];
  __shared__ int s_cl;
  __shared__ unsigned long long s_cnt[3];
  if (tid < 3) s_cnt[tid] = 0;
  const bool use_reg = a.lambda > 0;
  const bool lp = a.lp != 0;
  const uint32_t N = (uint32_t)a.N;
  unsigned int n_timeout = spin_limit < 0 ? 1u : 0u;  // below 0: never wait

  // 256 words of a stream from word n0, a multiple of 4
  auto draw_indices = [&](int64_t n0) {
    const U4 r = stream_block(seed, kIdx, a.epoch, (uint64_t)(n0 >> 2) + (uint64_t)lane);
    const uint4 v = make_uint4(__umulhi(r.x, N), __umulhi(r.y, N), __umulhi(r.z, N), __umulhi(r.w, N));
    *reinterpret_cast<uint4*>(&s_idx[(n0 + 4 * lane) & (kRing - 1)]) = v;
  };
  auto draw_gamma_words = [&](int64_t n0) {
    const U4 r = stream_block(seed, kGamma, a.epoch, (uint64_t)(n0 >> 2) + (uint64_t)lane);
    *reinterpret_cast<uint4*>(&s_rw[(n0 + 4 * lane) & (kRing - 1)]) = make_uint4(r.x, r.y, r.z, r.w);
  };
  auto draw_zround = [&](int e, int64_t win) {  // strips 64 e .. 64 e + 63 of the slice
    const int st = 64 * e + lane;
    const U4 r = zround_block(seed, a.epoch, (uint32_t)(part * kStrips + st), (uint32_t)win);
    uint32_t(&to)[4][kStrips] = s_zr[win & 1];
    to[0][st] = r.x; to[1][st] = r.y; to[2][st] = r.z; to[3][st] = r.w;
  };
  auto pack_z = [&](int c, int z) {
    if (BITS == 8) {
      reinterpret_cast<int8_t*>(s_zp[0])[c] = (int8_t)z;
    } else {
      // z = 256 zh + zl with zl in [-128, 127]: both parts at most 128 in magnitude, so a wave's sum
      // of 512 products with |x| <= 32767 stays below 2^31
      const int zh = (z + 128) >> 8;
      reinterpret_cast<int16_t*>(s_zp[0])[c] = (int16_t)(z - 256 * zh);
      reinterpret_cast<int16_t*>(s_zp[NV - 1])[c] = (int16_t)zh;
    }
  };

  // ---- set-up: the first words of every stream, z and h~ of the slice
  const int nthreads = 64 * (nrw + 1);
  int64_t drawn = 2 * kDraw;  // words of a ring drawn so far, kept by the wave that draws them
  if (wave < 2) {
    draw_indices(wave * kDraw);
    draw_gamma_words(wave * kDraw);
  }
  for (int e = wave; e < kStrips / 64; e += nrw + 1) draw_zround(e, 0);
  for (int c = tid; c < S; c += nthreads) {
    const int j = part * S + c;
    const int zj = j < d ? (int)reinterpret_cast<const XT*>(a.z)[(int64_t)chain * d + j] : 0;
    s_z[c] = zj;
    s_h[c] = j < d ? (int)reinterpret_cast<const HT*>(a.h)[(int64_t)chain * d + j] : 0;
    pack_z(c, zj);
  }
  for (int c = tid; c < kGroups * NV * S; c += nthreads) (&s_acc[0][0][0])[c] = 0;
  __syncthreads();

  if (wave == nrw) {
    // ===================================================================== service wave
    __builtin_amdgcn_s_setprio(3);
    const float* __restrict__ phi = a.phi + (int64_t)chain * a.N;
    const float* __restrict__ y = reinterpret_cast<const float*>(a.y) + (int64_t)chain * a.y_chain_stride;
    const double inv_s = sc[5];
    const double dscale = __dmul_rn(a.delta_d, sc[0]);
    const double alpha = a.hyper[2 * chain];
    const double aB = __ddiv_rn(alpha, (double)B);
    const double al = __dmul_rn(alpha, a.lambda);
    const bool logistic = a.loss == HALP_LOSS_LOGISTIC;
    const bool need_phi = a.loss != HALP_LOSS_SQUARED || lp;
    unsigned int n_gclamp[HB] = {}, n_reg = 0;
    unsigned long long* words = xbuf + (int64_t)chain * 2 * kCutMaxB;
    int cl64 = 0;  // lane l: the L2 draw of step 64 k + l
    // margins and labels, of even steps and of odd ones, gathered two steps ahead
    float phi_v[2][HB] = {}, y_v[2][HB] = {};
    unsigned long long prev[2][HB] = {};  // the words at their last use
    bool row[HB];
    int at[HB];  // this lane's rows, lanes past B the last one
#pragma unroll
    for (int u = 0; u < HB; ++u) {
      row[u] = lane + 64 * u < B;
      at[u] = min(lane + 64 * u, B - 1);
    }
    auto ring = [&](int64_t t, int u) { return ((uint32_t)t * (uint32_t)B + (uint32_t)at[u]) & (kRing - 1); };
    auto gather = [&](int q, int64_t t) {
#pragma unroll
      for (int u = 0; u < HB; ++u) {
        const int i = s_idx[ring(t, u)];
        if (need_phi) phi_v[q][u] = phi[i];
        if (logistic) y_v[q][u] = y[i];
      }
    };
    gather(0, 0);
    gather(1, 1);
    auto one_step = [&](int64_t t, int q) __attribute__((always_inline)) {
      // beside the row waves' update and dots
      if (use_reg && (t & 63) == 0) {
        const uint64_t n = (uint64_t)t + (uint64_t)lane;
        const uint32_t w = pick(stream_block(seed, kReg, a.epoch, n >> 2), (uint32_t)(n & 3));
        cl64 = (int)quantize_real(al, (double)(1 << BITS), w, 0.0, (double)QMAX, nullptr);
      }
      const int cl = use_reg ? __builtin_amdgcn_readlane(cl64, (int)(t & 63)) : 0;
      n_reg += (lane == 0 && cl != 0) ? 1u : 0u;
      double rho[HB], a0[HB], yi[HB], dl0[HB];
#pragma unroll
      for (int u = 0; u < HB; ++u) {
        rho[u] = __dmul_rn((double)s_rw[ring(t, u)], 0x1p-32);
        a0[u] = (double)phi_v[q][u];
        yi[u] = (double)y_v[q][u];
        dl0[u] = 0.0;
        if (logistic) dl0[u] = logistic_dl(a0[u], yi[u]);
        asm volatile("" : "+v"(rho[u]), "+v"(dl0[u]));  // stay where they are written
      }
      if (lane == 0) s_cl = cl;
      lds_barrier();  // the partial dots of this step are in LDS
      long long D[HB];
#pragma unroll
      for (int u = 0; u < HB; ++u) {
        D[u] = s_part[0][at[u]];
        if (BITS == 16) D[u] += (long long)s_part[NV - 1][at[u]] * 256;
      }
      if (P > 1) {
        unsigned long long* w = words + q * kCutMaxB + lane;
        unsigned long long v[HB];
#pragma unroll
        for (int u = 0; u < HB; ++u) {
          v[u] = prev[q][u];
          if (row[u])
            __hip_atomic_fetch_add(w + 64 * u, (1ull << 56) + (unsigned long long)D[u], __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
        }
        // polls that start before the additions can be back only add traffic
        if (n_timeout == 0) {
          for (int i = 0; i < poll_delay; ++i) __builtin_amdgcn_s_sleep(4);
        }
        for (int spin = 0; n_timeout == 0; ++spin) {  // after one wait ran out, none is tried again
          bool missing = false;
#pragma unroll
          for (int u = 0; u < HB; ++u)
            if (row[u]) v[u] = __hip_atomic_load(w + 64 * u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          // a signed sum below 2^55 in magnitude may borrow from the top byte
#pragma unroll
          for (int u = 0; u < HB; ++u)
            missing |= row[u] && (uint32_t)((v[u] - prev[q][u] + (1ull << 55)) >> 56) != (uint32_t)P;
          if (__ballot(missing) == 0) break;
          if (spin >= spin_limit) n_timeout = 1;  // only if a workgroup of the chain never ran: give up
        }
#pragma unroll
        for (int u = 0; u < HB; ++u) {
          if (n_timeout == 0) D[u] = (long long)(v[u] - prev[q][u] - ((unsigned long long)P << 56));
          prev[q][u] = v[u];
        }
      }
#pragma unroll
      for (int u = 0; u < HB; ++u) {
        // beta_m = (alpha / B) (l'(phi_m + x_m^T z) - l'(phi_m)), gamma_m = Q_(delta_s, b)(beta_m)
        const double delta = __dmul_rn(dscale, (double)D[u]);
        double diff;
        if (logistic) {
          const double a1 = lp ? delta : __dadd_rn(a0[u], delta);
          diff = __dadd_rn(logistic_dl(a1, yi[u]), -dl0[u]);
        } else {
          diff = lp ? __dadd_rn(delta, -a0[u]) : delta;
        }
        const double beta = __dmul_rn(aB, diff);
        const double fq = floor(__dadd_rn(__dmul_rn(beta, inv_s), rho[u]));
        const double fc = fmin(fmax(fq, (double)QMIN), (double)QMAX);
        const int g = row[u] ? (int)fc : 0;
        n_gclamp[u] += (row[u] && fq != fc) ? 1u : 0u;
        if (BITS == 16) {  // pairs of rows: low bytes without sign, high bytes with it
          const int gn = dpp_quad_swap1(g);
          if ((lane & 1) == 0) {
            s_gam[0][32 * u + (lane >> 1)] = (uint32_t)(g & 0xFF) | ((uint32_t)(gn & 0xFF) << 16);
            s_gam[NV - 1][32 * u + (lane >> 1)] = (uint32_t)((g >> 8) & 0xFFFF) | ((uint32_t)(gn >> 8) << 16);
          }
        } else {  // four rows
          const int two = (g & 0xFF) | ((dpp_quad_swap1(g) & 0xFF) << 8);
          const int four = (two & 0xFFFF) | (dpp_quad_swap2(two) << 16);
          if ((lane & 3) == 0) s_gam[0][16 * u + (lane >> 2)] = (uint32_t)four;
        }
      }
      lds_barrier();  // gamma is out
      gather(q, t + 2);
      lds_barrier();  // the waves' sums are in LDS
      lds_barrier();  // z is
    };
    int64_t t = 0;
    for (; t + 1 < T; t += 2) {
      one_step(t, 0);
      one_step(t + 1, 1);
    }
    if (t < T) one_step(t, 0);
#pragma unroll
    for (int u = 0; u < HB; ++u)
      if (n_gclamp[u]) atomicAdd(&s_cnt[1], (unsigned long long)n_gclamp[u]);
    if (n_reg) atomicAdd(&s_cnt[2], (unsigned long long)n_reg);
  } else {
    // ========================================================================== row wave
    const unsigned char* __restrict__ Xq = reinterpret_cast<const unsigned char*>(a.Xq) +
                                           (int64_t)chain * a.xq_chain_stride * (BITS / 8);
    const int64_t row_bytes = a.ldxq * (BITS / 8);
    // Rows are padded to whole 8-byte groups; a 16-byte fragment is only used when rows are 16-byte multiples
    // (checked on the host), so a fragment that starts below d lies inside the row.  Lanes past the row re-read
    // its first fragment; their z is 0 and stays 0.
    const int j0 = part * S + lane * CPT;
    const int frag_off = j0 < d ? j0 * (BITS / 8) : 0;
    const int row0 = wave * kRows;
    const bool has_rows = row0 < B;  // the last of the least waves may hold none
    const int idx_wave = nrw - 1, gam_wave = nrw - 2, zr_wave = nrw - 3;
    int64_t drawn_g = drawn;
    unsigned long long n_zclamp = 0;
    uint32_t x[kSets][kRows][NDW];
    auto load_step = [&](uint32_t (&dst)[kRows][NDW], int64_t t) {
      // lane r fetches the index of the wave's row r (one LDS read for all); rows past B repeat the last one
      const int mine = s_idx[((uint32_t)t * (uint32_t)B + (uint32_t)min(row0 + (lane & (kRows - 1)), B - 1)) & (kRing - 1)];
#pragma unroll
      for (int r = 0; r < kRows; ++r) {
        const unsigned char* rp = Xq + (int64_t)__builtin_amdgcn_readlane(mine, r) * row_bytes + frag_off;
        if constexpr (NDW == 1) {
          dst[r][0] = *reinterpret_cast<const uint32_t*>(rp);
        } else if constexpr (NDW == 2) {
          const uint2 v = *reinterpret_cast<const uint2*>(rp);
          dst[r][0] = v.x; dst[r][1] = v.y;
        } else {
          const uint4 v = *reinterpret_cast<const uint4*>(rp);
          dst[r][0] = v.x; dst[r][1] = v.y; dst[r][2] = v.z; dst[r][3] = v.w;
        }
      }
    };
#pragma unroll
    for (int u = 0; u < kSets - 1; ++u)
      if (has_rows) load_step(x[u], u);

    auto one_step = [&](int64_t t, uint32_t (&cur)[kRows][NDW], uint32_t (&nxt)[kRows][NDW]) __attribute__((always_inline)) {
      // ---- pass 1: dots
      if (has_rows) {
        uint32_t zp[NV][NDW];
#pragma unroll
        for (int v = 0; v < NV; ++v)
#pragma unroll
          for (int q = 0; q < NDW; ++q) zp[v][q] = s_zp[v][lane * NDW + q];
        int dot[NV][kRows];
#pragma unroll
        for (int r = 0; r < kRows; ++r)
#pragma unroll
          for (int v = 0; v < NV; ++v) {
            dot[v][r] = 0;
#pragma unroll
            for (int q = 0; q < NDW; ++q)
              dot[v][r] = BITS == 8 ? __builtin_amdgcn_sdot4((int)cur[r][q], (int)zp[v][q], dot[v][r], false)
                                    : __builtin_amdgcn_sdot2(__builtin_bit_cast(short2v, cur[r][q]),
                                                             __builtin_bit_cast(short2v, zp[v][q]), dot[v][r], false);
          }
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          if constexpr (kRows == 16) {
            int half[2][8];
#pragma unroll
            for (int r = 0; r < 16; ++r) half[r / 8][r % 8] = dot[v][r];
            const int s0 = wave_sums8_i32(half[0], lane), s1 = wave_sums8_i32(half[1], lane);
            if (lane < 16) s_part[v][row0 + lane] = lane < 8 ? s0 : s1;
          } else {
            const int sum = wave_sums_i32(dot[v], lane);  // row row0 + lane % kRows
            if (lane < kRows) s_part[v][row0 + lane] = sum;
          }
        }
      }
      lds_barrier();  // the partial dots of this step are in LDS
      // ---- beside the exchange: the rows two steps on, and draws
      if (has_rows) load_step(nxt, t + kSets - 1);
      if (wave == idx_wave && (t + kSets + 1) * B > drawn) {
        draw_indices(drawn);
        drawn += kDraw;
      }
      if (wave == gam_wave && (t + 2) * B > drawn_g) {
        draw_gamma_words(drawn_g);
        drawn_g += kDraw;
      }
      if (wave == zr_wave && (int)(t & 7) < kStrips / 64) draw_zround((int)(t & 7), (t >> 3) + 1);
      lds_barrier();  // gamma is out
      // ---- pass 2: sum_m gamma_m x_m over the wave's rows, per coordinate
      if (has_rows) {
        int acc[NV][CPT];
#pragma unroll
        for (int v = 0; v < NV; ++v)
#pragma unroll
          for (int k = 0; k < CPT; ++k) acc[v][k] = 0;
        if constexpr (BITS == 16) {
          // Two rows at a time: v_perm puts a coordinate of both rows into one register, one v_dot2 against the
          // pair of gammas then serves both.  gamma = 256 gh + gl with gl in [0, 255]: 128 products of
          // each part stay below 2^31.
          uint32_t gl[kRows / 2], gh[kRows / 2];
#pragma unroll
          for (int r = 0; r < kRows / 2; ++r) {
            gl[r] = s_gam[0][row0 / 2 + r];
            gh[r] = s_gam[NV - 1][row0 / 2 + r];
          }
#pragma unroll
          for (int r = 0; r < kRows; r += 2) {
            const short2v gl2 = __builtin_bit_cast(short2v, gl[r / 2]), gh2 = __builtin_bit_cast(short2v, gh[r / 2]);
#pragma unroll
            for (int q = 0; q < NDW; ++q) {
              const short2v pe = __builtin_bit_cast(short2v, __builtin_amdgcn_perm(cur[r + 1][q], cur[r][q], 0x05040100u));
              const short2v po = __builtin_bit_cast(short2v, __builtin_amdgcn_perm(cur[r + 1][q], cur[r][q], 0x07060302u));
              acc[0][2 * q] = __builtin_amdgcn_sdot2(pe, gl2, acc[0][2 * q], false);
              acc[NV - 1][2 * q] = __builtin_amdgcn_sdot2(pe, gh2, acc[NV - 1][2 * q], false);
              acc[0][2 * q + 1] = __builtin_amdgcn_sdot2(po, gl2, acc[0][2 * q + 1], false);
              acc[NV - 1][2 * q + 1] = __builtin_amdgcn_sdot2(po, gh2, acc[NV - 1][2 * q + 1], false);
            }
          }
        } else {
          // four rows at a time (two, beside two bytes of zero): a coordinate's bytes in one register, one v_dot4
          // against the gammas
          constexpr int kGroup = kRows < 4 ? kRows : 4;
          uint32_t g4[kRows / kGroup];
#pragma unroll
          for (int r = 0; r < kRows / kGroup; ++r) g4[r] = s_gam[0][row0 / 4 + r] >> (8 * (row0 & 3));
#pragma unroll
          for (int r = 0; r < kRows; r += kGroup) {
            const int gr = (int)g4[r / kGroup];
#pragma unroll
            for (int q = 0; q < NDW; ++q) {
              const uint32_t lo01 = __builtin_amdgcn_perm(cur[r + 1][q], cur[r][q], 0x05010400u);
              const uint32_t hi01 = __builtin_amdgcn_perm(cur[r + 1][q], cur[r][q], 0x07030602u);
              uint32_t lo23 = 0, hi23 = 0;
              if constexpr (kGroup == 4) {
                lo23 = __builtin_amdgcn_perm(cur[(r + 3) % kRows][q], cur[(r + 2) % kRows][q], 0x05010400u);
                hi23 = __builtin_amdgcn_perm(cur[(r + 3) % kRows][q], cur[(r + 2) % kRows][q], 0x07030602u);
              }
              auto add = [&](int k, uint32_t b23, uint32_t b01, uint32_t sel) {
                acc[0][k % CPT] = __builtin_amdgcn_sdot4((int)__builtin_amdgcn_perm(b23, b01, sel), gr, acc[0][k % CPT], false);
              };
              add(4 * q, lo23, lo01, 0x05040100u);
              add(4 * q + 1, lo23, lo01, 0x07060302u);
              add(4 * q + 2, hi23, hi01, 0x05040100u);
              add(4 * q + 3, hi23, hi01, 0x07060302u);
            }
          }
        }
#pragma unroll
        for (int v = 0; v < NV; ++v)
#pragma unroll
          for (int k = 0; k < CPT; k += 4)
            *reinterpret_cast<int4*>(&s_acc[wave][v][lane * CPT + k]) =
                make_int4(acc[v][k], acc[v][k + 1], acc[v][k + 2], acc[v][k + 3]);
      }
      lds_barrier();  // every wave's sums are in LDS
      // ---- u = z - sum gamma x - h~ - c_lambda z in (delta_i, 2b); z = Q_(delta_m, b)(u)
      for (int c = tid; c < S; c += 64 * nrw) {
        int sum[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          sum[v] = 0;
#pragma unroll
          for (int g = 0; g < kGroups; ++g) sum[v] += s_acc[g][v][c];  // zero where a wave holds no rows
        }
        const int z = s_z[c], cl = s_cl;
        const uint32_t field = s_zr[(t >> 3) & 1][(t & 7) >> 1][c / CT] >> (16u * (uint32_t)(t & 1));
        const long long re = (long long)((field >> ((c % CT) * BITS)) & ((1u << BITS) - 1u));
        const long long gsum = (long long)sum[0] + (BITS == 16 ? (long long)sum[NV - 1] * 256 : 0);
        const long long v = -(long long)s_h[c] - (long long)cl * (long long)z - gsum;
        const long long zu = (long long)z + ((v + re) >> BITS);
        const long long zc = zu > QMAX ? QMAX : (zu < QMIN ? QMIN : zu);
        if (part * S + c < d) {
          n_zclamp += zu != zc ? 1 : 0;
          s_z[c] = (int)zc;
          pack_z(c, (int)zc);
        }
      }
      lds_barrier();  // z is in LDS
    };
    for (int64_t t0 = 0; t0 < T; t0 += kSets) {
#pragma unroll
      for (int u = 0; u < kSets; ++u)
        if (t0 + u < T) one_step(t0 + u, x[u], x[(u + kSets - 1) % kSets]);
    }
    if (n_zclamp) atomicAdd(&s_cnt[0], n_zclamp);
  }
  __syncthreads();

  // ---- w~ <- w~ + delta_m z (option I; Algorithm 2: w~ = delta z); hand z out
  const double delta_m = sc[0];
  for (int c = tid; c < S; c += nthreads) {
    const int j = part * S + c;
    if (j >= d) continue;
    reinterpret_cast<XT*>(zout)[(int64_t)chain * d + j] = (XT)s_z[c];
    if (P == 1) {  // several workgroups per chain: split_finish applies the offset
      float* wj = a.w + (int64_t)chain * d + j;
      const double step = __dmul_rn(delta_m, (double)s_z[c]);
      *wj = lp ? (float)step : (float)__dadd_rn((double)*wj, step);
    }
  }
  if (P == 1) {
    if (tid < 4) cnt_out[tid] = tid < 3 ? s_cnt[tid] : 0ull;
  } else {
    // counters were cleared before the launch: clamped coordinates add up over the parts, the scalar counts are
    // the same in every part, a wait that ran out is flagged in the last word
    if (tid == 0 && s_cnt[0]) atomicAdd(reinterpret_cast<unsigned long long*>(&cnt_out[0]), s_cnt[0]);
    if (part == 0 && (tid == 1 || tid == 2)) cnt_out[tid] = s_cnt[tid];
    if (tid == 64 * nrw && n_timeout) atomicMax(reinterpret_cast<unsigned long long*>(&cnt_out[3]), 1ull);
  }
}

}  // namespace

// Rows per wave: as many waves as there can be, and no fewer rows than two to a wave.
int rows_per_wave(int B) { return B <= 8 ? 2 : (B <= 32 ? 4 : (B <= 64 ? 8 : 16)); }

bool inner_batch_cut_takes(int B, int ndw) {
  // sixteen rows of sixteen bytes per lane: two register sets of them would spill
  return B <= kCutMaxB && !(rows_per_wave(B) == 16 && ndw == 4);
}

size_t inner_batch_cut_workspace(const halp_params& p) {
  return sizeof(long long) * 2 * kCutMaxB * (size_t)p.R + (size_t)p.R * p.d * (p.b / 8);
}

// A wait that runs out (other work may hold the CUs) costs time only: z goes to the workspace, and the general kernel takes the chains of such waits from the z they came with.
int launch_inner_batch_cut(const halp_handle& h, const InArgs& a, int ndw, int P, hipStream_t s) {
  const halp_params& p = h.p;
  const int rows = rows_per_wave(p.B);
  const int nrw = std::max((p.B + rows - 1) / rows, kLeastWaves);
  const dim3 grid(p.R * P), block(64 * (nrw + 1));
  unsigned long long* xbuf = reinterpret_cast<unsigned long long*>(h.batch_xbuf);
  const int nwords = p.R * 2 * kCutMaxB;
  const bool report = h.spin_limit < 0;  // waits switched off: their outcome is what is asked for
  void* zout = P > 1 ? static_cast<void*>(xbuf + nwords) : a.z;
  if (P > 1) launch_split_prepare(h.batch_xbuf, nwords, h.buf.counters, p.R * 4, s);
#define HALP_BC(BITS_, NDW_, ROWS_)                                                                                   \
  if (p.b == BITS_ && ndw == NDW_ && rows == ROWS_)                                                                   \
    hipLaunchKernelGGL((inner_batch_cut_kernel<BITS_, NDW_, ROWS_>), grid, block, 0, s, a, zout, nrw, P, xbuf,         \
                       h.spin_limit, h.poll_delay);                                                                   \
  else
#define HALP_BC_ROWS(BITS_, NDW_) HALP_BC(BITS_, NDW_, 2) HALP_BC(BITS_, NDW_, 4) HALP_BC(BITS_, NDW_, 8)
  HALP_BC_ROWS(8, 1) HALP_BC_ROWS(8, 2) HALP_BC_ROWS(16, 2) HALP_BC_ROWS(16, 4)
  HALP_BC(8, 1, 16) HALP_BC(8, 2, 16) HALP_BC(16, 2, 16) return HALP_ERR_UNSUPPORTED;
#undef HALP_BC_ROWS
#undef HALP_BC
  int rc = hip_ok(hipGetLastError());
  if (rc != HALP_OK || P == 1) return rc;
  rc = launch_split_finish(a, h.buf.scales, zout, 0, p.R, report, p.b, s);
  return rc != HALP_OK || report ? rc : launch_inner_generic(h, a.epoch, TraceBufs{}, s, true);
}

}  // namespace halp
