// Inner loop of Algorithm 4 (LM-HALP) with a minibatch of B rows per step (K = 1):
// all rows of a step see the same z, each has its own gamma, z is quantized once per step.
//
// One workgroup per chain, its waves side by side along the row; or P workgroups per chain, each holding a
// slice of the coordinates (only where HALP_OPT_INNER_PARTS asks for it).  The P partial dots of a row
// then meet in global memory once per step: every workgroup adds its 64 partial sums, with one device-scope atomic
// each, to the rows' words, which also count the additions, waits (bounded) until all P are there and goes on
// alone; the update needs nothing from the others.
//
// A thread owns the coordinates of one 4/8/16-byte fragment of a row (CPT of them)
// with z, h~ and the window's Philox words in registers.  A step:
//   pass 1   per row: packed integer dot of the fragment with z (v_dot4 at 8 bits; at 16
//            bits v_dot2 against a low and a high part of z separately, so that
//            32-bit sums stay exact), eight wave sums at a time, one LDS slot per row | barrier
//   scalars  wave 0, one row per lane: D_m (with the other workgroups' shares), beta_m,
//            gamma_m = Q_(delta_s,b)(beta_m) into LDS                               | barrier
//   pass 2   per row: sum_m gamma_m x_m accumulated per coordinate (gamma split into its
//            low and high byte at 16 bits), then the rounding of z
// Wave 0 also draws the indices two steps ahead and gathers the margins and labels of the
// next step's rows.  The barriers wait for LDS only, loads stay in flight across them.
//
// The B rows of a step (512 KB at B = 64, d = 4096, b = 16: a CU's register file) cannot stay on chip, so
// they travel twice, in chunks of 8 through two register buffers: from HBM for the dots,
// from L2 for the update.  The full-step form, which keeps them in registers, is inner_batch_cut.hip.
#include <algorithm>

#include "inner_batch.hpp"

namespace halp {
namespace {

constexpr int kMaxB = 64;   // rows per step: one per service lane
constexpr int kChunk = 8;   // rows in flight per worker thread

// NDW: dwords of a row per thread; KT: most waves of the workgroup.
template <int BITS, int NDW, int KT>
__global__ __launch_bounds__(64 * KT) void inner_batch_kernel(InArgs a, int nwk, int P, long long* xbuf,
                                                              int spin_limit, int poll_delay) {
  using XT = typename std::conditional<BITS == 8, int8_t, int16_t>::type;
  using HT = typename std::conditional<BITS == 8, int16_t, int32_t>::type;
  constexpr int EPD = 32 / BITS;       // elements per dword
  constexpr int CPT = NDW * EPD;       // coordinates per thread
  constexpr int CT = 16 / BITS;        // coordinates per strip of 16 rounding bits
  constexpr int UPL = CPT / CT;        // strips per thread (= 2 NDW)
  constexpr int QMAX = (1 << (BITS - 1)) - 1, QMIN = -(1 << (BITS - 1));
  const int chain = (int)blockIdx.x / P;         // P workgroups per chain, nwk waves of z each
  const int part = (int)blockIdx.x - chain * P;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int d = a.d, B = a.B;
  const int64_t T = epoch_steps(a.seed + (uint64_t)chain, a.epoch, a.T, a.option2);
  const int64_t row_bytes = a.ldxq * (BITS / 8);
  const unsigned char* __restrict__ Xq = reinterpret_cast<const unsigned char*>(a.Xq) +
                                         (int64_t)chain * a.xq_chain_stride * (BITS / 8);
  const double* sc = a.scales + (int64_t)chain * 8;
  uint64_t* cnt_out = a.counters + (int64_t)chain * 4;
  const uint64_t seed = a.seed + (uint64_t)chain;

  if (sc[7] != 0.0) {
    if (tid < 4) cnt_out[tid] = 0;
    return;
  }
  // polls of the other workgroups' sums before a wait is given up for good; below 0: never wait
  unsigned int n_timeout = spin_limit < 0 ? 1u : 0u;

  __shared__ int s_idx[4][kMaxB];            // sampled rows of steps t .. t+2, slot = step % 4
  __shared__ int s_part[2][16][kMaxB];       // per wave and row: low / high partial dot
  __shared__ int s_gam[kMaxB];               // gamma_m
  __shared__ int s_cl;                       // c_lambda of the step
  __shared__ unsigned long long s_cnt[3];
  if (tid < 3) s_cnt[tid] = 0;
  const bool use_reg = a.lambda > 0;
  const bool lp = a.lp != 0;

  // ---- scalar duties (one row of the step per lane): wave 0, beside its share of z.  (A wave
  // of its own for them would put two waves on one SIMD and halve every wave's registers.)
  const bool svc = wave == 0;
  const int wv = wave;        // this wave's place among the nwk waves that hold z
  const uint32_t N = (uint32_t)a.N;
  const float* __restrict__ phi = a.phi + (int64_t)chain * a.N;
  const float* __restrict__ y = reinterpret_cast<const float*>(a.y) + (int64_t)chain * a.y_chain_stride;
  const double inv_s = sc[5];
  const double dscale = __dmul_rn(a.delta_d, sc[0]);
  const double alpha = a.hyper[2 * chain];
  const double aB = __ddiv_rn(alpha, (double)B);
  const double al = __dmul_rn(alpha, a.lambda);
  const bool row = lane < B;
  const bool need_phi = a.loss != HALP_LOSS_SQUARED || lp;
  unsigned int n_gclamp = 0, n_reg = 0;
  auto draw_idx = [&](int64_t t) {  // row `lane` of step t (any t names a valid row)
    const uint64_t n = (uint64_t)t * (uint64_t)B + (uint64_t)min(lane, B - 1);
    const U4 r = stream_block(seed, kIdx, a.epoch, n >> 2);
    return (int)__umulhi(pick(r, (uint32_t)(n & 3)), N);
  };
  float phi_c = 0.f, y_c = 0.f;
  int i_next = 0;
  // A chain cut across workgroups: every workgroup evaluates all scalars of a step, but only
  // part 0 gathers the margins and labels of the sampled rows (a 128-byte line per 4-byte
  // value and workgroup otherwise).  It does so a step before it needs them and ships them with
  // the sums of the step in between, in two more words per row.
  const bool shipper = P > 1 && part == 0;
  const bool receiver = P > 1 && part != 0;
  // exchange words of the last use, this step's parity first, then the other's
  unsigned long long prev_d[2] = {0, 0}, prev_phi[2] = {0, 0}, prev_y[2] = {0, 0};
  float phi_g = 0.f, y_g = 0.f;  // part 0: margins and labels gathered for the step after this one
  if (svc) {
    const int i0 = draw_idx(0), i1 = draw_idx(1);
    if (row) { s_idx[0][lane] = i0; s_idx[1][lane] = i1; }
    phi_c = need_phi ? phi[i0] : 0.f;
    y_c = a.loss == HALP_LOSS_LOGISTIC ? y[i0] : 0.f;
    i_next = i1;
    if (shipper) {
      phi_g = need_phi ? phi[i1] : 0.f;
      y_g = a.loss == HALP_LOSS_LOGISTIC ? y[i1] : 0.f;
    }
  }
  {
    // ========================================================================= worker
    const HT* __restrict__ hg = reinterpret_cast<const HT*>(a.h) + (int64_t)chain * d;
    XT* __restrict__ zg = reinterpret_cast<XT*>(a.z) + (int64_t)chain * d;
    float* __restrict__ wg = a.w + (int64_t)chain * d;
    // the waves of a workgroup (and the workgroups of a chain) hold consecutive slices
    const int j0 = (part * 64 * nwk + wv * 64 + lane) * CPT;
    const bool active = j0 < d;
    // Rows are padded to whole 8-byte groups; a 16-byte fragment is only used when rows are
    // 16-byte multiples (checked on the host), so a fragment that starts below d lies inside
    // the row.  Threads past the row re-read its first fragment; their z stays 0.
    const int frag_off = active ? j0 * (BITS / 8) : 0;
    int z[CPT], hv[CPT];
    bool ok[CPT];
#pragma unroll
    for (int k = 0; k < CPT; ++k) {
      ok[k] = j0 + k < d;
      const int j = min(j0 + k, d - 1);
      z[k] = ok[k] ? (int)zg[j] : 0;
      hv[k] = ok[k] ? (int)hg[j] : 0;
    }
    const uint32_t strip0 = (uint32_t)(j0 / CT);
    // At 8 strips per thread the window's 8 Philox blocks (32 registers) are parked in LDS
    // as [word][strips 0..3 | 4..7][thread] of 16 bytes (a wave reads consecutive addresses;
    // a thread reads only what it wrote) and the words of two steps are fetched at a time.
    constexpr bool kPark = UPL == 8;
    extern __shared__ __attribute__((aligned(16))) uint4 s_zr[];
    const int nworkers = 64 * nwk;      // threads that hold z
    const int wtid = wv * 64 + lane;    // this thread's place among them
    U4 zr[kPark ? 1 : UPL];
    uint32_t zw[kPark ? UPL : 1];
    unsigned long long n_zclamp = 0;
    auto load_frag = [&](uint32_t (&dst)[NDW], int i) {
      const unsigned char* rp = Xq + (int64_t)i * row_bytes + frag_off;
      if (NDW == 1) {
        dst[0] = *reinterpret_cast<const uint32_t*>(rp);
      } else if (NDW == 2) {
        const uint2 v = *reinterpret_cast<const uint2*>(rp);
        dst[0] = v.x; dst[NDW > 1 ? 1 : 0] = v.y;
      } else {
        const uint4 v = *reinterpret_cast<const uint4*>(rp);
        dst[0] = v.x; dst[NDW > 1 ? 1 : 0] = v.y; dst[NDW > 2 ? 2 : 0] = v.z; dst[NDW > 3 ? 3 : 0] = v.w;
      }
    };
    uint32_t xa[kChunk][NDW], xb[kChunk][NDW];
    auto load_chunk = [&](uint32_t (&dst)[kChunk][NDW], const int* idx, int m0) {
      const int mine = idx[min(m0 + (lane & (kChunk - 1)), B - 1)];  // lane r: row m0 + r, one LDS read
#pragma unroll
      for (int r = 0; r < kChunk; ++r)  // the row number is uniform: scalar address arithmetic
        load_frag(dst[r], __builtin_amdgcn_readlane(mine, r));
    };
    __syncthreads();
    load_chunk(xa, s_idx[0], 0);

    // wave 0: the rounding word of gamma_m and the L2 draw of a step, made a step ahead
    uint32_t rw_next = 0;
    int cl_next = 0;
    auto draw_scalars = [&](int64_t tn) {
      const uint64_t n = (uint64_t)tn * (uint64_t)B + (uint64_t)min(lane, B - 1);
      rw_next = pick(stream_block(seed, kGamma, a.epoch, n >> 2), (uint32_t)(n & 3));
      cl_next = 0;
      if (use_reg) {
        const uint32_t rr = pick(stream_block(seed, kReg, a.epoch, (uint64_t)tn >> 2), (uint32_t)(tn & 3));
        cl_next = (int)quantize_real(al, (double)(1 << BITS), rr, 0.0, (double)QMAX, nullptr);
      }
    };
    if (svc) draw_scalars(0);

    auto one_step = [&](int64_t t) {
      const int* idx = s_idx[t & 3];
      // wave 0: what the scalar stage needs and does not depend on the dots — margins and
      // labels of the next step's rows (used after the next barrier pair), the rounding word
      // of gamma_m, the L2 draw
      float phi_n = 0.f, y_n = 0.f;
      uint32_t rw = 0;
      int cl_draw = 0;
      if (svc) {
        if (P == 1) {
          const int inx = i_next;
          phi_n = need_phi ? phi[inx] : 0.f;
          y_n = a.loss == HALP_LOSS_LOGISTIC ? y[inx] : 0.f;
        } else if (shipper) {  // gathered after the last step's gamma (before the loop for step 0)
          phi_n = phi_g;
          y_n = y_g;
        }  // the other parts receive them with the sums below
        rw = rw_next;  // drawn during the previous step (or before the first)
        cl_draw = cl_next;
        n_reg += (lane == 0 && cl_draw != 0) ? 1u : 0u;
      }
      // What wave 0 prepares for later steps: with several workgroups per chain it runs while
      // the wave waits for the others' sums, else here, while the other waves take the dots.
      auto prepare_ahead = [&]() { draw_scalars(t + 1); };
      if (svc && P == 1) prepare_ahead();
      if ((t & 7) == 0) {
        if (kPark) {
#pragma unroll
          for (int q = 0; q < UPL / 4; ++q) {
            U4 blk[4];
#pragma unroll
            for (int u = 0; u < 4; ++u)
              blk[u] = zround_block(seed, a.epoch, strip0 + (uint32_t)(4 * q + u), (uint32_t)(t >> 3));
#pragma unroll
            for (int wd = 0; wd < 4; ++wd)
              s_zr[(wd * (UPL / 4) + q) * nworkers + wtid] =
                  make_uint4(pick(blk[0], wd), pick(blk[1], wd), pick(blk[2], wd), pick(blk[3], wd));
          }
        } else {
#pragma unroll
          for (int u = 0; u < (kPark ? 1 : UPL); ++u)
            zr[u] = zround_block(seed, a.epoch, strip0 + (uint32_t)u, (uint32_t)(t >> 3));
        }
      }
      if (kPark && (t & 1) == 0) {  // the block word that serves steps t and t + 1
#pragma unroll
        for (int q = 0; q < UPL / 4; ++q) {
          const uint4 v = s_zr[(((int)(t & 7) >> 1) * (UPL / 4) + q) * nworkers + wtid];
          zw[(4 * q) % UPL] = v.x; zw[(4 * q + 1) % UPL] = v.y;
          zw[(4 * q + 2) % UPL] = v.z; zw[(4 * q + 3) % UPL] = v.w;
        }
      }
      // z packed for the dots: bytes at 8 bits; low parts and high parts apart at 16 bits
      uint32_t zp[NDW], zq[NDW];
#pragma unroll
      for (int q = 0; q < NDW; ++q) {
        if (BITS == 8) {
          zp[q] = (uint32_t)(z[4 * q] & 0xFF) | ((uint32_t)(z[4 * q + 1] & 0xFF) << 8) |
                  ((uint32_t)(z[4 * q + 2] & 0xFF) << 16) | ((uint32_t)(z[4 * q + 3] & 0xFF) << 24);
          zq[q] = 0;
        } else {
          // z = 256 zh + zl with zl in [-128, 127]: both parts at most 128 in magnitude, so a
          // wave's sum of 512 products with |x| <= 32767 stays below 2^31
          const int za = z[(2 * q) % CPT], zb = z[(2 * q + 1) % CPT];
          const int ha = (za + 128) >> 8, hb = (zb + 128) >> 8;
          const int la = za - 256 * ha, lb = zb - 256 * hb;
          zp[q] = (uint32_t)(la & 0xFFFF) | ((uint32_t)lb << 16);
          zq[q] = (uint32_t)(ha & 0xFFFF) | ((uint32_t)hb << 16);
        }
      }
      // Rows come in chunks of 8 through two register buffers: while one chunk is worked on
      // the next is in flight, across the passes and across the steps (the chunk after the
      // last of pass 1 is the first of pass 2; after pass 2, the first of the next step).
      // ---- pass 1: dots
      auto dots = [&](uint32_t (&xf)[kChunk][NDW], int m0) {
        int lo[kChunk], hi[kChunk];
#pragma unroll
        for (int r = 0; r < kChunk; ++r) {
          lo[r] = hi[r] = 0;
#pragma unroll
          for (int q = 0; q < NDW; ++q) {
            if (BITS == 8) {
              lo[r] = __builtin_amdgcn_sdot4((int)xf[r][q], (int)zp[q], lo[r], false);
            } else {
              const short2v xv = __builtin_bit_cast(short2v, xf[r][q]);
              lo[r] = __builtin_amdgcn_sdot2(xv, __builtin_bit_cast(short2v, zp[q]), lo[r], false);
              hi[r] = __builtin_amdgcn_sdot2(xv, __builtin_bit_cast(short2v, zq[q]), hi[r], false);
            }
          }
        }
        const int slo = wave_sums8_i32(lo, lane);  // row m0 + lane % 8
        const int shi = BITS == 16 ? wave_sums8_i32(hi, lane) : 0;
        if (lane < kChunk && m0 + lane < B) {
          s_part[0][wv][m0 + lane] = slo;
          if (BITS == 16) s_part[1][wv][m0 + lane] = shi;
        }
      };
      for (int m0 = 0; m0 < B; m0 += 2 * kChunk) {
        load_chunk(xb, idx, m0 + kChunk);
        dots(xa, m0);
        load_chunk(xa, idx, m0 + 2 * kChunk < B ? m0 + 2 * kChunk : 0);
        if (m0 + kChunk < B) dots(xb, m0 + kChunk);
      }
      lds_barrier();  // the partial dots of this step are in LDS
      if (svc) {
        // l'(phi_m) does not depend on the dots: evaluated here, ahead of the wait for the other
        // workgroups' sums, so that only l'(phi_m + x_m^T z) follows it
        const double a0 = (double)phi_c, yi = (double)y_c;
        double rho_m = __dmul_rn((double)rw, 0x1p-32);  // the rounding draw of gamma_m
        asm volatile("" : "+v"(rho_m));
        double dl0 = 0.0;
        if (P == 1) {
          if (a.loss == HALP_LOSS_LOGISTIC) dl0 = logistic_dl(a0, yi);
          asm volatile("" : "+v"(dl0));  // stays where it is written
        }
        long long D = 0;
        for (int w2 = 0; w2 < nwk; ++w2) {
          const long long lo = s_part[0][w2][min(lane, B - 1)];
          const long long hi = BITS == 8 ? 0 : s_part[1][w2][min(lane, B - 1)];
          D += lo + hi * 256;
        }
        if (P > 1) {
          // The other workgroups' shares of the dots.  Every workgroup adds its share to the row's
          // 64-bit word with one device-scope atomic, the share in the low 56 bits and a 1 in the
          // top byte; the sum is there when the top byte has moved by P since the word's last use,
          // two steps ago (both fields are differences modulo 2^64, so nothing is reset).  A word
          // is used again only after every workgroup of the chain has read it: its next addition
          // follows this step's gamma, hence everyone's share of the step after.  Margins and
          // labels travel the same way, in words that part 0 alone adds to.
          unsigned long long* xb = reinterpret_cast<unsigned long long*>(xbuf) +
                                   (((int64_t)chain * 2 + (int64_t)(t & 1)) * kBatchSlots) * kMaxB;
          auto add = [&](int slot, unsigned long long v) {
            __hip_atomic_fetch_add(&xb[slot * kMaxB + lane], (1ull << 56) + v, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
          };
          add(0, (unsigned long long)D);
          const bool logistic = a.loss == HALP_LOSS_LOGISTIC;
          if (shipper && need_phi) add(1, (unsigned long long)__float_as_uint(phi_g));
          if (shipper && logistic) add(2, (unsigned long long)__float_as_uint(y_g));
          const bool want_phi = receiver && need_phi, want_y = receiver && logistic;
          if (logistic) dl0 = logistic_dl(a0, yi);  // behind the publish, ahead of the wait
          asm volatile("" : "+v"(dl0));
          prepare_ahead();
          // polls that start before the additions can be back only add traffic
          if (n_timeout == 0) {
            for (int i = 0; i < poll_delay; ++i) __builtin_amdgcn_s_sleep(4);
          }
          unsigned long long v = prev_d[0], vp = prev_phi[0], vy = prev_y[0];
          for (int spin = 0; n_timeout == 0; ++spin) {  // after one wait ran out, none is tried again
            v = __hip_atomic_load(&xb[lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (want_phi) vp = __hip_atomic_load(&xb[kMaxB + lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (want_y) vy = __hip_atomic_load(&xb[2 * kMaxB + lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            // a signed sum below 2^55 in magnitude may borrow from the top byte
            bool missing = (uint32_t)((v - prev_d[0] + (1ull << 55)) >> 56) != (uint32_t)P;
            if (want_phi) missing = missing || ((vp - prev_phi[0]) >> 56) != 1ull;
            if (want_y) missing = missing || ((vy - prev_y[0]) >> 56) != 1ull;
            if (__ballot(missing) == 0) break;
            if (spin >= spin_limit) n_timeout = 1;  // only if a workgroup of the chain never ran: give up
          }
          if (n_timeout == 0) D = (long long)(v - prev_d[0] - ((unsigned long long)P << 56));
          if (want_phi) phi_n = __uint_as_float((uint32_t)(vp - prev_phi[0]));
          if (want_y) y_n = __uint_as_float((uint32_t)(vy - prev_y[0]));
          prev_d[0] = prev_d[1]; prev_phi[0] = prev_phi[1]; prev_y[0] = prev_y[1];
          prev_d[1] = v; prev_phi[1] = vp; prev_y[1] = vy;
        }
        // beta_m = (alpha / B) (l'(phi_m + x_m^T z) - l'(phi_m)), gamma_m = Q_(delta_s, b)(beta_m)
        const double delta = __dmul_rn(dscale, (double)D);
        double diff;
        if (a.loss == HALP_LOSS_LOGISTIC) {
          const double a1 = lp ? delta : __dadd_rn(a0, delta);
          diff = __dadd_rn(logistic_dl(a1, yi), -dl0);
        } else {
          diff = lp ? __dadd_rn(delta, -a0) : delta;
        }
        const double beta = __dmul_rn(aB, diff);
        // gamma_m = Q_(delta_s, b)(beta_m): floor(beta / delta_s + rho), clamped -- the quantizer of
        // quantize_real with its draw converted ahead of the wait and the result taken as a
        // 32-bit integer (it lies in the box after the clamp)
        const double fq = floor(__dadd_rn(__dmul_rn(beta, inv_s), rho_m));
        const double fc = fmin(fmax(fq, (double)QMIN), (double)QMAX);
        const bool hit = fq != fc;
        const int gq = (int)fc;
        if (row) {
          s_gam[lane] = gq;
          n_gclamp += hit ? 1u : 0u;
        }
        if (lane == 0) s_cl = cl_draw;
        {  // indices two steps ahead (slot (t + 2) % 4 was last read in step t - 2)
          const int i2 = draw_idx(t + 2);
          if (row) s_idx[(t + 2) & 3][lane] = i2;
          i_next = i2;
        }
        phi_c = phi_n; y_c = y_n;
      }
      lds_barrier();  // gamma is out
      if (svc && shipper) {  // margins and labels of the rows two steps on, shipped with the next step's sums
        const int i2 = i_next;
        phi_g = need_phi ? phi[i2] : 0.f;
        y_g = a.loss == HALP_LOSS_LOGISTIC ? y[i2] : 0.f;
      }
      // ---- pass 2: sum_m gamma_m x_m per coordinate (low / high byte of gamma apart at 16 bits)
      int acc[CPT], acch[CPT];
#pragma unroll
      for (int k = 0; k < CPT; ++k) acc[k] = acch[k] = 0;
      auto accumulate = [&](uint32_t (&xf)[kChunk][NDW], int m0) {
        int gm[kChunk];
        const int gmine = s_gam[min(m0 + (lane & (kChunk - 1)), kMaxB - 1)];  // lane r: row m0 + r
#pragma unroll
        for (int r = 0; r < kChunk; ++r) gm[r] = m0 + r < B ? __builtin_amdgcn_readlane(gmine, r) : 0;
        if (BITS == 16) {
          // Two rows at a time: v_perm puts coordinate j of both rows into one register, one
          // v_dot2 against the pair of gammas then serves both rows.  gamma = 256 gh + gl with
          // gl in [0, 255]: 64 products of each part stay below 2^31.
#pragma unroll
          for (int r = 0; r < kChunk; r += 2) {
            const uint32_t glp = (uint32_t)(gm[r] & 0xFF) | ((uint32_t)(gm[r + 1] & 0xFF) << 16);
            const uint32_t ghp = (uint32_t)((gm[r] >> 8) & 0xFFFF) | ((uint32_t)(gm[r + 1] >> 8) << 16);
            const short2v gl2 = __builtin_bit_cast(short2v, glp), gh2 = __builtin_bit_cast(short2v, ghp);
#pragma unroll
            for (int q = 0; q < NDW; ++q) {
              const uint32_t xr0 = xf[r][q], xr1 = xf[r + 1][q];
              // (row r, row r + 1) of the even and of the odd coordinate of this dword
              const short2v pe = __builtin_bit_cast(short2v, __builtin_amdgcn_perm(xr1, xr0, 0x05040100u));
              const short2v po = __builtin_bit_cast(short2v, __builtin_amdgcn_perm(xr1, xr0, 0x07060302u));
              acc[(2 * q) % CPT] = __builtin_amdgcn_sdot2(pe, gl2, acc[(2 * q) % CPT], false);
              acch[(2 * q) % CPT] = __builtin_amdgcn_sdot2(pe, gh2, acch[(2 * q) % CPT], false);
              acc[(2 * q + 1) % CPT] = __builtin_amdgcn_sdot2(po, gl2, acc[(2 * q + 1) % CPT], false);
              acch[(2 * q + 1) % CPT] = __builtin_amdgcn_sdot2(po, gh2, acch[(2 * q + 1) % CPT], false);
            }
          }
        } else {
#pragma unroll
          for (int r = 0; r < kChunk; ++r) {
#pragma unroll
            for (int k = 0; k < CPT; ++k) {
              const uint32_t xv = xf[r][k / EPD];
              const int x = (int)(int8_t)(xv >> ((k % EPD) * 8));
              acc[k] = mad24(gm[r], x, acc[k]);
            }
          }
        }
      };
      const int* idn = s_idx[(t + 1) & 3];
      for (int m0 = 0; m0 < B; m0 += 2 * kChunk) {
        load_chunk(xb, idx, m0 + kChunk);
        accumulate(xa, m0);
        if (m0 + 2 * kChunk < B) load_chunk(xa, idx, m0 + 2 * kChunk);
        else load_chunk(xa, idn, 0);
        accumulate(xb, m0 + kChunk);
      }
      // ---- u = z - sum gamma x - h~ - c_lambda z in (delta_i, 2b); z = Q_(delta_m, b)(u)
      const int cl = use_reg ? s_cl : 0;
#pragma unroll
      for (int k = 0; k < CPT; ++k) {
        // the strip's 16-bit field of this step: half (t % 2) of word (t % 8) / 2 of its block
        const uint32_t field = kPark ? (zw[(k / CT) % (kPark ? UPL : 1)] >> (16u * (uint32_t)(t & 1))) & 0xFFFFu
                                     : zround_field(zr[kPark ? 0 : k / CT], (uint32_t)t);
        const long long re = (long long)((field >> ((k % CT) * BITS)) & ((1u << BITS) - 1u));
        const long long gsum = (long long)acc[k] + (BITS == 16 ? (long long)acch[k] * 256 : 0);
        const long long v = -(long long)hv[k] - (long long)cl * (long long)z[k] - gsum;
        const long long zu = (long long)z[k] + ((v + re) >> BITS);
        const long long zc = zu > QMAX ? QMAX : (zu < QMIN ? QMIN : zu);
        n_zclamp += (ok[k] && zu != zc) ? 1u : 0u;
        z[k] = ok[k] ? (int)zc : 0;
      }
    };
    for (int64_t t = 0; t < T; ++t) one_step(t);

    // ---- w~ <- w~ + delta_m z (option I; Algorithm 2: w~ = delta z); hand z out
    const double delta_m = sc[0];
#pragma unroll
    for (int k = 0; k < CPT; ++k) {
      if (ok[k]) {
        const int j = j0 + k;
        zg[j] = (XT)z[k];
        if (P == 1) {  // several workgroups per chain: split_finish applies the offset
          const double step = __dmul_rn(delta_m, (double)z[k]);
          wg[j] = lp ? (float)step : (float)__dadd_rn((double)wg[j], step);
        }
      }
    }
    if (n_zclamp) atomicAdd(&s_cnt[0], n_zclamp);
    if (n_gclamp) atomicAdd(&s_cnt[1], (unsigned long long)n_gclamp);
    if (n_reg) atomicAdd(&s_cnt[2], (unsigned long long)n_reg);
  }
  __syncthreads();
  if (P == 1) {
    if (tid < 4) cnt_out[tid] = tid < 3 ? s_cnt[tid] : 0ull;
  } else {
    // counters were cleared before the launch: clamped coordinates add up over the parts, the
    // scalar counts are the same in every part, a timed-out wait is flagged in the last word
    if (tid == 0 && s_cnt[0]) atomicAdd(reinterpret_cast<unsigned long long*>(&cnt_out[0]), s_cnt[0]);
    if (part == 0 && (tid == 1 || tid == 2)) cnt_out[tid] = s_cnt[tid];
    if (tid == 0 && n_timeout) atomicMax(reinterpret_cast<unsigned long long*>(&cnt_out[3]), 1ull);
  }
}

// Several workgroups per chain: w~ <- w~ + delta_m z is applied here, after the launch, and only
// for chains none of whose workgroups gave up a wait.  A chain with a wait that ran out keeps
// its w~ (its z is then not a trajectory of the method) and, with report, gets status -2 in scales[7].
template <int BITS>
__global__ __launch_bounds__(256) void split_finish(InArgs a, double* scales, const void* zs, int chain0, int report) {
  using XT = typename std::conditional<BITS == 8, int8_t, int16_t>::type;
  const int chain = chain0 + (int)blockIdx.y;
  const int j = (int)(blockIdx.x * 256 + threadIdx.x);
  double* sc = scales + (int64_t)chain * 8;
  if (a.counters[(int64_t)chain * 4 + 3] != 0) {
    if (report && j == 0) sc[7] = -2.0;
    return;
  }
  const int n = a.K * a.d;
  if (sc[7] != 0.0 || j >= n) return;  // a gradient of zero or not finite: the loop did not run
  const XT zk = reinterpret_cast<const XT*>(zs)[(int64_t)blockIdx.y * n + j];
  if (zs != a.z) reinterpret_cast<XT*>(a.z)[(int64_t)chain * n + j] = zk;
  float* wg = a.w + (int64_t)chain * n;
  const double step = __dmul_rn(sc[0], (double)zk);
  wg[j] = a.lp ? (float)step : (float)__dadd_rn((double)wg[j], step);
}

// clears what the split launch accumulates into or waits on
__global__ void split_prepare(long long* xbuf, int nwords, uint64_t* counters, int ncounters) {
  const int k = (int)(blockIdx.x * blockDim.x + threadIdx.x);
  if (k < nwords) xbuf[k] = 0;
  if (k < ncounters) counters[k] = 0;
}

template <int BITS, int NDW, int KT>
int launch_kt(const InArgs& a, int nwk, int P, long long* xbuf, int spin_limit, int poll_delay, dim3 grid, dim3 block,
              size_t smem, hipStream_t s) {
  auto kern = inner_batch_kernel<BITS, NDW, KT>;
  if (smem > 0 && hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                      hipFuncAttributeMaxDynamicSharedMemorySize,
                                      (int)smem) != hipSuccess)
    return HALP_ERR_HIP;
  hipLaunchKernelGGL(kern, grid, block, smem, s, a, nwk, P, xbuf, spin_limit, poll_delay);
  return hip_ok(hipGetLastError());
}

struct BtShape {
  int ndw, nwk;
};

// dwords per thread and worker waves: the widest fragment the row alignment allows that
// still gives every SIMD a wave, at most 15 worker waves
BtShape pick_shape(const halp_params& p, int64_t row_bytes) {
  const int epd = 32 / p.b;
  int ndw = row_bytes % 16 == 0 ? 4 : 2;
  while (ndw > 1 && (p.d + 64 * ndw * epd - 1) / (64 * ndw * epd) < 4) ndw /= 2;
  int nwk = (p.d + 64 * ndw * epd - 1) / (64 * ndw * epd);
  while (nwk > 16 && ndw < (row_bytes % 16 == 0 ? 4 : 2)) {
    ndw *= 2;
    nwk = (p.d + 64 * ndw * epd - 1) / (64 * ndw * epd);
  }
  return BtShape{ndw, nwk};
}

}  // namespace

void launch_split_prepare(long long* xbuf, int nwords, uint64_t* counters, int ncounters, hipStream_t s) {
  const int n = nwords > ncounters ? nwords : ncounters;
  hipLaunchKernelGGL(split_prepare, dim3((n + 255) / 256), dim3(256), 0, s, xbuf, nwords, counters, ncounters);
}

int launch_split_finish(const InArgs& a, double* scales, const void* zs, int chain0, int chains, bool report, int bits,
                        hipStream_t s) {
  const dim3 grid((a.K * a.d + 255) / 256, chains);
  if (bits == 8) hipLaunchKernelGGL(split_finish<8>, grid, dim3(256), 0, s, a, scales, zs, chain0, report ? 1 : 0);
  else hipLaunchKernelGGL(split_finish<16>, grid, dim3(256), 0, s, a, scales, zs, chain0, report ? 1 : 0);
  return hip_ok(hipGetLastError());
}

// K = 1, 2 <= B <= 64, squared or logistic loss, up to 16 waves of 16-byte fragments
int inner_batch_supported(const halp_handle& h) {
  const halp_params& p = h.p;
  if (p.K != 1 || p.B < 2 || p.B > kMaxB) return HALP_ERR_UNSUPPORTED;
  if (p.loss != HALP_LOSS_SQUARED && p.loss != HALP_LOSS_LOGISTIC) return HALP_ERR_UNSUPPORTED;
  if (p.b == 8 && p.d > 131071) return HALP_ERR_UNSUPPORTED;  // int32 dots stay exact
  if (!h.bound || !h.buf.Xq) return HALP_ERR_NOT_BOUND;
  const int64_t row_bytes = h.buf.ldxq * (p.b / 8);
  const BtShape sh = pick_shape(p, row_bytes);
  if (sh.nwk > 16) return HALP_ERR_UNSUPPORTED;
  // every fragment that starts below d must lie inside the row
  const int cpt = sh.ndw * 32 / p.b;
  if ((int64_t)((p.d + cpt - 1) / cpt) * sh.ndw * 4 > row_bytes) return HALP_ERR_UNSUPPORTED;
  if (sh.ndw == 4 && reinterpret_cast<uintptr_t>(h.buf.Xq) % 16 != 0) return HALP_ERR_UNSUPPORTED;
  return HALP_OK;
}

// Launch shape.  Full-step form (one slice of the row per workgroup, the rows of a step dealt
// to its waves and kept in registers): taken by default whenever the slices of a row are few
// enough for one workgroup each.  Otherwise, and whenever HALP_OPT_INNER_PARTS names a count,
// the chunked form with that many workgroups per chain.  Workgroups of a chain wait for each
// other, so there are only as many as are surely resident at once (at most one per CU).
struct BtLaunch {
  bool fs;
  int ndw, nwk, P;  // nwk: waves of z per workgroup
};

static BtLaunch pick_launch(const halp_handle& h, int64_t row_bytes) {
  const halp_params& p = h.p;
  const BtShape sh = pick_shape(p, row_bytes);
  int most = 1;
  if (h.batch_xbuf) {
    most = kBatchMaxParts;
    while (most > 1 && (int64_t)p.R * most > h.num_cus) most /= 2;
  }
  int most_any = 1;  // any count up to kBatchMaxParts
  if (h.batch_xbuf) {
    most_any = (int)(h.num_cus / p.R);
    if (most_any > kBatchMaxParts) most_any = kBatchMaxParts;
    if (most_any < 1) most_any = 1;
  }
  if (h.inner_parts == 0) {
    // full-step form (inner_batch_cut.hip): slices, one workgroup each, few enough to be resident together
    const int epd = 32 / p.b;
    const bool al16 = row_bytes % 16 == 0 && reinterpret_cast<uintptr_t>(h.buf.Xq) % 16 == 0;
    const int ndw_max = (al16 && p.b == 16) ? 4 : 2;  // 8 coordinates per thread at most
    auto fits = [&](int ndw, int& P) {
      const int cpt = ndw * epd;
      P = (p.d + 64 * cpt - 1) / (64 * cpt);
      if (P > most_any || !inner_batch_cut_takes(p.B, ndw)) return false;
      // Few small steps: a chain cut across workgroups takes three launches more, some 10 us.  us per epoch of 1, 3, 6 and 12
      // steps, one workgroup (the chunked form) / cut: rows of 600 bytes, B = 2, 64 chains 12 / 21, 19 / 24, 30 / 29, 51 / 38; of 2048 bytes
      // (8 bits, B = 2) 14 / 20, 23 / 24, 35 / 28, 61 / 37; (16 bits, 64 chains) 13 / 21, 21 / 24, 33 / 29, 57 / 40; of 4096, 64
      // chains 16 / 23, 25 / 27, 39 / 33, 67 / 44; of 6000, 1 and 4 steps 21 / 21, 35 / 26; of 1200, 4 and 5 steps 23 / 26, 26 / 28.  Steps of 16 KB of rows: cut at once,
      // 1024 x 16 bits B = 8 25 / 22, 31 / 27.
      const int64_t least_steps = row_bytes <= 1536 ? 6 : (row_bytes <= 4096 ? 4 : 0);
      if (P > 1 && p.T < least_steps && (int64_t)p.B * row_bytes < 16 * 1024) return false;
      return (int64_t)((p.d + cpt - 1) / cpt) * ndw * 4 <= row_bytes;  // fragments inside the row
    };
    // A chain cut across workgroups: the narrowest fragment of at least four coordinates whose
    // slices are few enough -- more, narrower slices shorten both passes over the rows of a step.  us per step, 4096 x 16
    // bits, B = 64, N = 100 000: 3.14 with 8 slices, 2.51 with 16; 4096 x 8 bits, N = 400 000: 2.26 and 2.00.
    // One workgroup where the widest fragment lets it hold the row, for the smaller steps (no exchange).  us per step, one
    // workgroup and two: 8 bits d = 300 B = 4 1.11 / 1.59, 500 B = 64 1.75 / 1.74, 500 B = 128 2.72 / 2.38;
    // 16 bits 500 B = 4 1.42 / 1.69, 300 B = 32 1.76 / 2.00, 500 B = 64 2.52 / 2.23.
    int P = 1;
    const bool alone = p.B <= (p.b == 8 ? 64 : 32) && fits(ndw_max, P) && P == 1;
    for (int ndw = p.b == 16 ? 2 : 1; ndw <= ndw_max && !alone; ndw *= 2)
      if (fits(ndw, P) && P > 1) return BtLaunch{true, ndw, 0, P};
    for (int ndw = ndw_max; ndw >= 1; ndw /= 2)
      if (fits(ndw, P)) return BtLaunch{true, ndw, 0, P};
  }
  int P = 1;
  if (h.inner_parts > 0) {
    while (most > sh.nwk) most /= 2;
    P = h.inner_parts < most ? h.inner_parts : (most < 1 ? 1 : most);
  }
  return BtLaunch{false, sh.ndw, (sh.nwk + P - 1) / P, P};
}

// 65 .. 128 rows per step: only where the full-step form takes them
bool inner_batch_wide_takes(const halp_handle& h) {
  const halp_params& p = h.p;
  if (p.K != 1 || p.B <= kMaxB || p.algorithm == HALP_ALG_SVRG || (p.b == 8 && p.d > 131071)) return false;
  return h.bound && h.buf.Xq && h.inner_parts == 0 && pick_launch(h, h.buf.ldxq * (p.b / 8)).fs;
}

// ... whatever is bound: at 8 bits a fragment is 8 bytes at most, which lies inside a row of any stride
bool inner_batch_wide_takes_all(const halp_handle& h) {
  const halp_params& p = h.p;
  if (p.K != 1 || p.b != 8 || p.B <= kMaxB || p.algorithm == HALP_ALG_SVRG || p.d > 131071) return false;
  return h.inner_parts == 0 && pick_launch(h, ((int64_t)p.d + 7) / 8 * 8).fs;
}

size_t inner_batch_workspace(const halp_params& p) {
  return std::max((size_t)p.R * 2 * kBatchSlots * 64 * sizeof(long long), inner_batch_cut_workspace(p));
}

int inner_batch_parts(const halp_handle& h) { return pick_launch(h, h.buf.ldxq * (h.p.b / 8)).P; }

int launch_inner_batch(const halp_handle& h, uint32_t epoch, hipStream_t s) {
  const halp_params& p = h.p;
  const int rc = p.B > kMaxB ? (inner_batch_wide_takes(h) ? HALP_OK : HALP_ERR_UNSUPPORTED) : inner_batch_supported(h);
  if (rc != HALP_OK) return rc;
  const InArgs a = make_inner_args(h, epoch);
  const BtLaunch L = pick_launch(h, h.buf.ldxq * (p.b / 8));
  if (L.fs) return launch_inner_batch_cut(h, a, L.ndw, L.P, s);
  const int nwk = L.nwk, P = L.P;
  const int nwaves = nwk;
  const dim3 grid(p.R * P), block(64 * nwaves);
  if (P > 1) {
    const int nwords = p.R * 2 * kBatchSlots * kMaxB, ncnt = p.R * 4;
    launch_split_prepare(h.batch_xbuf, nwords, h.buf.counters, ncnt, s);
  }
  // parked Philox blocks: 128 bytes per worker thread at 8 strips per thread (120 KB at most)
  const size_t smem = L.ndw == 4 ? (size_t)64 * nwk * 128 : 0;
#define HALP_BT(BITS_, NDW_)                                                                                               \
  if (p.b == BITS_ && L.ndw == NDW_) {                                                                                     \
    if (nwaves <= 4)                                                                                                       \
      return launch_kt<BITS_, NDW_, 4>(a, nwk, P, h.batch_xbuf, h.spin_limit, h.poll_delay, grid, block, smem, s);         \
    if (nwaves <= 8)                                                                                                       \
      return launch_kt<BITS_, NDW_, 8>(a, nwk, P, h.batch_xbuf, h.spin_limit, h.poll_delay, grid, block, smem, s);         \
    if (nwaves <= 12)                                                                                                      \
      return launch_kt<BITS_, NDW_, 12>(a, nwk, P, h.batch_xbuf, h.spin_limit, h.poll_delay, grid, block, smem, s);        \
    return launch_kt<BITS_, NDW_, 16>(a, nwk, P, h.batch_xbuf, h.spin_limit, h.poll_delay, grid, block, smem, s);          \
  }
  auto launch_loop = [&]() -> int {
    HALP_BT(8, 1) HALP_BT(8, 2) HALP_BT(8, 4)
    HALP_BT(16, 1) HALP_BT(16, 2) HALP_BT(16, 4)
    return HALP_ERR_UNSUPPORTED;
  };
#undef HALP_BT
  const int lrc = launch_loop();
  if (lrc != HALP_OK || P == 1) return lrc;
  return launch_split_finish(a, h.buf.scales, a.z, 0, p.R, true, p.b, s);
}

}  // namespace halp
