// Inner loop of Algorithm 4 (LM-HALP) with a minibatch at 8 bits, on the matrix cores: softmax
// with K <= 16 classes, 2 <= B <= 512 rows per step, and the scalar margins (K = 1, squared or
// logistic loss) of minibatches wider than the kernel for that case holds.
//
// A step is two integer contractions with a scalar stage between them,
//   D = X Z      [rows x classes], over the row's coordinates
//   G = X^T Gamma  [coordinates x classes], over the step's rows,
// and both run as 16x16x64 int8 products.  One workgroup per chain: eight owner waves hold z,
// four scalar waves (one per SIMD) take the scalars.  Coordinates are cut into blocks of 64,
// owner w holds blocks w and w + 8 (rows up to 1024 coordinates), all classes of them.  Lane
// (c = l % 16, q = l / 16) holds class c's coordinates 64 blk + 32 (q / 2) + 8 j + 4 (q % 2) + i,
// i, j = 0 .. 3: where the result of G lands when its left operand comes from the transposing LDS
// reads (ds_read_b64_tr_b8: 8 rows x 16 coordinates per 16 lanes, no byte shuffles).  Two lane
// exchanges (v_permlane16_swap) turn that into the 16 consecutive bytes per lane that the class
// operand of D takes, so z never leaves registers.
// Rows are taken up to 64 at a time (a wider minibatch 32 at a time, G accumulated in the products'
// accumulators, which start at h~: the update subtracts them from the rounding bits, shifts and
// adds z).
//
// One iteration (a chunk of rows of a step):
//   owners   D of their blocks, 16 rows at a time, parts into LDS                      | barrier
//   scalars  add up the parts of 16 rows per wave: lane (class, row group) has four rows of a
//            class; a 4 x 4 exchange inside every quad of lanes makes that four classes of a row,
//            so that the softmax after the offset takes two lane exchanges per fold and its fp64
//            work is four independent chains; gamma into LDS
//   owners   meanwhile: rows of the next iteration into the second LDS buffer, rows of the
//            one after requested                                                       | barrier
//   owners   G, and after the last chunk of a step the update of z
// Indices, margins, the softmax before the offset, rounding words and bits come from the
// segment's records (softmax_ahead.hpp), read an iteration ahead.
//
// What bounds it (K = 10, d = 784, B = 64, shader-clock stamps, cycles of an iteration of ~5700):
// D and its parts ~1300, adding them up and the fp64 softmax ~2200 (issue of one wave per SIMD,
// ~290 vector instructions in four chains), G and update ~1500-2100 (two owners per SIMD, ~66 vector
// instructions per block of 64 x 16).  us per step, the class-wave kernel with vector dot
// products before it in brackets: B = 64 2.4 (27), B = 8 2.2 (11), B = 256 13.8 (~105);
// 256 chains, B = 64: 6.2 (27).  Tried on the way: all sixteen waves in every role
// (spills, and the scalar stage is bound by issue: 3.2); z and D's sum through LDS atomics (8 cycles
// per wave and instruction: 3.8); rows copied by the scalar waves (they get one 1 KB load
// accepted per ~200 cycles each: 3.2).
#include <algorithm>

#include "halp_device.hpp"
#include "softmax_ahead.hpp"
#include "softmax_fused.hpp"

namespace halp {
namespace {

typedef int I4 __attribute__((ext_vector_type(4)));
typedef int I2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) I2 LdsI2;
typedef short S2 __attribute__((ext_vector_type(2)));

constexpr int kRows = 64;        // rows of an iteration at most
constexpr int kOwners = 8;   // waves that hold z
constexpr int kScal = 4;     // waves that take the scalars, one per SIMD
constexpr int kManyRows = 32;  // rows of an iteration at most where a step takes several: the sums of the
                               // update stay in registers between them, fewer rows are held ahead
constexpr int kWaves = kOwners + kScal;
constexpr int kNB = 2;       // blocks of 64 coordinates per owner
constexpr int kGamStride = 80;   // bytes per class of the gamma buffer (64 + 16: bank spread)
constexpr size_t kLdsCap = 158 * 1024;

// lane ^ 4 inside rows of 16: banks of four lanes trade places
__device__ __forceinline__ double bank_swap_f64(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  auto mv = [](int x) {
    const int up = __builtin_amdgcn_update_dpp(0, x, 0x104, 0xF, 0x5, false);  // row_shl:4 into banks 0, 2
    return __builtin_amdgcn_update_dpp(up, x, 0x114, 0xF, 0xA, false);          // row_shr:4 into banks 1, 3
  };
  const uint32_t lo = (uint32_t)mv((int)(uint32_t)u), hi = (uint32_t)mv((int)(u >> 32));
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
// lane ^ 8 inside rows of 16
__device__ __forceinline__ double half_swap_f64(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, 0x128, 0xF, 0xF, false);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(u >> 32), 0x128, 0xF, 0xF, false);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// lane r of a quad holds v[0..3] = M[0..3][r]; returns M[r][0..3]
__device__ __forceinline__ void quad_transpose(int (&v)[4], int lane) {
  const bool o1 = (lane & 1) != 0, o2 = (lane & 2) != 0;
#pragma unroll
  for (int k = 0; k < 4; k += 2) {  // pairs of lanes trade the off-diagonal of a 2 x 2 block
    const int t = dpp_quad_swap1(o1 ? v[k] : v[k + 1]);
    if (o1) v[k] = t;
    else v[k + 1] = t;
  }
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int t = dpp_quad_swap2(o2 ? v[k] : v[k + 2]);
    if (o2) v[k] = t;
    else v[k + 2] = t;
  }
}

// rows: rows of an iteration, a multiple of 16.  MANY: a step has more.  AL16: rows and their base are 16-byte aligned.  SOFT:
// softmax, else K = 1 with the squared or logistic loss.
template <bool MANY, bool AL16, bool SOFT>
__global__ __launch_bounds__(64 * kWaves) void inner_softmax_mfma_kernel(InArgs a, Ahead ah, int chain0, int last,
                                                                          int rows) {
  constexpr int QMAX = 127, QMIN = -128;
  constexpr int kR = MANY ? kManyRows : kRows;
  constexpr int kCopy = kR / kOwners;  // rows of an iteration an owner copies
  const int local = blockIdx.x, chain = chain0 + local;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lc = lane & 15, q = lane >> 4;
  const int d = a.d, K = a.K, B = a.B;
  const double* sc = a.scales + (int64_t)chain * 8;
  unsigned long long* cnt_out = reinterpret_cast<unsigned long long*>(a.counters + (int64_t)chain * 4);
  if (sc[7] != 0.0) {  // converged or unusable gradient: the epoch is a no-op
    if (tid < 4) cnt_out[tid] = 0;
    return;
  }
  const int64_t T = epoch_steps(a.seed + (uint64_t)chain, a.epoch, a.T, a.option2);
  const int steps = segment_steps(ah.t0, ah.t1, T);
  const int nblk = (d + 63) / 64;
  const int stride = 64 * nblk + 16;   // bytes between rows in LDS: 4 mod 16 dwords, 16 rows in distinct banks
  const int nchunk = MANY ? (B + rows - 1) / rows : 1;
  const int64_t row_bytes = a.ldxq;

  extern __shared__ __attribute__((aligned(16))) unsigned char s_dyn[];
  unsigned char* s_x = s_dyn;                              // [2][rows][stride]
  I4* s_part = reinterpret_cast<I4*>(s_dyn + 2 * rows * stride);  // [owner][rows / 16][lane] parts of D
  __shared__ __attribute__((aligned(16))) int8_t s_gam[16 * kGamStride];  // gamma, byte (row % 4) 16 + row / 4 of a class
  __shared__ unsigned long long s_cnt[2];
  for (int e = tid; e < 2 * rows * stride / 16; e += 64 * kWaves) reinterpret_cast<I4*>(s_dyn)[e] = I4{0, 0, 0, 0};
  for (int e = tid; e < 16 * kGamStride / 4; e += 64 * kWaves) reinterpret_cast<int*>(s_gam)[e] = 0;
  if (tid < 2) s_cnt[tid] = 0;

  const unsigned char* __restrict__ Xq = reinterpret_cast<const unsigned char*>(a.Xq) + (int64_t)chain * a.xq_chain_stride;
  const AheadRec* __restrict__ rec = ah.rec + (int64_t)local * ah.S * B * kAheadK;
  const int32_t* __restrict__ idx = ah.idx + (int64_t)local * ah.S * B;
  const int32_t* __restrict__ clv = ah.cl + (int64_t)local * ah.S;
  const uint16_t* __restrict__ zst = ah.zbits + (int64_t)local * ah.S * K * ah.UP;
  const double inv_s = sc[5];
  const double dscale = __dmul_rn(a.delta_d, sc[0]);
  const double aB = __ddiv_rn(a.hyper[2 * chain], (double)B);
  const bool lp = a.lp != 0;
  const bool use_reg = a.lambda > 0;

  const int niter = steps * nchunk;
  const bool cls_ok = lc < K;
  const int nown = min(kOwners, nblk);  // owners with a block
  unsigned long long n_zclamp = 0;
  unsigned int n_gclamp = 0, n_reg = 0;
  __syncthreads();  // LDS is cleared

  if (wave >= kOwners) {
    // ============================================================================== scalars
    __builtin_amdgcn_s_setprio(3);  // the owners on this SIMD copy rows meanwhile
    if (steps > 0) {
      const int tile = wave - kOwners;
      // after the exchange lane (q, k = lc / 4, r = lc % 4) holds row 16 tile + 4 q + r, classes 4 k .. 4 k + 3
      const int m0 = 16 * tile + 4 * q + (lc & 3), c0 = lc & 12;
      AheadRec rn[SOFT ? 4 : 1];
      float yn = 0.f;
      // softmax: the short chain to the gammas (softmax_fused.hpp) where the chain's scales allow it.  Four classes
      // per lane here, so that it saves instructions as much as latency: one reciprocal per row for four divisions
      // per lane, no maximum
      const bool fused = SOFT && soft_covers(dscale, aB, inv_s);
      const double k2 = __dmul_rn(aB, inv_s);
      SoftDraw sd[SOFT ? 4 : 1];
      double from[SOFT ? 4 : 1];
      auto draw = [&]() {
        if (fused) {
#pragma unroll
          for (int e = 0; e < (SOFT ? 4 : 1); ++e) {
            const bool live = c0 + e < K;
            sd[e] = soft_draw<false>(live, rn[e].p0, rn[e].phi, rn[e].rho, k2);
            from[e] = lp && live ? (double)rn[e].phi : 0.0;
          }
        }
      };
      auto fetch_rec = [&](AheadRec(&r)[SOFT ? 4 : 1], int it) {
        it = min(it, niter - 1);  // past the segment's end its last rows are repeated
        const int tl = MANY ? it / nchunk : it;
        const int mb = MANY ? (it - tl * nchunk) * rows : 0;
        const int64_t o = ((int64_t)tl * B + min(mb + m0, B - 1)) * kAheadK + c0;
#pragma unroll
        for (int e = 0; e < (SOFT ? 4 : 1); ++e) r[e] = rec[o + e];
        if (!SOFT && a.loss == HALP_LOSS_LOGISTIC) yn = rec[o + 1].phi;
      };
      // The short chain's draws of an iteration are made while the gammas of the one before are used.  With chunks that
      // is not long enough for the trip of the records, which are asked for two iterations ahead there
      const bool far = MANY && fused;
      fetch_rec(rn, 0);
      draw();
      if (far) fetch_rec(rn, 1);
      __syncthreads();
      int ch = 0;
      for (int it = 0; it < niter; ++it) {
        const int nrow = MANY ? min(rows, B - ch * rows) : B;
        lds_barrier();  // the parts of D are in LDS
        if (16 * tile < rows) {
          I4 dv{0, 0, 0, 0};
          {
            I4 part[kOwners];
#pragma unroll
            for (int w = 0; w < kOwners; ++w)  // owners without a block have no part: the first one's, not added
              part[w] = s_part[((w < nown ? w : 0) * (rows >> 4) + tile) * 64 + lane];
#pragma unroll
            for (int w = 0; w < kOwners; ++w)
              if (w < nown) dv += part[w];
          }
          int D[4] = {dv[0], dv[1], dv[2], dv[3]};
          quad_transpose(D, lane);
          // ---- gamma of row m0, classes c0 .. c0 + 3.  Algorithm 4 moves the margins by x^T z; in
          // Algorithm 2 (LP-SVRG) x^T w is the margin
          int8_t* gp = s_gam + c0 * kGamStride + (m0 & 3) * 16 + (m0 >> 2);
          bool done = false;
          if constexpr (SOFT) {
            // NE: classes per lane that may exist (of those past it the gammas are 0 and stay so)
            auto short_chain = [&](auto ne_tag) __attribute__((always_inline)) {
              constexpr int NE = decltype(ne_tag)::value;
              double delta[NE], ex[NE], sum = 0.0;
#pragma unroll
              for (int e = 0; e < NE; ++e) delta[e] = __fma_rn(dscale, (double)D[e], -from[e]);  // 0 past the classes
#pragma unroll
              for (int e = 0; e < NE; ++e) ex[e] = exp_short(delta[e]);
#pragma unroll
              for (int e = 0; e < NE; ++e) sum = __fma_rn(sd[e].p0, ex[e], sum);
              sum += bank_swap_f64(sum);
              sum += half_swap_f64(sum);
              double y = __builtin_amdgcn_rcp(sum);
              y = __fma_rn(__fma_rn(-sum, y, 1.0), y, y);
              bool bad = !(sum > 0x1p-4);
              int hi[NE];
#pragma unroll
              for (int e = 0; e < NE; ++e) {
                const uint64_t bits = __builtin_bit_cast(uint64_t, __fma_rn(sd[e].kp * ex[e], y, sd[e].c));
                hi[e] = (int)(bits >> 32);
                bad = bad || sd[e].wide || !(__builtin_fabs(delta[e]) <= 64.0) || (c0 + e < K && (uint32_t)bits <= 2 * kSoftNear);
              }
              done = __ballot(bad) == 0;
              if (__builtin_expect_with_probability(done, 1, 1.0)) {
#pragma unroll
                for (int e = 0; e < NE; ++e) {
                  const bool in = m0 < nrow && c0 + e < K;
                  const int g = min(max(hi[e], kSoftMagicHi + QMIN), kSoftMagicHi + QMAX);
                  n_gclamp += (in && g != hi[e]) ? 1u : 0u;
                  gp[e * kGamStride] = in ? (int8_t)(g & 0xFF) : (int8_t)0;
                }
              }
            };
            if (fused && MANY && K == 2) short_chain(std::integral_constant<int, MANY ? 2 : 4>{});
            else if (fused) short_chain(std::integral_constant<int, 4>{});
          }
          if (!done) {  // in the fixed order of roundings
            AheadRec rf[SOFT ? 4 : 1];
#pragma unroll
            for (int e = 0; e < (SOFT ? 4 : 1); ++e) rf[e] = rn[e];
            if (far) fetch_rec(rf, it);
            double diff[4];
            if constexpr (SOFT) {
              double v[4], ex[4];
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                const double moved = __dmul_rn(dscale, (double)D[e]);
                v[e] = c0 + e < K ? (lp ? moved : __dadd_rn((double)rf[e].phi, moved)) : -INFINITY;
              }
              double mx = fmax(fmax(v[0], v[1]), fmax(v[2], v[3]));
              mx = fmax(mx, bank_swap_f64(mx));
              mx = fmax(mx, half_swap_f64(mx));
#pragma unroll
              for (int e = 0; e < 4; ++e) ex[e] = c0 + e < K ? halp_exp(__dadd_rn(v[e], -mx)) : 0.0;
              // normaliser: pairwise over adjacent classes
              double sum = __dadd_rn(__dadd_rn(ex[0], ex[1]), __dadd_rn(ex[2], ex[3]));
              sum = __dadd_rn(sum, bank_swap_f64(sum));
              sum = __dadd_rn(sum, half_swap_f64(sum));
#pragma unroll
              for (int e = 0; e < 4; ++e) diff[e] = __dadd_rn(__ddiv_rn(ex[e], sum), -rf[e].p0);
            } else {
              const double a0 = (double)rf[0].phi, moved = __dmul_rn(dscale, (double)D[0]);
              if (a.loss == HALP_LOSS_SQUARED) {
                // Algorithm 4: (phi + Delta - y) - (phi - y) = Delta; Algorithm 2: (x^T w - y) - (phi - y)
                diff[0] = lp ? __dadd_rn(moved, -a0) : moved;
              } else {
                const double y = (double)yn, a1 = lp ? moved : __dadd_rn(a0, moved);
                diff[0] = __dadd_rn(__ddiv_rn(-y, __dadd_rn(1.0, halp_exp(__dmul_rn(y, a1)))), -rf[0].p0);
              }
            }
#pragma unroll
            for (int e = 0; e < (SOFT ? 4 : 1); ++e) {
              const double beta = __dmul_rn(aB, diff[e]);
              const double rho = __dmul_rn((double)rf[e].rho, 0x1p-32);
              const double f = floor(__dadd_rn(__dmul_rn(beta, inv_s), rho));
              const double fc = fmin(fmax(f, (double)QMIN), (double)QMAX);
              const bool in = m0 < nrow && c0 + e < K;
              n_gclamp += (in && f != fc) ? 1u : 0u;
              gp[e * kGamStride] = in ? (int8_t)(int)fc : (int8_t)0;
            }
          }
        }
        lds_barrier();  // gamma is out
        if (far) {
          draw();
          fetch_rec(rn, it + 2);
        } else {
          fetch_rec(rn, it + 1);
          draw();
        }
        if (MANY) ch = ch + 1 == nchunk ? 0 : ch + 1;
      }
    }
  } else {
    // ============================================================================== owners of z
    auto owns = [&](int nb) { return wave + kOwners * nb < nblk; };  // uniform
    // coordinate (j, i) of this lane in its block nb
    auto j_of = [&](int nb, int j) { return 64 * (wave + kOwners * nb) + 32 * (q >> 1) + 8 * j + 4 * (q & 1); };
    const int64_t row0 = ((int64_t)chain * K + (cls_ok ? lc : 0)) * d;
    S2 zp[kNB][8];   // pairs of coordinates: [2 j + i / 2][i % 2]
    // h~ [j][i], where the sums of the products start; with chunks, which keep the sums in
    // registers, two to a register
    I4 hC[MANY ? 1 : kNB][4];
    S2 hP[MANY ? kNB : 1][8];
#pragma unroll
    for (int nb = 0; nb < kNB; ++nb) {
      const int8_t* __restrict__ zg = reinterpret_cast<const int8_t*>(a.z) + row0;
      const int16_t* __restrict__ hg = reinterpret_cast<const int16_t*>(a.h) + row0;
      int zv[16], hv[16];
#pragma unroll
      for (int k = 0; k < 16; ++k) {  // unconditional: all loads in flight at once
        zv[k] = zg[min(j_of(nb, k / 4) + k % 4, d - 1)];
        hv[k] = hg[min(j_of(nb, k / 4) + k % 4, d - 1)];
      }
#pragma unroll
      for (int k = 0; k < 16; ++k) asm volatile("" : "+v"(zv[k]), "+v"(hv[k]));
#pragma unroll
      for (int k = 0; k < 16; ++k) {
        const bool ok = cls_ok && j_of(nb, k / 4) + k % 4 < d;
        zp[nb][k / 2][k % 2] = ok ? (short)zv[k] : (short)0;
        if constexpr (MANY) hP[nb][k / 2][k % 2] = ok ? (short)hv[k] : (short)0;
        else hC[nb][k / 4][k % 4] = ok ? hv[k] : 0;
      }
    }
    auto h_of = [&](int nb, int j) {
      if constexpr (MANY) {
        S2 lo = hP[nb][2 * j], hi = hP[nb][2 * j + 1];
        asm volatile("" : "+v"(lo), "+v"(hi));  // keeps the unpacked form from being carried through the loop
        return I4{(int)lo[0], (int)lo[1], (int)hi[0], (int)hi[1]};
      } else {
        return hC[nb][j];
      }
    };
    if (steps > 0) {
      // ---- rows 8 w .. 8 w + 7 of an iteration, one row per load
      const bool copier = lane < (d + 15) / 16 && kCopy * wave < rows;  // 16-byte chunks that hold coordinates
      const bool ragged = (d & 15) != 0;
      I4 tailm;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int nv = d - (16 * lane + 4 * k);
        tailm[k] = nv >= 4 ? -1 : (nv <= 0 ? 0 : (1 << (8 * nv)) - 1);
      }
      const uint32_t off_lo = (uint32_t)min(16 * (int64_t)lane, row_bytes - (AL16 ? 16 : 8));
      const uint32_t off_hi = (uint32_t)min(16 * (int64_t)lane + 8, row_bytes - 8);
      I4 xr[kCopy];
      int idxn = 0;  // lane i: number of row 8 w + (i & 7) of the next iteration to be requested
      auto fetch_idx = [&](int it) {
        it = min(it, niter - 1);
        const int tl = MANY ? it / nchunk : it;
        const int mb = MANY ? (it - tl * nchunk) * rows : 0;
        idxn = idx[(int64_t)tl * B + min(mb + kCopy * wave + (lane & (kCopy - 1)), B - 1)];
      };
      // the rows whose numbers fetch_idx brought (rows past B repeat the last one and meet a gamma of 0)
      auto request = [&]() {
        const int64_t off = (int64_t)idxn * row_bytes;
        uint32_t o_lo = off_lo, o_hi = off_hi;  // opaque here: a scalar base and a 32-bit lane offset per load
        asm volatile("" : "+v"(o_lo), "+v"(o_hi));
#pragma unroll
        for (int i = 0; i < kCopy; ++i) {
          const uint64_t o = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)off, i) |
                             ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(off >> 32), i) << 32);
          const unsigned char* rp = Xq + o;
          if (AL16) {
            xr[i] = *reinterpret_cast<const I4*>(rp + o_lo);
          } else {
            const uint2 lo = *reinterpret_cast<const uint2*>(rp + o_lo), hi = *reinterpret_cast<const uint2*>(rp + o_hi);
            xr[i] = I4{(int)lo.x, (int)lo.y, (int)hi.x, (int)hi.y};
          }
        }
      };
      unsigned char* const xput = s_x + kCopy * wave * stride + 16 * lane;
      auto stage = [&](int buf) {
        if (copier) {
          unsigned char* p = xput + buf * rows * stride;
          if (ragged) {
#pragma unroll
            for (int i = 0; i < kCopy; ++i) *reinterpret_cast<I4*>(p + i * stride) = xr[i] & tailm;
          } else {
#pragma unroll
            for (int i = 0; i < kCopy; ++i) *reinterpret_cast<I4*>(p + i * stride) = xr[i];
          }
        }
      };
      I4 zbn[kNB];
      int cln = 0;
      const uint16_t* __restrict__ zsl = zst + (cls_ok ? lc : 0) * ah.UP + 8 * q;
      auto fetch_bits = [&](int tl) {
        tl = min(tl, steps - 1);
#pragma unroll
        for (int nb = 0; nb < kNB; ++nb)  // a block past the row: the first block's bits, not used
          zbn[nb] = *reinterpret_cast<const I4*>(zsl + (int64_t)tl * K * ah.UP + (owns(nb) ? 32 * (wave + kOwners * nb) : 0));
        cln = use_reg ? clv[tl] : 0;
      };
      fetch_idx(0);
      request();
      fetch_idx(1);
      stage(0);
      fetch_bits(0);
      request();
      fetch_idx(2);
      __syncthreads();
      I4 G[kNB][4];  // MANY: the sums so far
      int tl = 0, ch = 0;
      const int lane_a = lc * stride + 64 * wave + 16 * q;  // 16 bytes of row lc, this lane's share of a block
      // transposing reads: lanes 2 k, 2 k + 1 of row group q name 8 bytes of row 4 k + q (the second
      // read: 32 rows on), 32 apart: four row groups in different banks.  Rows past the buffer's: its
      // last one, their gamma is 0
      const int lane_t0 = min(4 * (lc >> 1) + q, rows - 1) * stride + 64 * wave + 32 * (lc & 1);
      const int lane_t1 = min(32 + 4 * (lc >> 1) + q, rows - 1) * stride + 64 * wave + 32 * (lc & 1);
      for (int it = 0; it < niter; ++it) {
        const int buf = it & 1;
        const bool first = !MANY || ch == 0, done = !MANY || ch + 1 == nchunk;
        const int cl = cln;
        const unsigned char* xb = s_x + buf * rows * stride;
        // ---- D = X Z over this wave's blocks
        if (owns(0)) {
          I4 zb[kNB];
#pragma unroll
          for (int nb = 0; nb < kNB; ++nb) {
            uint32_t dw[4];  // bytes of coordinates (j, 0..3)
#pragma unroll
            for (int j = 0; j < 4; ++j)
              dw[j] = __builtin_amdgcn_perm(__builtin_bit_cast(uint32_t, zp[nb][2 * j + 1]),
                                            __builtin_bit_cast(uint32_t, zp[nb][2 * j]), 0x06040200u);
            // rows of 16 lanes trade halves: afterwards lane q holds 16 consecutive coordinates, 16 q on
            const auto s0 = __builtin_amdgcn_permlane16_swap(dw[0], dw[2], false, false);
            const auto s1 = __builtin_amdgcn_permlane16_swap(dw[1], dw[3], false, false);
            zb[nb] = I4{(int)s0[0], (int)s0[1], (int)s1[0], (int)s1[1]};
          }
          constexpr int kT = kR / 16;
          I4 xa[kT], acc[kT];  // all reads of a block in flight at once (tiles past the buffer repeat its last)
#pragma unroll
          for (int t = 0; t < kT; ++t) xa[t] = *reinterpret_cast<const I4*>(xb + min(16 * t, rows - 16) * stride + lane_a);
#pragma unroll
          for (int t = 0; t < kT; ++t) acc[t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(xa[t], zb[0], I4{0, 0, 0, 0}, 0, 0, 0);
          if (owns(1)) {
#pragma unroll
            for (int t = 0; t < kT; ++t)
              xa[t] = *reinterpret_cast<const I4*>(xb + min(16 * t, rows - 16) * stride + lane_a + 64 * kOwners);
#pragma unroll
            for (int t = 0; t < kT; ++t) acc[t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(xa[t], zb[1], acc[t], 0, 0, 0);
          }
#pragma unroll
          for (int t = 0; t < kT; ++t)
            if (16 * t < rows) s_part[(wave * (rows >> 4) + t) * 64 + lane] = acc[t];
        }
        lds_barrier();   // the parts of D are in LDS
        stage(buf ^ 1);  // rows of the next iteration, requested an iteration ago
        request();       // rows of the one after it
        fetch_idx(it + 3);
        lds_barrier();   // gamma is out, the next rows are in LDS
        const I4 gam = *reinterpret_cast<const I4*>(s_gam + lc * kGamStride + 16 * q);
        I4 op[4];
        auto read_block = [&](int nb) {  // this lane's share of a block: rows q + 4 k, transposed
          const unsigned char* xt = xb + 64 * kOwners * nb;
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const I2 lo = __builtin_amdgcn_ds_read_tr8_b64_v2i32((LdsI2*)(xt + lane_t0 + 8 * j));
            const I2 hi = __builtin_amdgcn_ds_read_tr8_b64_v2i32((LdsI2*)(xt + lane_t1 + 8 * j));
            op[j] = I4{lo[0], lo[1], hi[0], hi[1]};
          }
        };
        if (owns(0)) read_block(0);
#pragma unroll
        for (int nb = 0; nb < kNB; ++nb) {
          if (owns(nb)) {
            // ---- G = X^T Gamma
            if (MANY && nb > 0) read_block(nb);
            if (MANY && first) {
#pragma unroll
              for (int j = 0; j < 4; ++j) G[nb][j] = h_of(nb, j);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j)
              G[nb][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(op[j], gam, MANY ? G[nb][j] : h_of(nb, j), 0, 0, 0);
            if (!MANY && nb + 1 < kNB && owns(nb + 1)) read_block(nb + 1);  // in flight through this block's update
            // ---- u = z - sum_m gamma_m x_m - h~ (- c_lambda z) in (delta_i, 2b); z = Q_(delta_m, b)(u)
            auto update = [&](auto with_l2) {
              const auto r0 = __builtin_amdgcn_permlane16_swap((uint32_t)zbn[nb][0], (uint32_t)zbn[nb][1], false, false);
              const auto r1 = __builtin_amdgcn_permlane16_swap((uint32_t)zbn[nb][2], (uint32_t)zbn[nb][3], false, false);
              const uint32_t rb[4] = {r0[0], r1[0], r0[1], r1[1]};  // rounding bits of coordinates (j, 0..3)
              S2 vu[8];
              uint32_t hit = 0;
#pragma unroll
              for (int p = 0; p < 8; ++p) {  // coordinates (p / 2, 2 (p % 2) + {0, 1})
                int v[2];
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                  const int i = 2 * (p % 2) + e;
                  v[e] = (int)((rb[p / 2] >> (8 * i)) & 0xFFu) - G[nb][p / 2][i];
                  if (decltype(with_l2)::value) v[e] = mad24(-cl, (int)zp[nb][p][e], v[e]);
                }
                S2 zn;
                if (MANY) {  // up to 512 products: the shifted sum may leave 16 bits before the clamp
                  const S2 zo = zp[nb][p];
                  const int u0 = (int)zo[0] + (v[0] >> 8), u1 = (int)zo[1] + (v[1] >> 8);
                  const int c0 = min(max(u0, QMIN), QMAX), c1 = min(max(u1, QMIN), QMAX);
                  zn = S2{(short)c0, (short)c1};
                  vu[p] = S2{(short)(c0 ^ (u0 != c0)), (short)(c1 ^ (u1 != c1))};
                } else {  // |v| < 2^23: bytes 1 and 2 are floor(v / 256)
                  const uint32_t sh = __builtin_amdgcn_perm((uint32_t)v[1], (uint32_t)v[0], 0x06050201u);
                  vu[p] = __builtin_bit_cast(S2, sh) + zp[nb][p];
                  zn = __builtin_elementwise_min(__builtin_elementwise_max(vu[p], (S2)(QMIN)), (S2)(QMAX));
                }
                hit |= __builtin_bit_cast(uint32_t, vu[p]) ^ __builtin_bit_cast(uint32_t, zn);
                zp[nb][p] = zn;
              }
              if (__ballot(hit != 0) != 0) {  // rare: count the clamped coordinates exactly
#pragma unroll
                for (int p = 0; p < 8; ++p) {
                  const uint32_t df = __builtin_bit_cast(uint32_t, vu[p]) ^ __builtin_bit_cast(uint32_t, zp[nb][p]);
                  n_zclamp += (unsigned long long)__builtin_popcountll(__ballot((df & 0xFFFFu) != 0)) +
                              (unsigned long long)__builtin_popcountll(__ballot((df >> 16) != 0));
                }
              }
            };
            if (done) {
              if (cl == 0) update(std::false_type{});
              else update(std::true_type{});  // the L2 term is rare: c_lambda is mostly 0
            }
          }
        }
        if (done) {
          n_reg += cl != 0 ? 1u : 0u;
          fetch_bits(tl + 1);
        }
        if (MANY && !done) {
          ++ch;
        } else {
          ch = 0;
          ++tl;
        }
      }
    }

    // ---- hand z out; after the epoch's last segment w~ <- w~ + delta_m z (Algorithm 2: w~ = delta z)
    const double delta_m = sc[0];
    int8_t* __restrict__ zo = reinterpret_cast<int8_t*>(a.z) + row0;
    float* __restrict__ wo = a.w + row0;
#pragma unroll
    for (int nb = 0; nb < kNB; ++nb) {
      int jl = j_of(nb, 0);
      asm volatile("" : "+v"(jl));  // keeps the addresses below from being carried through the loop
      auto at = [&](int k) { return jl + 8 * (k / 4) + k % 4; };
      float wv[16];
#pragma unroll
      for (int k = 0; k < 16; ++k) wv[k] = wo[min(at(k), d - 1)];
#pragma unroll
      for (int k = 0; k < 16; ++k) asm volatile("" : "+v"(wv[k]));  // all loads in flight at once
#pragma unroll
      for (int k = 0; k < 16; ++k) {
        if (cls_ok && at(k) < d) {
          const int zk = (int)zp[nb][k / 2][k % 2];
          zo[at(k)] = (int8_t)zk;
          if (last) {
            const double step = __dmul_rn(delta_m, (double)zk);
            wo[at(k)] = lp ? (float)step : (float)__dadd_rn((double)wv[k], step);
          }
        }
      }
    }
  }
  if (lane == 0 && n_zclamp) atomicAdd(&s_cnt[0], n_zclamp);
  if (n_gclamp) atomicAdd(&s_cnt[1], (unsigned long long)n_gclamp);
  __syncthreads();
  if (tid == 0) {  // the segments of an epoch follow each other on the stream
    const bool begin = ah.t0 == 0;
    cnt_out[0] = (begin ? 0 : cnt_out[0]) + s_cnt[0];
    cnt_out[1] = (begin ? 0 : cnt_out[1]) + s_cnt[1];
    cnt_out[2] = (begin ? 0 : cnt_out[2]) + n_reg;
    cnt_out[3] = 0;
  }
}

int mfma_up(const halp_params& p) { return 32 * ((p.d + 63) / 64); }  // strips per class in the records

// LDS of an iteration of `rows` rows: two buffers of them, and the owners' parts of D
size_t mfma_lds(int d, int rows) {
  const int nblk = (d + 63) / 64;
  return (size_t)2 * rows * (64 * nblk + 16) + (size_t)std::min(nblk, kOwners) * rows * 64;
}

// rows of an iteration: all of a step's, in sixteens, where they are at most 64 and fit LDS, else 32
int mfma_rows(int d, int B) {
  const int rows = (B + 15) / 16 * 16;
  return rows <= kRows && mfma_lds(d, rows) <= kLdsCap ? rows : kManyRows;
}

// 8 bits, rows up to 1024 coordinates (16 blocks of 64 over eight waves, two buffers of 64 rows in LDS)
bool mfma_shape(const halp_params& p) {
  if (p.algorithm == HALP_ALG_SVRG || p.b != 8 || p.d > 1024 || p.K > 16 || p.B < 2 || p.B > 512) return false;
  return p.loss == HALP_LOSS_SOFTMAX ? p.K >= 2 : p.B > 64;
}

template <bool MANY, bool AL16, bool SOFT>
int launch_one(const InArgs& a, const Ahead& s, int c0, int chains, int last, hipStream_t st) {
  const int rows = mfma_rows(a.d, a.B);
  const size_t smem = mfma_lds(a.d, rows);
  auto kern = inner_softmax_mfma_kernel<MANY, AL16, SOFT>;
  if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                          (int)smem) != hipSuccess)
    return HALP_ERR_HIP;
  hipLaunchKernelGGL(kern, dim3(chains), dim3(64 * kWaves), smem, st, a, s, c0, last, rows);
  return hip_ok(hipGetLastError());
}

}  // namespace

// one workgroup per CU: twelve waves with the registers of three per SIMD
size_t plan_inner_softmax_mfma(halp_handle& h) {
  return mfma_shape(h.p) ? plan_ahead(h, mfma_up(h.p), h.num_cus) : 0;
}

int inner_softmax_mfma_supported(const halp_handle& h) {
  if (!mfma_shape(h.p)) return HALP_ERR_UNSUPPORTED;
  return (!h.bound || !h.buf.Xq || (!h.ahead_ws && !h.ahead_pending)) ? HALP_ERR_NOT_BOUND : HALP_OK;
}

int launch_inner_softmax_mfma(const halp_handle& h, uint32_t epoch, hipStream_t st) {
  const halp_params& p = h.p;
  const int rc = inner_softmax_mfma_supported(h);
  if (rc != HALP_OK) return rc;
  if (!h.ahead_ws) return HALP_ERR_UNSUPPORTED;  // the full-step form has the shape
  const InArgs a = make_inner_args(h, epoch);
  const bool many = p.B > mfma_rows(p.d, p.B), soft = p.loss == HALP_LOSS_SOFTMAX;
  const bool al16 = h.buf.ldxq % 16 == 0 && reinterpret_cast<uintptr_t>(h.buf.Xq) % 16 == 0;
  return for_segments(a, h, mfma_up(p), false, st, [&](const Ahead& s, int c0, int chains, int last) -> int {
#define HALP_MF(MANY_, AL_, SOFT_) \
  if (many == MANY_ && al16 == AL_ && soft == SOFT_) return launch_one<MANY_, AL_, SOFT_>(a, s, c0, chains, last, st);
    HALP_MF(false, true, true) HALP_MF(false, false, true) HALP_MF(true, true, true) HALP_MF(true, false, true)
    HALP_MF(true, true, false) HALP_MF(true, false, false)  // one class: more than 64 rows only
#undef HALP_MF
    return HALP_ERR_UNSUPPORTED;
  });
}

}  // namespace halp
