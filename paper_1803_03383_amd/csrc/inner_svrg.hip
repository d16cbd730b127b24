// Inner loop of full-precision SVRG (Algorithm 1) for linear models, one sampled row per
// step: the comparator the paper times HALP against (its Table 3), on the same index stream
// and with the same launch structure as the low-precision inner loop.
//
//   w <- w - alpha ( (l'(x_i^T w) - l'(phi_i)) x_i + lambda (w - w~) + g~ ),   phi_i = x_i^T w~
//
// One workgroup per chain.  inner_svrg_kernel: a thread owns CPL consecutive coordinates of w (fp32 registers)
// together with alpha g~ and w~; rows of the fp32 data are gathered in windows of 8 steps, the
// next window's fragments being requested at the top of the current one.  Vector work is
// fp32 (fused multiply-adds), the scalar l' difference fp64, the wave sums DPP folds, the
// cross-wave sum one LDS word per wave added in wave order.  Sample indices (and the margins
// and labels of the sampled rows) are produced 256 steps at a time into LDS.
#include <type_traits>

#include "halp_device.hpp"
#include "halp_internal.hpp"

namespace halp {
namespace {

constexpr int kBatch = 256;
constexpr int kWin = 8;

struct SvArgs {
  const float* X;    // [Rd][N][ldx]
  const float* y;    // [Rd][N]
  const float* phi;  // [R][N]
  const float* g;    // [R][d]
  float* w;          // [R][d] in: w~, out: w_T
  int64_t N, ldx, T;
  int64_t x_chain_stride, y_chain_stride;
  int d, loss;
  int option2;
  const double* hyper;  // [R][2] step size (and mu, unused here) of each chain
  double lambda;
  uint64_t seed;
  uint32_t epoch;
};

__device__ __forceinline__ double logistic_dl(double a, double y) {
  return __ddiv_rn(-y, __dadd_rn(1.0, halp_exp(__dmul_rn(y, a))));
}

template <int CPL, int NWT, int LOSS>
__global__ __launch_bounds__(64 * NWT) void inner_svrg_kernel(SvArgs a) {
  const int chain = blockIdx.x;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = NWT > 1 ? tid >> 6 : 0;
  const int d = a.d;
  const uint32_t N = (uint32_t)a.N;
  const int64_t T = epoch_steps(a.seed + (uint64_t)blockIdx.x, a.epoch, a.T, a.option2);
  const float* __restrict__ X = a.X + (int64_t)chain * a.x_chain_stride;
  const float* __restrict__ y = a.y + (int64_t)chain * a.y_chain_stride;
  const float* __restrict__ phi = a.phi + (int64_t)chain * a.N;
  const float* __restrict__ g = a.g + (int64_t)chain * d;
  float* __restrict__ wg = a.w + (int64_t)chain * d;
  const uint64_t seed = a.seed + (uint64_t)chain;
  constexpr bool logistic = LOSS == HALP_LOSS_LOGISTIC;
  constexpr int kMask = 2 * kBatch - 1;

  __shared__ __attribute__((aligned(16))) int s_idx[2 * kBatch];
  __shared__ __attribute__((aligned(16))) float s_phi[2 * kBatch];
  __shared__ __attribute__((aligned(16))) float s_y[2 * kBatch];
  __shared__ float s_part[2][16];
  __shared__ float s_dump[NWT > 1 ? 64 * NWT : 1];
  using LdsF = __attribute__((address_space(3))) float;
  LdsF* const slot0 = (LdsF*)((NWT > 1 && lane != 63) ? &s_dump[tid] : &s_part[0][wave]);
  LdsF* const slot1 = (LdsF*)((NWT > 1 && lane != 63) ? &s_dump[tid] : &s_part[1][wave]);

  // ---- per-thread state; coordinates past d hold zeros and never change
  const int j0 = tid * CPL;
  // Rows are padded to a multiple of 4 floats, so the fragment at j0 < d lies inside the row
  // even when it runs past d (the excess is masked); threads past the row re-read its start.
  const int jc = j0 < d ? j0 : 0;
  const double alpha = a.hyper[2 * chain];
  float w[CPL], wt[CPL], ag[CPL];
  bool keep[CPL];
#pragma unroll
  for (int k = 0; k < CPL; ++k) {
    const bool ok = j0 + k < d;
    const int j = min(j0 + k, d - 1);
    w[k] = wt[k] = ok ? wg[j] : 0.f;
    ag[k] = ok ? (float)__dmul_rn(alpha, (double)g[j]) : 0.f;
    keep[k] = ok;
  }
  const float al = (float)__dmul_rn(alpha, a.lambda);
  const bool use_reg = a.lambda > 0;

  auto fill_batch = [&](int64_t bb) {
    const int half = (int)(bb & 1) * kBatch;
    if (tid < 64) {
      const U4 ri = stream_block(seed, kIdx, a.epoch, (uint64_t)bb * 64 + (uint64_t)tid);
      int4 iv;
      iv.x = (int)__umulhi(ri.x, N); iv.y = (int)__umulhi(ri.y, N);
      iv.z = (int)__umulhi(ri.z, N); iv.w = (int)__umulhi(ri.w, N);
      *reinterpret_cast<int4*>(&s_idx[half + 4 * tid]) = iv;
      float4 pv;
      pv.x = phi[iv.x]; pv.y = phi[iv.y]; pv.z = phi[iv.z]; pv.w = phi[iv.w];
      *reinterpret_cast<float4*>(&s_phi[half + 4 * tid]) = pv;
      if (logistic) {
        float4 yv;
        yv.x = y[iv.x]; yv.y = y[iv.y]; yv.z = y[iv.z]; yv.w = y[iv.w];
        *reinterpret_cast<float4*>(&s_y[half + 4 * tid]) = yv;
      }
    }
  };
  fill_batch(0);
  fill_batch(1);
  __syncthreads();

  // ---- row fragments: two buffers of one window each.  Any step number names a valid row
  // (the index batches are whole), so every load is unconditional.
  float xa[kWin][CPL], xb[kWin][CPL];
  auto request = [&](float (&dst)[CPL], int i) {
    const float* rp = X + (int64_t)i * a.ldx + jc;
    if (CPL == 1) {
      dst[0] = rp[0];
    } else if (CPL == 2) {
      const float2 v = *reinterpret_cast<const float2*>(rp);
      dst[0] = v.x; dst[CPL > 1 ? 1 : 0] = v.y;
    } else {
      const float4 v = *reinterpret_cast<const float4*>(rp);
      dst[0] = v.x; dst[CPL > 1 ? 1 : 0] = v.y; dst[CPL > 2 ? 2 : 0] = v.z; dst[CPL > 3 ? 3 : 0] = v.w;
    }
  };
#pragma unroll
  for (int s = 0; s < kWin; ++s) request(xa[s], __builtin_amdgcn_readfirstlane(s_idx[s]));

  auto window = [&](int64_t t0, float (&xr)[kWin][CPL], float (&xnext)[kWin][CPL]) {
    const int base = (int)(t0 & kMask);
    float phi8[kWin], y8[kWin];
    int nidx[kWin];
    {
      const float4 p0 = *reinterpret_cast<const float4*>(&s_phi[base]);
      const float4 p1 = *reinterpret_cast<const float4*>(&s_phi[base + 4]);
      phi8[0] = p0.x; phi8[1] = p0.y; phi8[2] = p0.z; phi8[3] = p0.w;
      phi8[4] = p1.x; phi8[5] = p1.y; phi8[6] = p1.z; phi8[7] = p1.w;
#pragma unroll
      for (int s = 0; s < kWin; ++s) y8[s] = 0.f;
      if (logistic) {
        const float4 y0 = *reinterpret_cast<const float4*>(&s_y[base]);
        const float4 y1 = *reinterpret_cast<const float4*>(&s_y[base + 4]);
        y8[0] = y0.x; y8[1] = y0.y; y8[2] = y0.z; y8[3] = y0.w;
        y8[4] = y1.x; y8[5] = y1.y; y8[6] = y1.z; y8[7] = y1.w;
      }
      const int nb = (base + kWin) & kMask;
      const int4 i0 = *reinterpret_cast<const int4*>(&s_idx[nb]);
      const int4 i1 = *reinterpret_cast<const int4*>(&s_idx[nb + 4]);
      nidx[0] = i0.x; nidx[1] = i0.y; nidx[2] = i0.z; nidx[3] = i0.w;
      nidx[4] = i1.x; nidx[5] = i1.y; nidx[6] = i1.z; nidx[7] = i1.w;
    }
    // this window's fragments leave the load buffer (masked) before the next ones are requested
    float xw[kWin][CPL];
#pragma unroll
    for (int s = 0; s < kWin; ++s)
#pragma unroll
      for (int k = 0; k < CPL; ++k) xw[s][k] = keep[k] ? xr[s][k] : 0.f;
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < kWin; ++s) request(xnext[s], __builtin_amdgcn_readfirstlane(nidx[s]));

#pragma unroll
    for (int s = 0; s < kWin; ++s) {
      if (t0 + s < T) {
        float part = 0.f;
#pragma unroll
        for (int k = 0; k < CPL; ++k) part = __builtin_fmaf(xw[s][k], w[k], part);
        // several waves: lane 63, where the fold leaves the sum, stores it; the other lanes store
        // into a dump row, so that no lane mask is set up and no lane is read
        float dot = NWT > 1 ? wave_fold_f32(part) : wave_sum_f32(part);
        if (NWT > 1) {
          *((s & 1) ? slot1 : slot0) = dot;
          __syncthreads();
          float tot = 0.f;
#pragma unroll
          for (int w2 = 0; w2 < NWT; ++w2) tot += s_part[s & 1][w2];
          dot = tot;
        }
        // alpha (l'(x_i^T w) - l'(phi_i)): the scalar path in fp64
        const double a1 = (double)dot, a0 = (double)phi8[s];
        double diff;
        if (logistic) diff = __dadd_rn(logistic_dl(a1, (double)y8[s]), -logistic_dl(a0, (double)y8[s]));
        else diff = __dadd_rn(a1, -a0);  // (a1 - y) - (a0 - y)
        const float c = (float)__dmul_rn(alpha, diff);
#pragma unroll
        for (int k = 0; k < CPL; ++k) {
          float u = __builtin_fmaf(-c, xw[s][k], w[k]) - ag[k];
          if (use_reg) u = __builtin_fmaf(-al, w[k] - wt[k], u);
          w[k] = u;
        }
      }
    }
  };

  int64_t t0 = 0;
  for (; t0 < T; t0 += 2 * kWin) {
    if ((t0 & (kBatch - 1)) == 0 && t0 > 0) {  // batch t0/256 - 1 is finished: refill its half
      __syncthreads();
      fill_batch(t0 / kBatch + 1);
      __syncthreads();
    }
    window(t0, xa, xb);
    if (t0 + kWin < T) window(t0 + kWin, xb, xa);
  }

  // ---- w~ <- w_T (option I)
#pragma unroll
  for (int k = 0; k < CPL; ++k)
    if (j0 + k < d) wg[j0 + k] = w[k];
}

// The form for few chains per CU: ONE chain wave that holds all of w, helper waves on the other SIMDs.
//
// Such a chain is bound by its step's dependent instructions (8 cycles each on a lone wave) and, in the form
// above, by the LDS exchange and the barrier between its waves in every step.  Here the chain wave adds up x^T w
// alone: DPP over 16 lanes in fp32, then one fp64 4x4x4 matrix instruction across the four rows of lanes, which for
// squared loss also takes the step size and the margin along (-alpha x^T w + alpha phi_i).  w - alpha g~ (and the L2
// term) is taken while the dot is under way, so that one multiply-add per coordinate follows it.  Helper wave v
// fetches the float4s 4 (lane + 64 v) of the sampled rows, kSets - 1 windows of 8 steps ahead, clears what lies
// past d and puts them into a ring of three windows in LDS; the service wave refills the 256-step batches of
// indices, margins, labels.  One barrier per window: in period w the chain wave consumes window w while the helpers
// store window w + 2.
constexpr int kSvSlots = 3;
constexpr int sv_waves(int nv) { return nv == 1 ? 3 : (nv == 2 ? 4 : 7); }

typedef float float4r __attribute__((ext_vector_type(4)));

// NV: float4s of w per lane.  PAIR: built for two workgroups per CU, at most 128 registers.
template <int NV, int LOSS, bool PAIR>
__global__ __launch_bounds__(64 * sv_waves(NV), PAIR ? 4 : 2) void inner_svrg_lone_kernel(SvArgs a) {
  constexpr bool logistic = LOSS == HALP_LOSS_LOGISTIC;
  constexpr int kMask = 2 * kBatch - 1;
  constexpr int kSets = PAIR ? 3 : 4;  // windows of rows a helper has in flight
  const int chain = blockIdx.x;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int d = a.d;
  const uint32_t N = (uint32_t)a.N;
  const uint64_t seed = a.seed + (uint64_t)chain;
  const int64_t T = epoch_steps(seed, a.epoch, a.T, a.option2);
  const int64_t nwin = (T + kWin - 1) / kWin;
  const double alpha = a.hyper[2 * chain];

  __shared__ __attribute__((aligned(16))) int s_idx[2 * kBatch];
  // squared loss: alpha phi_i; logistic: l'(phi_i) and the label
  __shared__ __attribute__((aligned(16))) double s_at[2 * kBatch];
  __shared__ __attribute__((aligned(16))) float s_y[logistic ? 2 * kBatch : 4];
  extern __shared__ __attribute__((aligned(16))) float4r s_row[];  // [slot][step][v][lane]

  // waves w and w + 4 share a SIMD, wave 4 only keeps the barriers
  const int helper = wave == 1 || wave == 2 ? wave - 1 : (NV == 4 && (wave == 5 || wave == 6) ? wave - 3 : -1);
  if (wave == (NV == 1 ? 2 : 3)) {
    // ============================ service wave ============================
    const float* __restrict__ phi = a.phi + (int64_t)chain * a.N;
    const float* __restrict__ y = a.y + (int64_t)chain * a.y_chain_stride;
    auto fill_batch = [&](int64_t bb) {
      const int at = (int)(bb & 1) * kBatch + 4 * lane;
      const U4 ri = stream_block(seed, kIdx, a.epoch, (uint64_t)bb * 64 + (uint64_t)lane);
      int4 iv;
      iv.x = (int)__umulhi(ri.x, N); iv.y = (int)__umulhi(ri.y, N);
      iv.z = (int)__umulhi(ri.z, N); iv.w = (int)__umulhi(ri.w, N);
      *reinterpret_cast<int4*>(&s_idx[at]) = iv;
      const float pv[4] = {phi[iv.x], phi[iv.y], phi[iv.z], phi[iv.w]};
      if constexpr (logistic) {
        const float yv[4] = {y[iv.x], y[iv.y], y[iv.z], y[iv.w]};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          s_y[at + k] = yv[k];
          s_at[at + k] = logistic_dl((double)pv[k], (double)yv[k]);
        }
      } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) s_at[at + k] = __dmul_rn(alpha, (double)pv[k]);
      }
    };
    fill_batch(0);
    __syncthreads();  // P0: the first batch is in place
    __syncthreads();  // P1: windows 0 and 1 are in the ring
    for (int64_t w = 0; w < nwin; ++w) {
      // window w = 32 m: every reader has left batch m - 1, whose half takes batch m + 1 (the first to read indices out
      // of it are the helpers in period 32 m + 27 or later; an epoch that ends before then has nobody who does)
      if ((w & (kBatch / kWin - 1)) == 0) fill_batch(w / (kBatch / kWin) + 1);
      __syncthreads();
    }
    return;
  }

  if (helper >= 0 && helper < NV) {
    // ============================ helper wave =============================
    const int c0 = 4 * (lane + 64 * helper);  // first coordinate
    const uint64_t row_bytes = (uint64_t)a.ldx * 4;
    // rows are padded to a multiple of 4 floats: a float4 that starts inside the row ends inside it; lanes
    // past the row re-read its start
    const unsigned char* const frag = reinterpret_cast<const unsigned char*>(a.X + (int64_t)chain * a.x_chain_stride + (c0 < d ? c0 : 0));
    const bool whole = __ballot(c0 + 3 >= d) == 0;  // every coordinate of this wave exists
    auto request = [&](float4r (&dst)[kWin], int64_t win) {
      const int base = (int)((win * kWin) & kMask);
      const int4 i0 = *reinterpret_cast<const int4*>(&s_idx[base]);
      const int4 i1 = *reinterpret_cast<const int4*>(&s_idx[base + 4]);
      const int iv[kWin] = {i0.x, i0.y, i0.z, i0.w, i1.x, i1.y, i1.z, i1.w};
#pragma unroll
      for (int s = 0; s < kWin; ++s) {
        const unsigned char* at = frag + (uint64_t)(uint32_t)iv[s] * (uint32_t)row_bytes;
        if (row_bytes >> 32) at += (uint64_t)(uint32_t)iv[s] * (uint32_t)(row_bytes >> 32) << 32;  // uniform
        dst[s] = *reinterpret_cast<const float4r*>(at);
      }
    };
    auto store = [&](const float4r (&src)[kWin], int slot) {
#pragma unroll
      for (int s = 0; s < kWin; ++s) {
        float4r v = src[s];
        if (!whole) {
#pragma unroll
          for (int k = 0; k < 4; ++k) v[k] = c0 + k < d ? v[k] : 0.f;
        }
        s_row[((slot * kWin + s) * NV + helper) * 64 + lane] = v;
      }
    };
    float4r f[kSets][kWin];  // window v in set v % kSets
    __syncthreads();  // P0
#pragma unroll
    for (int v = 0; v < kSets; ++v) request(f[v], v);
    store(f[0], 0);
    request(f[0], kSets);
    store(f[1], 1);
    __syncthreads();  // P1
    int slot = 2;
    // period w: the rows of window w + 1 + kSets go into the set window w + 1 left, window w + 2 into the ring
    // (nothing may be scheduled across the borders of a period: the loads of all sets would be waited for)
    auto period = [&](int64_t w, float4r (&freq)[kWin], const float4r (&fuse)[kWin]) {
      __builtin_amdgcn_sched_barrier(0);
      request(freq, w + 1 + kSets);
      __builtin_amdgcn_sched_barrier(0);
      store(fuse, slot);
      slot = slot == kSvSlots - 1 ? 0 : slot + 1;
      // LDS only: the rows in flight are not waited for
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
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
    return;
  }

  if (wave != 0) {
    // ============================== idle wave ==============================
    __syncthreads();
    __syncthreads();
    for (int64_t w = 0; w < nwin; ++w) __syncthreads();
    return;
  }

  // ============================== chain wave ==============================
  const float* __restrict__ g = a.g + (int64_t)chain * d;
  float* __restrict__ wg = a.w + (int64_t)chain * d;
  float wv[4 * NV], ag[4 * NV], wt[4 * NV];  // coordinates past d hold zeros and never change
#pragma unroll
  for (int k = 0; k < 4 * NV; ++k) {
    const int j = 4 * (lane + 64 * (k / 4)) + k % 4;
    wv[k] = wt[k] = j < d ? wg[j] : 0.f;
    ag[k] = j < d ? (float)__dmul_rn(alpha, (double)g[j]) : 0.f;
  }
  const float al = (float)__dmul_rn(alpha, a.lambda);
  __syncthreads();  // P0
  __syncthreads();  // P1
  __builtin_amdgcn_s_setprio(3);

  struct Step {  // what a step needs from LDS, requested two steps ahead (logistic: one)
    float4r x[NV];
    double at;
    float y;
  };
  constexpr int kAhead = logistic ? 1 : 2;
  auto load_step = [&](Step& st, int slot, int base, int s) __attribute__((always_inline)) {
#pragma unroll
    for (int v = 0; v < NV; ++v) st.x[v] = s_row[((slot * kWin + s) * NV + v) * 64 + lane];
    st.at = s_at[base + s];
    if constexpr (logistic) st.y = s_y[base + s];
  };
  auto step = [&](const Step& st, auto reg_tag, auto&& prefetch) __attribute__((always_inline)) {
    constexpr int NA = 4;  // partial sums of a lane
    float p[NA];
#pragma unroll
    for (int k = 0; k < NA; ++k) p[k] = st.x[0][k] * wv[k];
#pragma unroll
    for (int k = NA; k < 4 * NV; ++k) p[k % NA] = __builtin_fmaf(st.x[k / 4][k % 4], wv[k], p[k % NA]);
    float v = (p[0] + p[1]) + (p[2] + p[3]);
    v += dpp_quad_swap1(v);
    v += dpp_quad_swap2(v);
    v += dpp_half_mirror(v);
    v += dpp_row_mirror(v);
    // -alpha (l'(x_i^T w) - l'(phi_i))
    const double row = (double)v;
    double t = logistic ? __builtin_amdgcn_mfma_f64_4x4x4f64(row, 1.0, 0.0, 0, 0, 0)
                        : __builtin_amdgcn_mfma_f64_4x4x4f64(row, -alpha, st.at, 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
    prefetch();
#pragma unroll
    for (int k = 0; k < 4 * NV; ++k) {
      const float moved = wv[k] - ag[k];
      if constexpr (decltype(reg_tag)::value) wv[k] = __builtin_fmaf(-al, wv[k] - wt[k], moved);
      else wv[k] = moved;
    }
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (logistic) t = __dmul_rn(-alpha, __dadd_rn(logistic_dl(t, (double)st.y), -st.at));
    const float c = (float)t;
#pragma unroll
    for (int k = 0; k < 4 * NV; ++k) wv[k] = __builtin_fmaf(c, st.x[k / 4][k % 4], wv[k]);
  };
  auto run = [&](auto reg_tag) __attribute__((always_inline)) {
    int slot = 0;
    int64_t t0 = 0;
    Step ahead[kAhead];
#pragma unroll
    for (int k = 0; k < kAhead; ++k) load_step(ahead[k], 0, 0, k);
    for (; t0 + kWin <= T; t0 += kWin) {
      const int base = (int)(t0 & kMask), next_base = (base + kWin) & kMask;  // (any window has its place in the ring)
      const int next_slot = slot == kSvSlots - 1 ? 0 : slot + 1;
#pragma unroll
      for (int s = 0; s < kWin; ++s) {
        const Step st = ahead[s % kAhead];
        step(st, reg_tag, [&]() __attribute__((always_inline)) {
          if (s + kAhead < kWin) load_step(ahead[s % kAhead], slot, base, s + kAhead);
          else load_step(ahead[s % kAhead], next_slot, next_base, s + kAhead - kWin);
        });
      }
      // the window is consumed, the one after the next is in place; nothing of this wave is waited for
      asm volatile("s_barrier" ::: "memory");
      slot = next_slot;
    }
    if (t0 < T) {
      const int base = (int)(t0 & kMask);
#pragma unroll 1
      for (int s = 0; t0 + s < T; ++s) {
        Step st;
        load_step(st, slot, base, s);
        step(st, reg_tag, []() {});
      }
      asm volatile("s_barrier" ::: "memory");
    }
  };
  if (a.lambda > 0) run(std::true_type{});
  else run(std::false_type{});

  // ---- w~ <- w_T (option I)
#pragma unroll
  for (int k = 0; k < 4 * NV; ++k) {
    const int j = 4 * (lane + 64 * (k / 4)) + k % 4;
    if (j < d) wg[j] = wv[k];
  }
}

template <int NV, bool PAIR>
int launch_lone(const SvArgs& a, int R, hipStream_t s) {
  const dim3 grid(R), block(64 * sv_waves(NV));
  const size_t smem = (size_t)kSvSlots * kWin * NV * 64 * sizeof(float4r);
#define HALP_SVL(LOSS_)                                                                                   \
  do {                                                                                                    \
    auto kern = inner_svrg_lone_kernel<NV, LOSS_, PAIR>;                                                  \
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, \
                            (int)smem) != hipSuccess)                                                     \
      return HALP_ERR_HIP;                                                                                \
    hipLaunchKernelGGL(kern, grid, block, smem, s, a);                                                    \
  } while (0)
  if (a.loss == HALP_LOSS_LOGISTIC) HALP_SVL(HALP_LOSS_LOGISTIC);
  else HALP_SVL(HALP_LOSS_SQUARED);
#undef HALP_SVL
  return hip_ok(hipGetLastError());
}

template <int CPL, int NWT>
int launch_loss(const SvArgs& a, int R, hipStream_t s) {
  const dim3 grid(R), block(64 * NWT);
  if (a.loss == HALP_LOSS_LOGISTIC)
    hipLaunchKernelGGL((inner_svrg_kernel<CPL, NWT, HALP_LOSS_LOGISTIC>), grid, block, 0, s, a);
  else
    hipLaunchKernelGGL((inner_svrg_kernel<CPL, NWT, HALP_LOSS_SQUARED>), grid, block, 0, s, a);
  return hip_ok(hipGetLastError());
}

struct SvShape {
  int cpl, nw;
};

// coordinates per thread and waves per chain: as many waves (up to 4 when chains are few, else
// 1) as keep every thread busy, then wider fragments
SvShape pick_shape(const halp_handle& h) {
  const int d = h.p.d;
  int nw = 1;
  const int64_t simds = 4 * (int64_t)h.num_cus;
  if (h.inner_waves > 0) nw = h.inner_waves;
  else while (nw < 4 && (int64_t)h.p.R * nw * 2 <= simds && 64 * nw < d) nw *= 2;
  int cpl = 1;
  while (cpl < 4 && 64 * nw * cpl < d) cpl *= 2;
  while (64 * nw * cpl < d && nw < 16) nw *= 2;
  return SvShape{cpl, nw};
}

// Where the form with one chain wave is taken, in chains per CU.  ns per step of all chains (shared data, squared
// loss), with it / without: d = 64 512 chains 81 / 121, 1280 112 / 143, 1536 170 / 143; d = 200 1 chain 70 / 235, 512 80 / 234,
// 1280 112 / 201, 2048 198 / 211; d = 512 1 chain 92 / 249, 512 107 / 265 (two workgroups fit a CU; 600 chains would take two
// turns: 267 / 268); d = 1000 256 157 / 294.  Logistic: d = 60 1280 443 / 471, d = 200 1280 445 / 534, d = 512 512 205 / 601.
// The L2 term costs it two instructions per coordinate: squared loss with lambda > 0, d = 64 1280 116 / 138, d = 128 1280
// 117 / 155, 1536 182 / 155, 2048 215 / 191 (without L2 158 / 156, 185 / 190), d = 200 2048 218 / 245.
bool lone_pays(const halp_handle& h) {
  const int d = h.p.d;
  if (h.inner_waves > 0 || d > 1024) return false;
  const bool few = d <= 64 || (d <= 128 && h.p.lambda > 0 && h.p.loss == HALP_LOSS_SQUARED);
  const int per_cu = few ? 5 : (d <= 256 ? 8 : (d <= 512 ? 2 : 1));
  return (int64_t)h.p.R <= (int64_t)h.num_cus * per_cu;
}

}  // namespace

// squared or logistic loss, one row per step, d <= 4096 (16 waves of 64 threads of 4 coordinates)
int inner_svrg_supported(const halp_handle& h) {
  const halp_params& p = h.p;
  if (p.K != 1 || p.B != 1) return HALP_ERR_UNSUPPORTED;
  if (p.loss != HALP_LOSS_SQUARED && p.loss != HALP_LOSS_LOGISTIC) return HALP_ERR_UNSUPPORTED;
  const SvShape sh = pick_shape(h);
  if (64 * sh.nw * sh.cpl < p.d) return HALP_ERR_UNSUPPORTED;
  const bool built = (sh.nw <= 4 && (sh.nw == 1 || sh.nw == 2 || sh.nw == 4)) ||
                     (sh.cpl == 4 && (sh.nw == 8 || sh.nw == 16));
  return built ? HALP_OK : HALP_ERR_UNSUPPORTED;
}

int launch_inner_svrg(const halp_handle& h, uint32_t epoch, hipStream_t s) {
  const halp_params& p = h.p;
  const int rc = inner_svrg_supported(h);
  if (rc != HALP_OK) return rc;
  SvArgs a;
  a.X = h.buf.X; a.y = reinterpret_cast<const float*>(h.buf.y); a.phi = h.buf.phi; a.g = h.buf.g;
  a.w = h.buf.w;
  a.N = p.N; a.ldx = h.buf.ldx; a.T = p.T;
  a.x_chain_stride = p.share_data ? 0 : p.N * h.buf.ldx;
  a.y_chain_stride = p.share_data ? 0 : p.N;
  a.d = p.d; a.loss = p.loss; a.hyper = h.hyper; a.lambda = p.lambda; a.option2 = h.option2 ? 1 : 0;
  a.seed = p.seed; a.epoch = epoch;
  if (lone_pays(h)) {
    const bool pair = p.R > h.num_cus;
    if (p.d <= 256) return pair ? launch_lone<1, true>(a, p.R, s) : launch_lone<1, false>(a, p.R, s);
    if (p.d <= 512) return pair ? launch_lone<2, true>(a, p.R, s) : launch_lone<2, false>(a, p.R, s);
    return launch_lone<4, false>(a, p.R, s);
  }
  const SvShape sh = pick_shape(h);
#define HALP_SV(C_, W_) \
  if (sh.cpl == C_ && sh.nw == W_) return launch_loss<C_, W_>(a, p.R, s);
  HALP_SV(1, 1) HALP_SV(2, 1) HALP_SV(4, 1)
  HALP_SV(1, 2) HALP_SV(2, 2) HALP_SV(4, 2)
  HALP_SV(1, 4) HALP_SV(2, 4) HALP_SV(4, 4)
  HALP_SV(4, 8) HALP_SV(4, 16)
#undef HALP_SV
  return HALP_ERR_UNSUPPORTED;
}

}  // namespace halp
