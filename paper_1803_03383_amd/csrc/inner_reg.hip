// Launch-shape selection of the register-resident inner loop (Algorithm 4, inner
// `for t`; kernel in inner_reg_impl.hpp): how many waves share a chain and how
// many 16-bit strips of z a lane owns.
#include "inner_args.hpp"

namespace halp {

int launch_inner_reg_b8(const InArgs& a, int nw, int upl, int R, bool packed, hipStream_t s);
int launch_inner_reg_b16(const InArgs& a, int nw, int upl, int R, bool few, hipStream_t s);
int launch_inner_reg_helped_b8(const InArgs& a, int nw, int upl, int R, hipStream_t s);
int launch_inner_reg_helped_b16(const InArgs& a, int nw, int upl, int R, hipStream_t s);
int launch_inner_reg_lone_b8(const InArgs& a, int upl, int lanes, int R, bool pair, hipStream_t s);
int launch_inner_reg_lone_b8_l2(const InArgs& a, int upl, int lanes, int R, bool pair, hipStream_t s);
int launch_inner_reg_lone_b16(const InArgs& a, int upl, int lanes, int R, bool pair, hipStream_t s);
int launch_inner_reg_lone_b16_l2(const InArgs& a, int upl, int lanes, int R, bool pair, hipStream_t s);

namespace {

struct Shape {
  int nw, upl;
};

bool launchable(Shape sh) {
  if (sh.upl != 1 && sh.upl != 2 && sh.upl != 4 && sh.upl != 8) return false;
  if (sh.nw == 1 || sh.nw == 2 || sh.nw == 4) return true;
  return (sh.nw == 8 || sh.nw == 16) && sh.upl >= 4;
}

// `want_nw` waves per chain if the strips can be spread that thin, else as many
// strips per lane as it takes (at most 8, then more waves)
Shape pick_shape(const halp_params& p, int want_nw) {
  const int ct = 16 / p.b;
  const int U = (p.d + ct - 1) / ct;
  int nw = want_nw < 1 ? 1 : (want_nw > 16 ? 16 : want_nw);
  while (nw > 1 && (nw / 2) * 64 >= U) nw /= 2;  // no wave without a strip
  auto strips = [&](int w) {
    const int upl = (U + 64 * w - 1) / (64 * w);
    int u2 = 1;
    while (u2 < upl) u2 *= 2;
    return u2;
  };
  int upl = strips(nw);
  while (upl > 8 && nw < 16) {
    nw *= 2;
    upl = strips(nw);
  }
  if ((nw == 8 || nw == 16) && upl < 4) upl = 4;  // only wide lanes are built for 8 / 16 waves
  return Shape{nw, upl};
}

// the form with a helper wave beside every chain wave exists for these shapes
bool helped_shape(Shape sh) { return (sh.nw == 2 || sh.nw == 4) && sh.upl <= 2; }

// Chains per CU up to which that form pays, by chain waves (measured at d = 512, b = 8, epochs of
// 16384 steps: four chain waves win up to 2 chains per CU -- 3.0 ms at 256 chains, 3.7 at 512,
// where one wave per chain takes 5.5 -- two chain waves up to 5 per CU -- 4.2 ms at 576 chains,
// 6.0 at 1280 against 4.8 and 7.6 -- beyond that one wave per chain and no helpers)
constexpr int kHelpedChainsPerCu4 = 2, kHelpedChainsPerCu2 = 5;

// Strips per lane and lanes of the form with one chain wave and its helpers on the other SIMDs (rows
// of up to 512 strips: 1024 coordinates at 8 bits, 512 at 16); upl 0 if the shape does not fit it.
// 16 lanes at 8 bits and up to 32 strips: 71 ns per step with two strips per lane; with four, for up to 64
// strips, 93 against the 78 of two strips on 64 lanes.
struct Lone {
  int upl, lanes;
};
Lone lone_shape(const halp_handle& h) {
  const halp_params& p = h.p;
  if (p.B != 1 || p.K != 1) return Lone{0, 0};
  const int U = p.b == 8 ? (p.d + 1) / 2 : p.d;
  if (p.b == 8 && U <= 32) return Lone{2, 16};
  if (p.b == 16 && U <= 64) return Lone{1, 64};
  return Lone{U <= 128 ? 2 : (U <= 256 ? 4 : (U <= 512 ? 8 : 0)), 64};
}

// Where the library takes that form by itself, in chains per CU.  Measured in ns per step of all chains (256 CUs, 2000
// rows and steps, shared data), what runs without it / this form, in three kinds of epoch: -h~ rides in the records; it
// does not (mu = 8); lambda = 0.01 with alpha = 0.1, a draw in every fourth step at 8 bits and in every one at 16:
//   8 bits, squared    d = 64    256 chains 141/80 141/92 158/87, 1280 202/145 201/174 224/175, 1536 202/169 202/211 225/206
//                      d = 128   520 144/126 145/148 161/147, 768 145/127 145/149 161/148, 900 (first kind alone) 147/147
//                      d = 256   256 132/85 131/99 194/92, 1024 206/153 208/179 224/177, 1536 276/231 278/267 311/273
//                      d = 512   256 157/112 159/134 230/126 (two workgroups fit a CU; 600 chains would take two turns)
//                      d = 1024  256 244/172 245/209 337/200 (one fits)
//   8 bits, logistic   d = 64    256 243/194 244/203 262/203, 768 (first kind) 247/298, 1024 393/364 391/391 416/389
//                      d = 256   520 394/220 394/241 417/249, 1024 442/410 437/438 456/426; d = 1024 256 349/275 349/304 451/301
//   16 bits, squared   d = 64    520 158/100 158/103 172/120, 1536 224/167 221/171 244/181
//                      d = 128   520 212/122 212/126 235/138, 1536 265/241 266/241 295/257; d = 256 256 213/128 206/129 225/133
//                      d = 512   256 240/186 233/194 242/197
//   16 bits, logistic  d = 64    768 (first kind) 259/324, 1024 410/354 408/365 431/358; d = 128 1024 482/423 484/425 500/435
// So 1536 chains of up to 64 coordinates and 768 of 65 .. 128 lose 2 - 5 % where -h~ is large and gain 12 - 17 % where it is not.
// (Epochs of a few steps take 2 - 4 us more than without it, up to 40 steps; 150 at 512 coordinates of 16 bits.)
bool lone_pays(const halp_handle& h, Lone sh) {
  const bool logistic = h.p.loss == HALP_LOSS_LOGISTIC;
  const int64_t R = h.p.R, cus = h.num_cus;
  // Logistic rows of up to 64 coordinates: with three workgroups to a CU two chain waves share a SIMD and take turns at
  // the exponential, while one wave per chain still has a SIMD each
  if (logistic && (sh.lanes == 16 || sh.upl == 1) && R > 2 * cus && R <= 3 * cus) return false;
  int64_t per_cu = 1;
  if (sh.upl <= 2) per_cu = h.p.b == 8 && h.p.d > 64 && h.p.d <= 128 ? 3 : (logistic ? 4 : 6);
  else if (sh.upl == 4) per_cu = 2;
  return R <= per_cu * cus;
}

// waves per chain: use the chip's SIMDs when chains are few, one wave per chain
// when they are many
int auto_waves(const halp_handle& h) {
  if (h.inner_waves > 0) return h.inner_waves;
  if (h.inner_helpers != 2) {
    const int64_t R = h.p.R, cus = h.num_cus;
    if (R <= kHelpedChainsPerCu4 * cus) {
      const Shape sh = pick_shape(h.p, 4);
      if (sh.nw == 4 && helped_shape(sh)) return 4;
    }
    if (R <= kHelpedChainsPerCu2 * cus) {
      const Shape sh = pick_shape(h.p, 2);
      if (sh.nw == 2 && helped_shape(sh)) return 2;
    }
  }
  const int64_t simds = 4 * (int64_t)h.num_cus;
  int nw = 1;
  while (nw < 4 && (int64_t)h.p.R * nw * 2 <= simds) nw *= 2;
  return nw;
}

}  // namespace

int inner_reg_supported(const halp_params& p) {
  if (p.B != 1 || p.K != 1) return HALP_ERR_UNSUPPORTED;
  if (p.loss != HALP_LOSS_SQUARED && p.loss != HALP_LOSS_LOGISTIC) return HALP_ERR_UNSUPPORTED;
  if (p.b == 8 && p.d > 131071) return HALP_ERR_UNSUPPORTED;  // int32 dot product stays exact
  const Shape sh = pick_shape(p, 16);
  return sh.upl <= 8 ? HALP_OK : HALP_ERR_UNSUPPORTED;
}

int launch_inner_reg(const halp_handle& h, uint32_t epoch, hipStream_t s) {
  const halp_params& p = h.p;
  int rc = inner_reg_supported(p);
  if (rc != HALP_OK) return rc;
  const InArgs a = make_inner_args(h, epoch);
  // few chains per CU: one chain wave with all of z, helpers on the other SIMDs
  const Lone lone = lone_shape(h);
  const bool lone_forced = h.inner_helpers == 3 && p.b == 8;
  if (lone.upl > 0 && (lone_forced || (h.inner_helpers == 0 && h.inner_waves == 0 && lone_pays(h, lone)))) {
    const bool pair = (int64_t)p.R > (int64_t)h.num_cus;  // the build with at most 128 registers
    const auto launch = p.b == 8 ? (p.lambda > 0 ? launch_inner_reg_lone_b8_l2 : launch_inner_reg_lone_b8)
                                 : (p.lambda > 0 ? launch_inner_reg_lone_b16_l2 : launch_inner_reg_lone_b16);
    return launch(a, lone.upl, lone.lanes, p.R, pair, s);
  }
  if (h.inner_helpers == 3) return HALP_ERR_UNSUPPORTED;
  Shape sh = pick_shape(p, auto_waves(h));
  const int ct = 16 / p.b;
  const int U = (p.d + ct - 1) / ct;
  // a lane reads whole fragments of 2*UPL bytes: the last one must lie inside the row, and
  // 16-byte fragments want 16-byte aligned rows
  const int64_t row_bytes = h.buf.ldxq * (p.b / 8);
  const bool base16 = (reinterpret_cast<uintptr_t>(h.buf.Xq) % 16) == 0 && row_bytes % 16 == 0;
  while (sh.upl > 1 && ((int64_t)((U + sh.upl - 1) / sh.upl) * sh.upl * 2 > row_bytes ||
                        (sh.upl == 8 && !base16))) {
    if (sh.nw >= 16) return HALP_ERR_UNSUPPORTED;
    sh.nw *= 2;  // spread the strips over more waves instead
    sh.upl /= 2;
  }
  if (!launchable(sh)) return HALP_ERR_UNSUPPORTED;
  // Few chains, two or four waves each: a helper wave beside every chain wave takes whatever
  // does not depend on z off the step's dependent chain.  Worth it while a CU holds a few chains.
  const bool helped_built = helped_shape(sh);
  if (helped_built &&
      (h.inner_helpers == 1 || (h.inner_helpers == 0 && (int64_t)p.R <= (int64_t)kHelpedChainsPerCu2 * h.num_cus)))
    return p.b == 8 ? launch_inner_reg_helped_b8(a, sh.nw, sh.upl, p.R, s)
                    : launch_inner_reg_helped_b16(a, sh.nw, sh.upl, p.R, s);
  // 8 bits, one wave per chain: the packed form once every SIMD holds two chains or more (its
  // steps issue fewer instructions but take longer alone), or as HALP_OPT_INNER_PACKED says
  const bool many = (int64_t)p.R >= 8 * (int64_t)h.num_cus;
  const bool packed = p.b == 8 && sh.nw == 1 && (h.inner_packed == 1 || (h.inner_packed == 0 && many));
  return p.b == 8 ? launch_inner_reg_b8(a, sh.nw, sh.upl, p.R, packed, s)
                  : launch_inner_reg_b16(a, sh.nw, sh.upl, p.R, 2 * (int64_t)p.R <= h.num_cus, s);
}

}  // namespace halp
