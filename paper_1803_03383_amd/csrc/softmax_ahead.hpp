// What the softmax inner loops (and the scalar margins of wide minibatches) need at every step
// and what does not depend on z, made ahead of the loop by the whole chip: sample indices,
// margins and softmax of the sampled rows before the offset, rounding words of gamma, L2 draws
// and the rounding bits of z.  A chain's loop is one workgroup's dependent chain; with these
// made elsewhere it keeps only what follows from z.  An epoch is cut into segments whose
// records fit the workspace: records of a segment, then its steps, then the next segment.
#pragma once

#include "inner_args.hpp"
#include "segments.hpp"

namespace halp {

struct AheadRec {  // one (row, class) of a step, 16 bytes
  double p0;       // softmax of the margins (K = 1: l'(phi_i), logistic only)
  float phi;       // margin (class 1 of a row with K = 1: the label)
  uint32_t rho;    // rounding word of gamma
};
constexpr int kWholeH = 16000;  // |gamma x| + r + |h~| < 2^15 at 8 bits
constexpr int kAheadK = 16;  // records of a row (those past its classes may hold anything)

struct Ahead {
  AheadRec* rec;    // [chain][step][row][16]
  int32_t* idx;     // [chain][step][rows]
  int32_t* cl;      // [chain][step] c_lambda
  uint16_t* zbits;  // [chain][step][class][UP] rounding bits of the strips, or null; expanded: two 16-bit halves
                    // per strip (8 bits), r - h~ of its coordinates
  bool expanded;
  int64_t S;        // steps per segment, a multiple of 8 (buffer dimension)
  int UP;           // strips per class, padded
  int64_t t0;       // first step of the segment
  int64_t t1;       // one past its last step
};

// bytes of workspace for S steps
size_t ahead_bytes(const halp_params& p, int chains, int64_t S, int UP, bool expanded);
// steps per segment that fit `bytes`: a multiple of 8, 0 if not even 8 fit
int64_t ahead_steps(const halp_params& p, int chains, int UP, bool expanded, size_t bytes);
Ahead ahead_layout(const halp_params& p, int chains, int64_t S, int UP, bool expanded, void* ws);
// Sets how an epoch is cut and returns the bytes of workspace.  Chains per launch: even shares of at
// most `resident`, those the device holds at once, since launches run one after the other.  Steps per
// segment: from a workspace of 64 MB, more for many chains (4 MB each) up to 1 GB: a segment costs its
// three launches and the loop's way in and out, ~30 us, which 256 chains at 125 steps a segment paid
// with 10 % (2 GB instead of 1: no faster at 512 and 1024 chains).
size_t plan_ahead(halp_handle& h, int UP, int resident, bool expanded = false);
// fills the segment [t0, t1) of chains chain0 .. chain0 + chains - 1 (zbits only where UP > 0)
int launch_ahead(const InArgs& a, const Ahead& s, int bits, int chain0, int chains, hipStream_t stream);

// The epoch's launches: for every group of chains, segment after segment, the records and then
// loop(segment, first chain, chains, last segment?).  An epoch without steps is one empty segment.
template <typename F>
int for_segments(const InArgs& a, const halp_handle& h, int UP, bool expanded, hipStream_t st, F loop) {
  const halp_params& p = h.p;
  for (int c0 = 0; c0 < p.R; c0 += h.ahead_chains) {
    const int nc = h.ahead_chains < p.R - c0 ? h.ahead_chains : p.R - c0;
    Ahead s = ahead_layout(p, h.ahead_chains, h.ahead_steps, UP, expanded, h.ahead_ws);
    do {
      s.t0 = s.t1;
      s.t1 = s.t0 + s.S < p.T ? s.t0 + s.S : p.T;
      if (s.t1 > s.t0) {
        const int r = launch_ahead(a, s, p.b, c0, nc, st);
        if (r != HALP_OK) return r;
      }
      const int r = loop(s, c0, nc, s.t1 == p.T ? 1 : 0);
      if (r != HALP_OK) return r;
    } while (s.t1 < p.T);
  }
  return HALP_OK;
}

}  // namespace halp
