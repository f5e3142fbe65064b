// Split of a channel's stages over workgroups for the general kernels
// (wbmm_gen.hip).  Host code, run on every call.
#pragma once

#include <stdint.h>

namespace wbmm {

// Workgroups per channel: consecutive stages of one channel per workgroup,
// as many workgroups as the chip holds at a time (slots) or a few rounds of
// them, whichever leaves the fewest stages in a row; a workgroup's prologue
// (coefficients, first rows) costs about ov stages.  Of splits that cost the
// same, the one of fewest workgroups; at most max_parts of them and about
// eight rounds.
//
// Within a number of rounds the most workgroups are the best, so only those
// splits are looked at, ten at most.  Every split in turn took up to 5.7 us
// at 8 channels and 45 at one; these 0.1.
inline void gen_plan(int64_t C, int64_t stages, int64_t slots, double ov, int64_t max_parts, int *spw, int *parts) {
  int64_t last = 8 * slots / C + 1;  // the first split beyond eight rounds
  last = last < stages ? last : stages;
  last = last < max_parts ? last : max_parts;
  double best = 1e300;
  int64_t bper = stages;
  for (int64_t p = 0, r = 1; p < last; ++r) {
    // (at least one more: several rounds a split where channels exceed slots)
    const int64_t most = r * slots / C;
    p = most > p ? most : p + 1;
    p = p < last ? p : last;
    const int64_t per = (stages + p - 1) / p;
    const int64_t rounds = (C * ((stages + per - 1) / per) + slots - 1) / slots;
    const double cost = (double)rounds * ((double)per + ov);
    if (cost < best - 1e-9) {
      best = cost;
      bper = per;
    }
  }
  *spw = (int)bper;
  *parts = (int)((stages + bper - 1) / bper);
}

}  // namespace wbmm
