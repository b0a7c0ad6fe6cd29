// Work split of an attention launch (host arithmetic only, no HIP calls, so the CPU tests
// exercise it): one work-group per 256-query tile over its whole key range, every query tile cut
// into the same number of equal parts, or the launch's (query tile, key tile) units shared equally
// and contiguously by one work-group per compute unit; query tiles cut between work-groups are
// merged afterwards by log-sum-exp.
#include <algorithm>
#include <cmath>
#include <cstdint>

#include "kernels.hpp"

namespace unstep {

namespace {

AttnPlan balanced(int64_t groups, int64_t qtiles) {
  return AttnPlan{int32_t(groups), attn_workspace_bytes(int32_t(groups)), int32_t(qtiles),
                  size_t(groups) * 2 * kAttnBlockQ * kHeadDim, groups % qtiles == 0 ? int32_t(groups / qtiles) : 0};
}

// Times (us) of long ranges of 50-128 query tiles, split contiguously over 256 work-groups (two ends of
// segments each) and into equal parts on `groups` work-groups, of which fewer draw less power and run
// faster: fitted to 79 shapes, on which the choice between the two is within 1% of the better one
// (96 query tiles, 2 parts on 192 work-groups: [1015 queries, 6100 keys] 81 in parts, 85 contiguous;
// [1002, 16000] 184 and 181; [3852, 21900] 235 and 227).
double contiguous_us(int64_t units) { return 23.8 + 1.63 * double(units) / kAttnMaxGroups; }
double parts_us(int64_t longest, int64_t groups) { return 16.9 + double(longest) * (0.483 + 0.00423 * double(groups)); }

// The plan with at most `slots` work-groups when it splits.
AttnPlan plan_of(int32_t B, int32_t H, int32_t N, int32_t n_keys, int64_t slots) {
  constexpr int64_t kSlots = kAttnMaxGroups;
  const int64_t qtiles = int64_t(B) * H * ((N + kAttnBlockQ - 1) / kAttnBlockQ);
  const int64_t tk = (n_keys + kAttnBlockK - 1) / kAttnBlockK;
  const int64_t units = qtiles * tk;
  const AttnPlan plain{int32_t(qtiles), 0, int32_t(qtiles), 0, 1};
  const int64_t g = std::min<int64_t>(kSlots, units / 4);
  if (2 * qtiles > kSlots) {
    // At most one work-group per query tile fits beside the others: the whole range each, or the
    // contiguous split.  Costs measured on MI355X (us): a 256-query x 64-key tile takes ~1.66 when a
    // work-group walks one query tile's whole range and ~1.82 per unit in the split schedule (two
    // segments per work-group, fp32 partials written, and all compute units drawing power, which
    // lowers the clock of the power-limited chip); the merge reads the partials at ~4.5 TB/s plus
    // ~2 us.
    if (g <= qtiles) return plain;
    const double t_plain = double((qtiles + kSlots - 1) / kSlots) * double(tk) * 1.66;
    const double t_bal = double((units + g - 1) / g) * 1.82 + double(attn_workspace_bytes(int32_t(g))) / 4.5e6 + 2.0;
    return t_bal < t_plain && g <= slots ? balanced(g, qtiles) : plain;
  }
  // Few query tiles: every tile cut into the same number of equal parts of at least four key tiles,
  // so that each work-group walks one segment (one pipeline fill, one partial): as many parts as
  // the chip holds, less those that do not shorten the longest.  Measured (us): a key tile takes 1.08
  // while the chip has power to spare (1.1 with the slower first tiles of a short range) and 1.66
  // with every compute unit at work.  In short ranges a split costs 2.5 plus 2.4 times the square root of
  // its partials' MB (stores, launch and loads of the merge), so a tile is left whole when that is
  // more than it saves: within 2% of the better of the two over 136 shapes of 6-126 query tiles and
  // 8-41 key tiles (24 heads of [540 queries, 720 keys] 21.1 whole, 26.7 in 3 parts; 16 of [600, 1600]
  // 35.8 and 27.1 in 5; 40 of [540, 1620] 37.9 and 35.1 in 2).  With this
  // a [390 queries, 3315 keys] call of 24 heads takes 34.5 in 5 parts (65.1 whole, 40.7 split
  // contiguously over 256 work-groups), [324, 4544] of 12 heads 30.0 in 9 (84.6, 34.6), [300, 1200]
  // of 8 heads 21.0 in 4 (28.1, 28.5), [256, 25600] of 2 heads 27.6 in 100 (432), and [300, 500] of
  // 8 heads 16.3 whole (18.3 in 2).
  int64_t parts = std::max<int64_t>(1, std::min(slots / qtiles, tk / 4));
  const int64_t longest = (tk + parts - 1) / parts;
  parts = (tk + longest - 1) / longest;
  const double partial_mb = double(B) * H * N * double(parts) * (kHeadDim + 2) * 4e-6;
  if (parts > 1 && double(tk - longest) * 1.1 < 2.5 + 2.4 * std::sqrt(partial_mb)) parts = 1;
  if (parts > 1 && g == kSlots && slots >= g && contiguous_us(units) < parts_us(longest, parts * qtiles))
    return balanced(g, qtiles);
  return parts > 1 ? balanced(parts * qtiles, qtiles) : plain;
}

}  // namespace

// The part count falls now and then as the window grows, so a scratch sized once for the widest window can
// hold fewer parts than a narrower one wants: that one then gets as many as fit.
AttnPlan attn_plan(int32_t B, int32_t H, int32_t N, int32_t n_keys, size_t scratch) {
  const AttnPlan full = plan_of(B, H, N, n_keys, kAttnMaxGroups);
  if (full.workspace <= scratch) return full;
  return plan_of(B, H, N, n_keys, int64_t(scratch / attn_workspace_bytes(1)));
}

}  // namespace unstep
