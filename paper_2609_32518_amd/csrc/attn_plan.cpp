// Work split of an attention launch (host arithmetic only, no HIP calls, so the CPU tests
// exercise it): one work-group per 256-query tile over its whole key range, every query tile cut
// into the same number of equal parts, or the launch's (query tile, key tile) units shared equally
// and contiguously by one work-group per compute unit; query tiles cut between work-groups are
// merged afterwards by log-sum-exp.
#include <algorithm>
#include <cstdint>

#include "kernels.hpp"

namespace unstep {

namespace {

AttnPlan balanced(int64_t groups, int64_t qtiles) {
  return AttnPlan{int32_t(groups), attn_workspace_bytes(int32_t(groups)), int32_t(qtiles),
                  size_t(groups) * 2 * kAttnBlockQ * kHeadDim, groups % qtiles == 0 ? int32_t(groups / qtiles) : 0};
}

// Two ends of segments per work-group: units of ~1.82 us plus ~20 us of fill, partials and merge (12
// heads: [1560 queries, 18720 keys] 183 us at 96 units each, [1800, 9000] 62 us at 22).
double contiguous_us(int64_t units, int64_t groups) { return 1.82 * double(units) / double(groups) + 20.0; }

}  // namespace

AttnPlan attn_plan(int32_t B, int32_t H, int32_t N, int32_t n_keys, size_t scratch) {
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
    return t_bal < t_plain && attn_workspace_bytes(int32_t(g)) <= scratch ? balanced(g, qtiles) : plain;
  }
  // Few query tiles: every tile cut into the same number of equal parts of at least four key tiles,
  // so that each work-group walks one segment (one pipeline fill, one partial): as many parts as
  // the chip holds, less those that do not shorten the longest.  Measured (us): a key tile takes 1.08
  // while the chip has power to spare (~1.25 with the slower first tiles of a short range) and 1.66
  // with every compute unit at work; the merge adds 4.5 plus up to 0.75 per part, so a tile is left
  // whole when the split saves less than that.  With this
  // a [390 queries, 3315 keys] call of 24 heads takes 34.5 in 5 parts (65.1 whole, 40.7 split
  // contiguously over 256 work-groups), [324, 4544] of 12 heads 30.0 in 9 (84.6, 34.6), [300, 1200]
  // of 8 heads 21.0 in 4 (28.1, 28.5), [256, 25600] of 2 heads 27.6 in 100 (432), and [300, 500] of
  // 8 heads 16.3 whole (18.3 in 2).
  // The part count falls now and then as the window grows, so a scratch sized once for the widest
  // window can hold fewer parts than a narrower one wants: it then gets as many as fit (a scratch that
  // holds the parts of the full plan gives that plan).
  const int64_t fit = std::min<int64_t>(kSlots, int64_t(scratch / attn_workspace_bytes(1)));
  int64_t parts = std::max<int64_t>(1, std::min(fit / qtiles, tk / 4));
  const int64_t longest = (tk + parts - 1) / parts;
  parts = (tk + longest - 1) / longest;
  const double merge = 4.5 + 0.75 * double(parts) / attn_merge_slices(int32_t(qtiles), int32_t(parts));
  if (parts > 1 && double(tk - longest) * 1.25 < merge) parts = 1;
  const double tile = std::max(1.08, 0.55 + 0.0044 * double(parts * qtiles));
  const double t_parts = 8.0 + double(longest) * tile + merge;
  if (parts > 1 && g == kSlots && fit >= g && contiguous_us(units, g) < t_parts) return balanced(g, qtiles);
  return parts > 1 ? balanced(parts * qtiles, qtiles) : plain;
}

}  // namespace unstep
