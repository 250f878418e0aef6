// Host-side planning of the streaming window kernels: which shapes they take, how a batch is cut
// into segments, and the workspace those segments need.
#include "stream_common.h"

namespace kv {

bool stream_shape_ok(const Shape& s, float scale) {
  const int G = s.group();
  // pass 1 takes a tile's maximum logit as the scaled maximum of the raw dot products
  const bool window = s.w == 32 ? G == 1 || G == 2 || G == 4 : (s.w == 8 || s.w == 16) && s.rows() <= 64;
  return s.dtype == kDtBf16 && window && (s.d == 64 || s.d == 128) && scale > 0.f;
}

namespace {

constexpr int64_t kCus = 256, kXcds = 8;                            // MI355X
constexpr int64_t kStep = stream::kWaves * stream::kTileKeys;       // keys of a step of the eight waves
constexpr int64_t kMaxScheduled = 1024;                             // workgroups that `scheduled_within` follows

// Whether no CU streams more than `limit` keys when every workgroup takes `keys` keys of a unit, one
// workgroup to a CU (the key rings fill its LDS).  Workgroup i of a launch goes to XCD i mod 8, the
// grid's empty workgroups (`columns` to a unit) counted, and there to the CU that is free first.
bool scheduled_within(const Shape& s, const int32_t* lens, int64_t keys, int columns, int64_t limit) {
  constexpr int kPer = kCus / kXcds;
  int32_t busy[kXcds][kPer] = {};  // keys of each CU, at most limit (2^25)
  int64_t id = 0;
  for (int p = 0; p < s.n_prob; ++p)
    for (int g = 0; g < s.h_kv; ++g, id += columns)
      for (int64_t w = 0; w * keys < lens[p]; ++w) {
        int32_t* cus = busy[(id + w) % kXcds];
        int32_t least = cus[0];
        for (int c = 1; c < kPer; ++c) least = std::min(least, cus[c]);
        const int64_t sum = least + std::min(keys, lens[p] - w * keys);
        if (sum > limit) return false;
        int c = 0;
        while (cus[c] != least) ++c;
        cus[c] = (int32_t)sum;
      }
  return true;
}

}  // namespace

StreamPlan stream_plan(const Shape& s, const int32_t* lens, WgRule rule) {
  const int64_t max_seg = ((int64_t)s.max_len + kStep - 1) / kStep * kStep;
  int64_t total = 0;
  for (int p = 0; p < s.n_prob; ++p) total += (int64_t)s.h_kv * lens[p];
  auto work_items = [&](int64_t keys) {  // workgroups that take `keys` keys each
    int64_t n = 0;
    for (int p = 0; p < s.n_prob; ++p) n += s.h_kv * ((lens[p] + keys - 1) / keys);
    return n;
  };
  const bool many_units = (int64_t)s.n_prob * s.h_kv > kCus;  // nothing fits the chip at once
  // about one segment per compute unit, whole steps
  int64_t seg = ((total + kCus - 1) / kCus + kStep - 1) / kStep * kStep;
  // Segments over the chip's CUs: one launch of longer ones (or of workgroups of several) ends when
  // its busiest CU does, the segments' own two launches take about two rounds.  A CU streams alone
  // hardly faster than beside 255 others (33 GB/s against 27), so past two segments' keys on one CU
  // two launches are shorter.  Over 60 batches of unequal lengths (d = 128, G = 4) mu and sigma take
  // 0.33 to 1.08 times as long as in two launches always at w = 32, 0.84 in the median, and 0.27 to 1.08
  // times the chunked kernels' time at w = 8 (0.77).  In one launch always, a prompt of 100001 keys
  // beside 30 of 1000 took 815 us (w = 32) and 495 (w = 8), now 149 and 105; in two launches always,
  // 20 layers of 14000 keys 366 us, in one 257.
  StreamPlan plan;
  auto set_segments = [&](int64_t keys) {
    plan.seg_keys = (int)keys;
    plan.max_segs = (int)((s.max_len + keys - 1) / keys);
    plan.ragged = (int64_t)s.n_prob * s.h_kv * plan.max_segs > work_items(keys);
  };
  // the plan's segments, `per` to a workgroup, against segments of `even` keys
  auto one_launch = [&](int64_t per, int64_t even) {
    const int64_t keys = per * plan.seg_keys;
    if (std::min<int64_t>(keys, s.max_len) > 2 * even) return false;
    return work_items(keys) > kMaxScheduled ||
           scheduled_within(s, lens, keys, plan.columns((int)((s.max_len + keys - 1) / keys)), 2 * even);
  };
  if (s.w == 32) {
    // four tiles per wave at least.  Not the fastest: mu and sigma of one layer of 4096 keys take 31 us
    // with segments of 1024 keys, 24 with 512 and 21 with 256, of 32768 keys 43 with each; the segments
    // are the unit of the row statistics, whose last bits shorter ones would change.
    seg = std::min(std::max<int64_t>(1024, seg), max_seg);
  } else {
    // a tile of a short window is a quarter or half of the work, so segments go down to one tile
    // per wave (L = 4096, 8 units: 14.1 us against 19.6 with four); up to 1024 keys a unit stays
    // whole, which needs no exchange (9.3 us against 13.0 in four segments).  A few workgroups over
    // the chip's CUs would cost a second round: then longer segments (160 units of 2500 keys whole
    // 37 us, as 320 segments 58)
    seg = std::min(std::max<int64_t>(s.max_len <= 1024 ? 1024 : kStep, seg), max_seg);
    int64_t longer = many_units ? max_seg : seg;
    while (longer < max_seg && work_items(longer) > kCus)
      longer = std::min(max_seg, longer + std::max<int64_t>(kStep, longer / 16 / kStep * kStep));
    set_segments(longer);
    if (longer > seg && one_launch(1, seg)) seg = longer;
    // what the chunked kernels do within the static scratch is not refused for the partials' size
    // (a thousand short units beside a long one in segments under 1024 keys)
    const size_t most = std::max(window_stats_ws_bytes(s), kNoAllocScratchBytes);
    for (set_segments(seg); seg < max_seg && stream_ws_bytes(s, plan) > most; set_segments(seg))
      seg = std::min(max_seg, 2 * seg);
  }
  set_segments(seg);
  int64_t per_wg = 1;
  if (rule == WgRule::kWhole && plan.max_segs <= kStreamMaxPerWg) {
    per_wg = plan.max_segs;
  } else {
    if (many_units) per_wg = plan.max_segs;
    while (per_wg < plan.max_segs && work_items(seg * per_wg) > kCus) ++per_wg;
    if (per_wg > 1 && rule != WgRule::kAny && !one_launch(per_wg, seg)) per_wg = 1;
  }
  plan.per_wg = (int)per_wg;
  plan.max_wgs = (plan.max_segs + plan.per_wg - 1) / plan.per_wg;
  plan.n_wgs = work_items(seg * plan.per_wg);
  return plan;
}

size_t stream_counter_offset(const Shape& s, const StreamPlan& plan) {
  const size_t part = (size_t)s.n_prob * s.h_kv * plan.max_segs * s.row_blocks() * 32 * sizeof(float2);
  return (part + 255) & ~(size_t)255;
}

size_t stream_ws_bytes(const Shape& s, const StreamPlan& plan) {
  // segment partials, then one arrival counter per unit (both passes in one launch)
  return stream_counter_offset(s, plan) + (size_t)s.n_prob * s.h_kv * sizeof(uint32_t);
}

}  // namespace kv
