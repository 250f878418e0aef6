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

StreamPlan stream_plan(const Shape& s, const int32_t* lens, bool whole) {
  // about one segment per compute unit (256 on MI355X), whole 256-key steps of the eight waves
  constexpr int64_t kTarget = 256, kStep = stream::kWaves * stream::kTileKeys;
  const int64_t max_seg = ((int64_t)s.max_len + kStep - 1) / kStep * kStep;
  int64_t total = 0;
  for (int p = 0; p < s.n_prob; ++p) total += (int64_t)s.h_kv * lens[p];
  auto work_items = [&](int64_t keys) {  // workgroups that take `keys` keys each
    int64_t n = 0;
    for (int p = 0; p < s.n_prob; ++p) n += s.h_kv * ((lens[p] + keys - 1) / keys);
    return n;
  };
  int64_t seg = ((total + kTarget - 1) / kTarget + kStep - 1) / kStep * kStep;
  if (s.w == 32) {
    // four tiles per wave at least: shorter segments cost more in exchanges than they save
    seg = std::min(std::max<int64_t>(1024, seg), max_seg);
  } else {
    // a tile of a short window is a quarter or half of the work, so segments go down to one tile
    // per wave (L = 4096, 8 units: 14.1 us against 19.6 with four); up to 1024 keys a unit stays
    // whole, which needs no exchange (9.3 us against 13.0 in four segments).  A few workgroups over
    // the chip's CUs would cost a second round: then longer segments (160 units of 2500 keys whole
    // 37 us, as 320 segments 58)
    seg = std::min(std::max<int64_t>(s.max_len <= 1024 ? 1024 : kStep, seg), max_seg);
    while (seg < max_seg && work_items(seg) > kTarget)
      seg = std::min(max_seg, seg + std::max<int64_t>(kStep, seg / 16 / kStep * kStep));
  }
  StreamPlan plan;
  plan.seg_keys = (int)seg;
  plan.max_segs = (int)(((int64_t)s.max_len + seg - 1) / seg);
  // segments over the chip's CUs go to workgroups of several, as few as it takes to fit
  plan.per_wg = whole && plan.max_segs <= kStreamMaxPerWg ? plan.max_segs : 1;
  while (plan.per_wg < plan.max_segs && work_items(seg * plan.per_wg) > kTarget) ++plan.per_wg;
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
