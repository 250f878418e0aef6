// Both streaming passes in one launch when units span several segments (section 3.1, Eq. (1);
// section 3.2, Eq. (3)).  The per-segment loops are in stream_passes.h, the key stream in
// stream_common.h.
#include "stream_passes.h"

namespace kv {
namespace stream {
namespace {

// ------------------------------------------------------------------------------------------------
// Units split over several workgroups, one launch: every workgroup runs pass 1 over each of its
// segments (per_wg consecutive ones), publishes the segments' (m, z) per row and adds them to its
// unit's arrival counter, issues pass 2's first tile loads, and waits (a bounded poll) until every
// segment of the unit has arrived; then it merges the unit's partials into the normalisers and runs
// pass 2 over its keys, with the queries still in registers.  Segments stay the unit of the
// statistics whatever per_wg is: 80 units of 30000 keys in four segments are 320 workgroups, over
// the chip's CUs, so two segments each go to 160 (the eviction pass 421 -> 368 us, before with two
// launches and mu, sigma in memory).  Nothing assumes that all workgroups are resident at once: a
// workgroup whose poll runs out computes the partials of the unit's other segments itself (the
// same code over the same keys, hence the same values, written to the same slots) and goes on,
// so a launch that shares the chip with other work is slower, never wrong or stuck.
// ------------------------------------------------------------------------------------------------
__device__ __forceinline__ void store_partial(float2* dst, float2 v) {
  __hip_atomic_store(reinterpret_cast<uint64_t*>(dst), __builtin_bit_cast(uint64_t, v),
                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float2 load_partial(const float2* src) {
  return __builtin_bit_cast(float2, __hip_atomic_load(reinterpret_cast<const uint64_t*>(src),
                                                      __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}

// In base-score mode (SC) pass 2 stores each key's base score instead of mu and sigma (see
// stream_window.hip).  MULTI: workgroups of several segments; those of one (per_wg is 1) are
// compiled without the loop over segments (32 launches of one layer of 32768 keys each, 32 segments
// of 1024 keys per unit: 1.52 -> 1.43 ms).
template <int D, int NB, int W, bool ALL, int NW, int S, bool SC, bool MULTI>
__global__ __launch_bounds__(NW * 64, 1) void window_coop_kernel(StreamArgs a, uint32_t* arrive,
                                                                 uint32_t spin_limit) {
  using Gm = SGeo<D, NB>;
  constexpr int R = Gm::R, NS = Gm::NS, NT = NW * 64, P = NT / R;
  __shared__ __align__(16) uint16_t ring[NW][S * Gm::TE];
  __shared__ float2 red[NW][R];
  __shared__ float2 mz_part[P][R];
  __shared__ __align__(16) float bsh[R];
  __shared__ uint32_t all_arrived;

  const int seg = blockIdx.x * (MULTI ? a.per_wg : 1), g = blockIdx.y, p = blockIdx.z;  // its first segment
  const int L = a.lens[p];
  if ((int64_t)seg * a.seg_keys >= L) return;  // none of this unit's segments
  const int n_seg = (L + a.seg_keys - 1) / a.seg_keys;
  const int seg_end = MULTI ? min(seg + a.per_wg, n_seg) : seg + 1;  // one past its last
  const int k0 = seg * a.seg_keys;
  const int k1 = (int)min((int64_t)seg_end * a.seg_keys, (int64_t)L);
  const int G = a.h_q / a.h_kv;
  const int lane = threadIdx.x & 63, half = lane >> 5, l32 = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const float c = a.c;
  const float inv_g = 1.f / (float)G;
  const size_t unit = (size_t)p * a.h_kv + g;
  const size_t stat_base = (size_t)a.tok_off[p] * a.h_kv + (size_t)g * L;
  const uint16_t* kg = a.k + stat_base * D;
  float2* part_u = a.part + unit * a.max_segs * R;
  auto tiles_of = [&](int s0, int s1) {
    const int n_tiles = (s1 - s0 + kTileKeys - 1) / kTileKeys;
    return n_tiles > wave ? (n_tiles - wave + NW - 1) / NW : 0;
  };

  KeyStream<D, NB, NW, S> ks{ring[wave], kg, k0, k1, wave, lane};
  const int my_tiles = tiles_of(k0, k1);
  // the key stream of segment sg alone and the wave's tiles in it
  auto stream_of = [&](int sg) {
    const int s0 = sg * a.seg_keys;
    return KeyStream<D, NB, NW, S>{ring[wave], kg, s0, (int)min((int64_t)s0 + a.seg_keys, (int64_t)L), wave, lane};
  };

  bf16x8_t q[NB][NS];
  load_queries<D, NB, W>(q, a.q_win + ((size_t)p * a.h_q + (size_t)g * G) * W * D, l32, half, G * W);
  {
    const auto st = stream_of(seg);
    st.prologue(tiles_of(st.k0, st.k1));
  }
  hold_until_loaded<D, NB>(q);

  // pass 1 over segment `sg`, whose first tiles are loading, by the whole workgroup; its partial
  // goes to its slot with device-coherent stores, complete before the workgroup leaves the final
  // barrier.  The first tiles of segment `next` (none: negative) load meanwhile.
  auto pass1 = [&](int sg, int next) {
    const auto st = stream_of(sg);
    float m_run[NB], z_run[NB];
    stats_tiles<D, NB, NW, S, W>(st, q, tiles_of(st.k0, st.k1), st.k1, L, c, l32, half, m_run, z_run);
    if (next >= 0) {
      const auto sn = stream_of(next);
      sn.prologue(tiles_of(sn.k0, sn.k1));
    }
    stats_to_lds<NB>(m_run, z_run, red[wave], l32, half);
    __syncthreads();
    if (threadIdx.x < R) store_partial(part_u + (size_t)sg * R + threadIdx.x, merge_waves<NW, R>(&red[0][0], threadIdx.x));
    wait_vmem<0>();
    __syncthreads();  // red is free again, every partial store has completed
  };
  for (int sg = seg; sg < seg_end; ++sg) pass1(sg, sg + 1 < seg_end ? sg + 1 : -1);
  // The partials and the counter are device-coherent atomics (no cache-wide write-back or
  // invalidation, which would disturb every workgroup streaming keys through the same L2).
  if (threadIdx.x == 0)
    __hip_atomic_fetch_add(arrive + unit, (uint32_t)(seg_end - seg), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  // the ring is free (pass 1's last wait covered all its loads): pass 2's first tiles load while
  // the other segments arrive
  ks.prologue(my_tiles);
  if (threadIdx.x == 0) {
    uint32_t spins = 0, n = 0;
    while ((n = __hip_atomic_load(arrive + unit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) < (uint32_t)n_seg &&
           spins < spin_limit) {
      __builtin_amdgcn_s_sleep(1);
      ++spins;
    }
    all_arrived = n >= (uint32_t)n_seg ? 1u : 0u;
  }
  __syncthreads();
  if (!all_arrived) {
    // Not every segment arrived in time: the other segments' partials are computed here.
    wait_vmem<0>();  // pass 2's prologue loads own the ring until they land
    for (int sg = 0; sg < n_seg; ++sg) {
      if (sg >= seg && sg < seg_end) continue;
      const auto st = stream_of(sg);
      st.prologue(tiles_of(st.k0, st.k1));
      pass1(sg, -1);
    }
    ks.prologue(my_tiles);
  }
  // normalisers: thread (row, part) merges segments part, part + P, ... of its row (partials read
  // with device-coherent loads), then one thread per row merges the P results in a fixed order
  // (the same order as the two-launch path)
  {
    const int row = threadIdx.x % R, pt = threadIdx.x / R;
    float M = -INFINITY, Z = 0.f;
    for (int q0 = pt; q0 < n_seg; q0 += 4 * P) {
      float2 v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int qq = q0 + u * P;
        v[u] = qq < n_seg ? load_partial(part_u + (size_t)qq * R + row) : make_float2(-INFINITY, 0.f);
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) merge_mz(M, Z, v[u].x, v[u].y);
    }
    mz_part[pt][row] = make_float2(M, Z);
  }
  __syncthreads();
  if (threadIdx.x < R) {
    float M = mz_part[0][threadIdx.x].x, Z = mz_part[0][threadIdx.x].y;
#pragma unroll
    for (int pt = 1; pt < P; ++pt) merge_mz(M, Z, mz_part[pt][threadIdx.x].x, mz_part[pt][threadIdx.x].y);
    const bool real_row = W == 32 || threadIdx.x < G * W;  // else padding of the last block
    bsh[threadIdx.x] = real_row ? M + __builtin_log2f(Z) : INFINITY;
    if (seg == 0 && real_row) {
      const size_t ri = ((size_t)p * a.h_q + (size_t)g * G) * W + threadIdx.x;
      a.row_max_out[ri] = M * kLn2;
      a.row_sum_out[ri] = Z;
    }
  }
  __syncthreads();
  if constexpr (SC) {
    const ScoreOut so{a.score + stat_base, a.lambda1[p], a.w_mu};
    mu_sigma_tiles<D, NB, ALL, NW, S, kOutScore, W>(ks, q, bsh, my_tiles, k1, L, c, inv_g, nullptr, nullptr,
                                            l32, half, so, nullptr, G);
  } else {
    mu_sigma_tiles<D, NB, ALL, NW, S, kOutMuSigma, W>(ks, q, bsh, my_tiles, k1, L, c, inv_g, a.mu + stat_base,
                                      a.sigma + stat_base, l32, half, {}, nullptr, G);
  }
  wait_vmem<0>();  // no load into the ring may outlive the workgroup
}

__global__ void zero_words_kernel(uint32_t* w, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) w[i] = 0u;
}

// One launch of window_coop_kernel after its counters are cleared.  Used when the whole grid fits
// the chip at once (then no workgroup normally waits long); `launched` tells the caller whether it
// ran.
template <int D, int NB, int W> struct CoopLaunch {
  using Kernel = void (*)(StreamArgs, uint32_t*, uint32_t);
  template <bool MULTI> static Kernel kernel(bool all, bool sc) {
    if (all)
      return sc ? window_coop_kernel<D, NB, W, true, kWaves, 2, true, MULTI>
                : window_coop_kernel<D, NB, W, true, kWaves, 2, false, MULTI>;
    return sc ? window_coop_kernel<D, NB, W, false, kWaves, 2, true, MULTI>
              : window_coop_kernel<D, NB, W, false, kWaves, 2, false, MULTI>;
  }
  static hipError_t run(const Shape& s, const StreamArgs& args, hipStream_t st, uint32_t* arrive,
                        uint32_t spin_limit, int64_t n_wgs, bool* launched) {
    const bool sc = args.score != nullptr;
    const Kernel kern = args.per_wg > 1 ? kernel<true>(args.sigma_all, sc) : kernel<false>(args.sigma_all, sc);
    int dev = 0, n_cu = 0, per_cu = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev);
    if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, kThreads, 0);
    if (e != hipSuccess) return e;
    const dim3 grid(args.wg_columns, s.h_kv, s.n_prob);
    if (n_wgs > (int64_t)per_cu * n_cu) {  // (the grid's other workgroups leave at once)
      *launched = false;
      return hipSuccess;
    }
    const int n_units = s.n_prob * s.h_kv;
    zero_words_kernel<<<(n_units + 255) / 256, 256, 0, st>>>(arrive, n_units);
    kern<<<grid, kThreads, 0, st>>>(args, arrive, spin_limit);
    e = hipGetLastError();
    *launched = e == hipSuccess;
    return e;
  }
};

}  // namespace
}  // namespace stream

hipError_t launch_stream_window_coop(const Shape& s, const StreamPlan& plan, const void* q_win,
                                     const void* k, float scale, void* ws, float* row_max,
                                     float* row_sum, float* mu, float* sigma, bool sigma_all,
                                     uint32_t spin_limit, hipStream_t stream, bool* launched,
                                     const ScoreMode* sm) {
  *launched = false;
  stream::StreamArgs a = stream::base_args(s, plan, q_win, k, scale);
  a.part = static_cast<float2*>(ws);
  a.row_max_out = row_max;
  a.row_sum_out = row_sum;
  a.mu = mu;
  a.sigma = sigma;
  a.sigma_all = sigma_all ? 1 : 0;
  if (sm) {
    a.score = sm->score;
    a.lambda1 = sm->lambda1;
    a.w_mu = sm->w_mu;
  }
  uint32_t* arrive = reinterpret_cast<uint32_t*>(static_cast<char*>(ws) + stream_counter_offset(s, plan));
  return stream::launch_for_shape<stream::CoopLaunch>(s, a, stream, arrive, spin_limit,
                                                        plan.n_wgs, launched);
}

}  // namespace kv
