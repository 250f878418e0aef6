// Base scores of the keys that can be candidates, for units of several workgroups (section 3.1,
// Eq. (1), Eq. (3); section 3.2, Eq. (5) and the top-4B restriction): the two passes of
// stream_prune.hip as two launches, reading the keys once in full.
//
// Launch 1 runs pass 1 over every segment: the segment's partial (m, z) per window row, and per tile
// the codes of its row maxima and its reference into the workspace.  In launch 2 every workgroup
// merges its unit's partials into the normalisers, bounds and orders the tiles of its own segments,
// and revisits them in that order until their bounds fall below its cut, the C-th best score among
// its own keys.  That cut is at most the unit's, so every candidate of the unit is evaluated; the
// scores of the keys left out read -inf, and the selection kernel cuts the candidates from the row.
// No workgroup waits for another, and none shares its cut: a histogram of the unit in memory, raised
// by every workgroup and read every second tile, cost more in atomics than it saved (16 units of
// 30000 keys 198 us against 116 with both passes in full, 64 units of 100001 446 against 451).
//
// Bound by the first launch's stream of the keys.  Eight layers of 100001 keys (64 units of four
// workgroups, C = 256): both passes in full 552 us, these two launches 350, the eviction pass 651 and
// 451.
#include "stream_bounds.h"

namespace kv {
namespace stream {
namespace {

struct SegArgs {
  float* refs;      // [n_units][ref_stride] tile references
  int ref_stride;
};

template <int D, int NB, int NW, int S>
__global__ __launch_bounds__(NW * 64, 1) void stats_codes_kernel(StreamArgs a, SegArgs sa) {
  using Gm = SGeo<D, NB>;
  constexpr int R = Gm::R, NS = Gm::NS;
  __shared__ __align__(16) uint16_t ring[NW][S * Gm::TE];
  __shared__ float2 red[NW][R];

  const int seg = blockIdx.x, g = blockIdx.y, p = blockIdx.z;
  const int L = a.lens[p];
  if ((int64_t)seg * a.seg_keys >= L) return;
  const int k0 = seg * a.seg_keys;
  const int k1 = (int)min((int64_t)k0 + a.seg_keys, (int64_t)L);
  const int G = a.h_q / a.h_kv;
  const int lane = threadIdx.x & 63, half = lane >> 5, l32 = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const size_t unit = (size_t)p * a.h_kv + g;
  const int tile0 = k0 / kTileKeys;

  KeyStream<D, NB, NW, S> ks{ring[wave], a.k + ((size_t)a.tok_off[p] * a.h_kv + (size_t)g * L) * D, k0, k1,
                             wave, lane};
  const int n_tiles = (k1 - k0 + kTileKeys - 1) / kTileKeys;
  const int my_tiles = n_tiles > wave ? (n_tiles - wave + NW - 1) / NW : 0;
  bf16x8_t q[NB][NS];
  load_queries<D, NB>(q, a.q_win + ((size_t)p * a.h_q + (size_t)g * G) * 32 * D, l32, half);
  ks.prologue(my_tiles);
  hold_until_loaded<D, NB>(q);
  float m_run[NB], z_run[NB];
  stats_tiles<D, NB, NW, S>(ks, q, my_tiles, k1, L, a.c, l32, half, m_run, z_run,
                            TileCodes<NB, true>{a.codes + unit * a.code_stride + 32 * tile0,
                                                sa.refs + unit * sa.ref_stride + tile0, a.c, l32, lane});
  wait_vmem<0>();  // no load into the ring may outlive the workgroup
  stats_to_lds<NB>(m_run, z_run, red[wave], l32, half);
  __syncthreads();
  if (threadIdx.x < R)
    a.part[(unit * a.max_segs + seg) * R + threadIdx.x] = merge_waves<NW, R>(&red[0][0], threadIdx.x);
}

template <int D, int NB, bool ALL, int NW, int S>
__global__ __launch_bounds__(NW * 64, 1) void prune_segs_kernel(StreamArgs a, SegArgs sa) {
  using Gm = SGeo<D, NB>;
  constexpr int R = Gm::R, NS = Gm::NS, NT = NW * 64, P = NT / R;
  __shared__ __align__(16) uint16_t ring[NW][S * Gm::TE];
  __shared__ __align__(16) uint32_t hist[kPruneBins];
  __shared__ __align__(16) float bsh[R];
  __shared__ float ub[kPruneMaxTiles];
  __shared__ uint16_t order[kPruneMaxTiles];
  __shared__ __align__(16) uint32_t bins[2 * kOrderBins];
  __shared__ uint32_t cut, bmax_bits, n_eval;
  static_assert(sizeof(bins) >= P * R * sizeof(float2), "the partial merges fit the bins");

  const int g = blockIdx.y, p = blockIdx.z, tid = threadIdx.x;
  const int L = a.lens[p];
  const int64_t first = (int64_t)blockIdx.x * a.per_wg * a.seg_keys;
  if (first >= L) return;
  const int k0 = (int)first;
  const int k1 = (int)min(first + (int64_t)a.per_wg * a.seg_keys, (int64_t)L);
  const int G = a.h_q / a.h_kv;
  const int lane = tid & 63, half = lane >> 5, l32 = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const float inv_g = 1.f / (float)G;
  const float lam1 = a.lambda1[p];
  const size_t unit = (size_t)p * a.h_kv + g;
  const size_t stat_base = (size_t)a.tok_off[p] * a.h_kv + (size_t)g * L;
  const int tile0 = k0 / kTileKeys, n_tiles = (k1 - k0 + kTileKeys - 1) / kTileKeys;
  const int n_cand = L - a.keep_tail;
  float* score_u = a.score + stat_base;

  bf16x8_t q[NB][NS];
  load_queries<D, NB>(q, a.q_win + ((size_t)p * a.h_q + (size_t)g * G) * 32 * D, l32, half);
  // the unit's normalisers from the segment partials, merged as by the other two-launch path
  float2* mz = reinterpret_cast<float2*>(bins);
  {
    const int n_seg = (L + a.seg_keys - 1) / a.seg_keys;
    const int row = tid % R, pt = tid / R;
    const float2* src = a.part + unit * a.max_segs * R + row;
    float M = -INFINITY, Z = 0.f;
    for (int q0 = pt; q0 < n_seg; q0 += 4 * P) {
      float2 v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int qq = q0 + u * P;
        v[u] = qq < n_seg ? src[(size_t)qq * R] : make_float2(-INFINITY, 0.f);
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) merge_mz(M, Z, v[u].x, v[u].y);
    }
    mz[pt * R + row] = make_float2(M, Z);
  }
  for (int i = tid; i < n_tiles; i += NT) ub[i] = sa.refs[unit * sa.ref_stride + tile0 + i];
  for (int i = k0 + tid; i < k1; i += NT) score_u[i] = -INFINITY;
  for (int i = tid; i < kPruneBins; i += NT) hist[i] = 0u;
  if (tid == 0) {
    cut = 0u;
    bmax_bits = 0u;
  }
  wait_vmem<0>();  // the fill has landed before any score is stored over it (below, after barriers)
  __syncthreads();
  if (tid < R) {
    float M = mz[tid].x, Z = mz[tid].y;
#pragma unroll
    for (int pt = 1; pt < P; ++pt) merge_mz(M, Z, mz[pt * R + tid].x, mz[pt * R + tid].y);
    bsh[tid] = M + __builtin_log2f(Z);
    if (blockIdx.x == 0) {
      const size_t ri = ((size_t)p * a.h_q + (size_t)g * G) * 32 + tid;
      a.row_max_out[ri] = M * kLn2;
      a.row_sum_out[ri] = Z;
    }
  }
  __syncthreads();
  const float bmax = order_tiles<NB, ALL, NT>(a.codes + unit * a.code_stride + 32 * tile0, n_tiles, k0, n_cand,
                                              bsh, a.w_mu, lam1, inv_g, ub, order, bins, &bmax_bits,
                                              &n_eval, tid);
  const int n_ord = (int)n_eval;
  const int my_tiles = n_ord > wave ? (n_ord - wave + NW - 1) / NW : 0;
  const int bp = a.budgets ? a.budgets[p] : a.budget;
  KeyStream<D, NB, NW, S> ks{ring[wave], a.k + stat_base * D, k0, k1, wave, lane, order, true};
  ks.prologue(my_tiles);
  hold_until_loaded<D, NB>(q);
  const int scan_top = bmax > 0.f ? (int)(order_key(bmax) >> kPruneShift) : kPruneBins - 1;
  Prune pr{ub, hist, &cut, score_u, scan_top, n_cand, min(a.cand_mult * bp, n_cand), -INFINITY, 0};
  mu_sigma_tiles<D, NB, ALL, NW, S, kOutCand>(ks, q, bsh, my_tiles, k1, L, a.c, inv_g, nullptr, nullptr, l32,
                                              half, ScoreOut{nullptr, lam1, a.w_mu}, &pr);
  wait_vmem<0>();  // no load into the ring may outlive the workgroup
}

template <int D, int NB, int W> struct PruneSegsLaunch {
  static hipError_t run(const Shape& s, const StreamArgs& a, hipStream_t st, SegArgs sa) {
    if constexpr (W != 32) {
      return hipErrorInvalidValue;  // the tile codes hold 32 window rows
    } else {
      stats_codes_kernel<D, NB, kWaves, 2><<<dim3(a.seg_columns, s.h_kv, s.n_prob), kThreads, 0, st>>>(a, sa);
      hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
      const dim3 grid(a.wg_columns, s.h_kv, s.n_prob);
      if (a.sigma_all) prune_segs_kernel<D, NB, true, kWaves, 2><<<grid, kThreads, 0, st>>>(a, sa);
      else prune_segs_kernel<D, NB, false, kWaves, 2><<<grid, kThreads, 0, st>>>(a, sa);
      return hipGetLastError();
    }
  }
};

}  // namespace
}  // namespace stream

bool prune_segs_ok(const StreamPlan& plan, int max_cand) {
  // A workgroup's tiles must fit its tables.  Its cut rests on its own keys, so it stops early only
  // where those hold C keys above the rest: three tiles to a candidate leave room for that (about one
  // key in a hundred).  Where they do not, most tiles are revisited and the call takes a sixth longer
  // than with both passes in full: 64 units of flat scores, 131072 keys 1235 us against 1047, 100001 keys
  // 943 against 812 (with repeated passages and salient clusters 459 against 784); at 391 tiles a
  // workgroup (C = 256) it was 409 against 365 for salient keys too.
  const int64_t tiles = (int64_t)plan.per_wg * plan.seg_keys / stream::kTileKeys;
  return plan.max_wgs > 1 && tiles <= stream::kPruneMaxTiles && tiles >= 3 * (int64_t)max_cand;
}

static int prune_segs_tiles(const Shape& s) {  // tiles of the longest unit, whole 256-byte rows of refs
  return ((s.max_len + stream::kTileKeys - 1) / stream::kTileKeys + 63) / 64 * 64;
}

size_t prune_segs_bytes(const Shape& s) {
  return (size_t)s.n_prob * s.h_kv * prune_segs_tiles(s) * (32 + 1) * sizeof(uint32_t);
}

hipError_t launch_prune_segs(const Shape& s, const StreamPlan& plan, const void* q_win, const void* k,
                             float scale, const float* lambda1, float w_mu, int budget,
                             const int32_t* budgets, int cand_mult, int keep_tail, void* part_ws,
                             void* codes_ws, float* row_max, float* row_sum, float* score,
                             bool sigma_all, hipStream_t stream) {
  if (plan.max_wgs < 2 || !part_ws || !codes_ws || !score) return hipErrorInvalidValue;
  stream::StreamArgs a = stream::base_args(s, plan, q_win, k, scale);
  const int tiles = prune_segs_tiles(s);
  a.part = static_cast<float2*>(part_ws);
  a.row_max_out = row_max;
  a.row_sum_out = row_sum;
  a.sigma_all = sigma_all ? 1 : 0;
  a.lambda1 = lambda1;
  a.w_mu = w_mu;
  a.score = score;
  a.budget = budget;
  a.budgets = budgets;
  a.cand_mult = cand_mult;
  a.keep_tail = keep_tail;
  a.codes = static_cast<uint32_t*>(codes_ws);
  a.code_stride = 32 * tiles;
  const stream::SegArgs sa{reinterpret_cast<float*>(a.codes + (size_t)s.n_prob * s.h_kv * a.code_stride), tiles};
  return stream::launch_for_shape<stream::PruneSegsLaunch>(s, a, stream, sa);
}

}  // namespace kv
