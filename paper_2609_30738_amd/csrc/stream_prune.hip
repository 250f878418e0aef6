// Window statistics and the candidate set of the selection in one workgroup per unit, reading the
// keys once in full (section 3.1, Eq. (1), Eq. (3); section 3.2, Eq. (5) and the top-4B
// restriction).
//
// Pass 1 streams every key tile, as in stream_window.hip, and also records, per tile and per
// (head, window row), the tile's largest logit as a one-byte code below the tile's largest logit
// (TileCodes; 128 bytes per tile in the workspace).  Once the row normalisers b are complete, these
// codes bound the base score of every key of each tile from above (tile_bound).  The tiles are
// then ordered by their bounds (a counting sort into bins of 1/16 of an octave below the largest
// bound, each tile standing for its bin's upper edge) and pass 2 evaluates the exact base scores
// tile by tile in that order, wave w taking positions w, w + 8, ... of the order.  The evaluated
// keys of the candidate range go into an LDS histogram (Prune), which gives a lower bound of the
// unit's cut (the C-th best score), and a wave stops at its first tile whose bound lies below it:
// every key of the tiles left out scores below the cut.  The evaluated scores are stored over the
// tiles' codes; after the pass the C-th largest (score, position) entry among them is found digit
// by digit, and the C candidates are written in position order.  Scores are formed by the same
// code as in the other window kernels, so each evaluated key's score is the one
// kv_window_base_scores writes, bit for bit, and the candidates are exactly the unit's C best.
//
// On the 32-layer Mistral-shaped pass at L = 32768 (C = 256) the bounds leave about one tile in
// twenty to pass 2.
#include "select_gram.h"
#include "stream_bounds.h"

namespace kv {
namespace stream {
namespace {

// Bitmap words over the candidate positions of a unit (one bit per position).
constexpr int kBitmapWords = kCandMaxLen / 32;
// Entries that share every digit found so far and are ranked directly (by counting).
constexpr int kRankDirect = 512;

// The bin (order key >> kPruneShift) of the C-th largest entry counted in hist, scanning down from
// top (a bin at or above every nonempty one), into *cut_bin, and the number of entries in the bins
// above it into *above.  One wave; hist holds at least C entries.
__device__ __forceinline__ void find_cut_bin(const uint32_t* hist, uint32_t top, int C, int lane,
                                             uint32_t* cut_bin, uint32_t* above) {
  uint32_t cum = 0;
  for (int b0 = (int)top; b0 >= 0; b0 -= 64) {
    const int b = b0 - lane;
    const uint32_t own = b >= 0 ? hist[b] : 0u;
    const uint32_t pre = wave_inclusive_sum(own);
    const uint64_t hit = __ballot(cum + pre >= (uint32_t)C);
    if (hit) {
      const int hl = __ffsll((unsigned long long)hit) - 1;
      if (lane == hl) {
        *cut_bin = (uint32_t)b;
        *above = cum + pre - own;
      }
      return;
    }
    cum += (uint32_t)__builtin_amdgcn_readlane((int)pre, 63);
  }
}

// With PRUNE = false (units whose tiles hardly outnumber the candidates, so that almost every tile
// would be revisited) pass 1 writes no codes, nothing is bounded or ordered, and pass 2 evaluates
// every tile in its own order, as kv_window_base_scores does; the rest is the same.
template <int D, int NB, bool ALL, int NW, int S, bool SEL, bool PRUNE>
__global__ __launch_bounds__(NW * 64, 1) void window_prune_kernel(StreamArgs a) {
  using Gm = SGeo<D, NB>;
  constexpr int R = Gm::R, NS = Gm::NS, NT = NW * 64;
  constexpr int kRedWords = NW * R * 2;
  static_assert(NT % kTileKeys == 0, "whole tiles per visit");
  static_assert(kTileKeys == 32, "a half-wave visits the keys of one tile");
  static_assert(2 * kOrderBins >= kBitmapWords + 2 * kRankDirect,
                "the bitmap and the ranked group fit the order's bins");
  static_assert(kPruneBins >= kBitmapWords, "the word prefixes fit the histogram");
  // the waves' key rings; after the second pass, the order keys of the evaluated scores
  constexpr int kRingElems = NW * S * Gm::TE > 2 * kCandMaxLen ? NW * S * Gm::TE : 2 * kCandMaxLen;
  __shared__ __align__(16) uint16_t ring[kRingElems];
  static_assert(!SEL || gram::region_bytes<D>(gram::kMaxCand) <= sizeof(ring),
                "the staged key rows and the cosine triangle fit the ring");
  static_assert(!SEL || 4 * gram::kMaxCand <= kPruneMaxTiles, "the slot arrays fit the bounds");
  // the waves' statistics after pass 1, the histogram of evaluated scores in pass 2
  __shared__ __align__(16) uint32_t red_hist[kRedWords > kPruneBins ? kRedWords : kPruneBins];
  __shared__ __align__(16) float bsh[R];
  // pass 1: the tile's largest t; from the order on: the bound of the i-th tile of the order
  __shared__ float ub[kPruneMaxTiles];
  __shared__ uint16_t order[kPruneMaxTiles];
  // pass 1: the statistics of the unit's segments but the last; then the bin counts and offsets of
  // the order
  constexpr int kSegWords = (kStreamMaxPerWg - 1) * kRedWords;
  __shared__ __align__(16) uint32_t bins[kSegWords > 2 * kOrderBins ? kSegWords : 2 * kOrderBins];
  __shared__ float c_max[NW];
  __shared__ uint32_t ev[NW];
  __shared__ uint32_t cut, bmax_bits, n_eval;
  __shared__ uint64_t cut_entry;

  const int g = blockIdx.y, p = blockIdx.z;
  const int L = a.lens[p];
  const int G = a.h_q / a.h_kv;
  const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, l32 = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const float c = a.c;
  const float inv_g = 1.f / (float)G;
  const float lam1 = a.lambda1[p];
  const size_t stat_base = (size_t)a.tok_off[p] * a.h_kv + (size_t)g * L;
  float2* red = reinterpret_cast<float2*>(red_hist);
  uint32_t* codes_u = a.codes + ((size_t)p * a.h_kv + g) * a.code_stride;

  const uint16_t* kg = a.k + stat_base * D;
  KeyStream<D, NB, NW, S> ks{ring + wave * S * Gm::TE, kg, 0, L, wave, lane};
  const int n_tiles = (L + kTileKeys - 1) / kTileKeys;
  const int my_tiles = n_tiles > wave ? (n_tiles - wave + NW - 1) / NW : 0;
  bf16x8_t q[NB][NS];
  load_queries<D, NB>(q, a.q_win + ((size_t)p * a.h_q + (size_t)g * G) * 32 * D, l32, half);
  ks.prologue(my_tiles);
  hold_until_loaded<D, NB>(q);

  // ---- pass 1: statistics and tile codes
  float m_run[NB], z_run[NB];
  const int n_segs = (L + a.seg_keys - 1) / a.seg_keys;  // at most kStreamMaxPerWg (the plan)
  float2* const red_first = reinterpret_cast<float2*>(bins);
  using Hook = std::conditional_t<PRUNE, TileCodes<NB>, NoTileHook>;
  Hook hook;
  if constexpr (PRUNE) hook = Hook{codes_u, ub, c, l32, lane};
  stats_tiles<D, NB, NW, S>(ks, q, my_tiles, L, L, c, l32, half, m_run, z_run, hook,
                            n_segs > 1 ? red_first + wave * R : nullptr, NW * R,
                            a.seg_keys / (NW * kTileKeys), n_segs);
  const int n_cand = L - a.keep_tail;
  if constexpr (PRUNE) wait_vmem<0>();  // the wave's code stores have landed (others read them below)
  else ks.prologue(my_tiles);           // pass 2's first tiles load while the statistics are merged
  stats_to_lds<NB>(m_run, z_run, red + wave * R, l32, half);
  if (tid == 0) {
    cut = 0u;
    bmax_bits = 0u;
  }
  __syncthreads();
  if (tid < R) {
    const float2 v = merge_unit<NW, R>(red_first, NW * R, n_segs, red, tid);
    bsh[tid] = v.x + __builtin_log2f(v.y);  // b = M + log2 Z, base 2
    const size_t ri = ((size_t)p * a.h_q + (size_t)g * G) * 32 + tid;
    a.row_max_out[ri] = v.x * kLn2;
    a.row_sum_out[ri] = v.y;
  }
  __syncthreads();  // the normalisers are complete; red is free

  for (int i = tid; i < kPruneBins; i += NT) red_hist[i] = 0u;
  float* score_u = reinterpret_cast<float*>(codes_u);  // a tile's codes are dead once bounded
  const ScoreOut so{score_u, lam1, a.w_mu};
  const int bp = a.budgets ? a.budgets[p] : a.budget;
  const int C = min(a.cand_mult * bp, n_cand);
  int n_ord;   // tiles in the order of pass 2
  float smax;  // the lane's largest evaluated score
  if constexpr (PRUNE) {
  // ---- bounds of the tiles and their order
  const float bmax = order_tiles<NB, ALL, NT>(codes_u, n_tiles, 0, n_cand, bsh, a.w_mu, lam1, inv_g, ub,
                                              order, bins, &bmax_bits, &n_eval, tid);  // the ring is free

  // ---- pass 2: exact scores of the wanted tiles, stored over their codes
  n_ord = (int)n_eval;
  const int my_tiles2 = n_ord > wave ? (n_ord - wave + NW - 1) / NW : 0;
  // the second visit keeps its tiles in the caches: the selection reads the candidates' rows next
  KeyStream<D, NB, NW, S> ks2{ring + wave * S * Gm::TE, kg, 0, L, wave, lane, order, true};
  ks2.prologue(my_tiles2);
  // the cut's scan starts at the bin of the largest finite bound: scores above it (in tiles with a
  // masked key) are left out of the scan, which only lowers the cut
  const int scan_top = bmax > 0.f ? (int)(order_key(bmax) >> kPruneShift) : kPruneBins - 1;
  Prune pr{ub, red_hist, &cut, score_u, scan_top, n_cand, C, -INFINITY, 0};
  mu_sigma_tiles<D, NB, ALL, NW, S, kOutCand>(ks2, q, bsh, my_tiles2, L, L, c, inv_g, nullptr,
                                              nullptr, l32, half, so, &pr);
  smax = pr.smax;
  if (lane == 0) ev[wave] = (uint32_t)pr.evaluated;
  } else {
    n_ord = (n_cand + kTileKeys - 1) / kTileKeys;  // the tiles with candidates, in their own order
    for (int i = tid; i < n_ord; i += NT) order[i] = (uint16_t)i;
    if (lane == 0) ev[wave] = (uint32_t)my_tiles;
    mu_sigma_tiles<D, NB, ALL, NW, S, kOutScore>(ks, q, bsh, my_tiles, L, L, c, inv_g, nullptr,
                                                 nullptr, l32, half, so);
    smax = -INFINITY;
  }
  wait_vmem<0>();  // the score stores have landed; no load into the ring outlives the workgroup

  // ---- the unit's candidates: the C largest entries (order key of the score, position) among
  //      the evaluated keys, written in ascending position order.  The C-th largest entry is
  //      found digit by digit (11 bits at a time, most significant first): the histogram of the
  //      pass gives the first digit; each further digit counts the evaluated entries that share
  //      the digits found so far, until few enough remain to rank them directly.
  __syncthreads();  // the scores, the histogram and every wave's tile count are final
  int max_ev = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) max_ev = max(max_ev, (int)ev[w]);
  const int n_pos = min(n_ord, max_ev * NW);  // order positions at or after this one: not evaluated
  // the order keys of the evaluated scores, copied once into the ring (free after the pass) at
  // [order position][key in tile] by waves 1.. while wave 0 finds the first digit of the cut; the
  // passes below visit them there
  uint32_t* okc = reinterpret_cast<uint32_t*>(ring);
  // device-coherent load: the line may still sit in this CU's vector cache with the tile's codes,
  // read before the score was stored over them
  auto load_score = [&](int key) __attribute__((always_inline)) {
    return __uint_as_float(__hip_atomic_load(reinterpret_cast<uint32_t*>(score_u + key),
                                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
  };
  if constexpr (!PRUNE) {
    // the scores of every candidate key: copied, counted and their maximum taken by all waves, four
    // loads of a thread in flight (the last half-wave without keys stays for the histogram's ballots)
    for (int i0 = tid; i0 < (n_ord * kTileKeys + 63) / 64 * 64; i0 += 4 * NT) {
      float sv[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) sv[u] = i0 + u * NT < n_cand ? load_score(i0 + u * NT) : 0.f;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int i = i0 + u * NT;
        const bool in = i < n_cand;
        const uint32_t ok = order_key(sv[u]);
        if (in) {
          smax = fmaxf(smax, sv[u]);
          okc[i] = ok;
        }
        wave_hist_add(red_hist, ok >> kPruneShift, in);
      }
    }
  }
  {
    float m = smax;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
    if (lane == 0) c_max[wave] = m;
  }
  if constexpr (!PRUNE) __syncthreads();  // the histogram is complete
  if (wave == 0) {
    find_cut_bin(red_hist, kPruneBins - 1, C, lane, &cut, &bmax_bits);
  } else if constexpr (PRUNE) {
    constexpr int kVisit = (NT - 64) / kTileKeys;  // tiles per visit
    for (int p0 = 0; p0 < n_pos; p0 += kVisit) {
      const int pos = p0 + (tid - 64) / kTileKeys;
      if (pos < n_pos && (pos / NW) < (int)ev[pos % NW]) {
        const int key = (int)order[pos] * kTileKeys + (tid % kTileKeys);
        if (key < n_cand) okc[pos * kTileKeys + tid % kTileKeys] = order_key(load_score(key));
      }
    }
  }
  __syncthreads();
  // visit every evaluated key of the candidate range once: fn(entry, key)
  auto for_each_entry = [&](auto fn) __attribute__((always_inline)) {
    for (int p0 = 0; p0 < n_pos; p0 += NT / kTileKeys) {
      const int pos = p0 + tid / kTileKeys;
      if (pos < n_pos && (pos / NW) < (int)ev[pos % NW]) {
        const int key = (int)order[pos] * kTileKeys + (tid % kTileKeys);
        if (key < n_cand) fn(cand_entry(okc[pos * kTileKeys + tid % kTileKeys], (uint32_t)key), key);
      }
    }
  };
  uint64_t prefix = (uint64_t)cut << (64 - (32 - kPruneShift));  // the digits found so far
  int pbits = 32 - kPruneShift;                                   // their count
  int need = C - (int)bmax_bits;  // how many entries of the group the candidates still take
  uint32_t group = red_hist[cut];
  while (group > (uint32_t)kRankDirect && pbits < 64) {
    const int dbits = min(32 - kPruneShift, 64 - pbits);
    const int shift = 64 - pbits - dbits;
    __syncthreads();  // the last digit's readers are done with the histogram
    for (int i = tid; i < kPruneBins; i += NT) red_hist[i] = 0u;
    __syncthreads();
    for_each_entry([&](uint64_t e, int) {
      if ((e >> (64 - pbits)) == (prefix >> (64 - pbits)))
        atomicAdd(&red_hist[(uint32_t)(e >> shift) & ((1u << dbits) - 1u)], 1u);
    });
    __syncthreads();
    if (wave == 0) find_cut_bin(red_hist, (1 << dbits) - 1, need, lane, &cut, &bmax_bits);
    __syncthreads();
    prefix |= (uint64_t)cut << shift;
    pbits += dbits;
    need -= (int)bmax_bits;
    group = red_hist[cut];
  }
  // the group: at most kRankDirect entries (or one, once every digit is found); its need-th
  // largest entry is the C-th largest overall, found by counting the larger ones.  A half-wave
  // visits the 32 keys of one evaluated tile: the group is appended by ballot, the candidates'
  // bits of a tile are a ballot too.
  uint64_t* gb = reinterpret_cast<uint64_t*>(bins + kBitmapWords);
  uint32_t* bm = bins;          // the candidates in a bitmap over the positions (word = tile)
  uint32_t* gcnt = red_hist;    // [kRankDirect] entries of the group larger than each member
  const int n_words = (n_cand + 31) >> 5;
  if (tid == 0) {
    n_eval = 0u;
    cut_entry = ~0ull;
  }
  __syncthreads();  // every thread has read the group's size from the histogram
  for (int i = tid; i < kRankDirect; i += NT) gcnt[i] = 0u;
  for (int i = tid; i < n_words; i += NT) bm[i] = 0u;
  // entry of this thread's key in visit p0 (0: none)
  auto entry_at = [&](int p0, int* tile) __attribute__((always_inline)) -> uint64_t {
    const int pos = p0 + tid / kTileKeys;
    *tile = -1;
    if (pos < n_pos && (pos / NW) < (int)ev[pos % NW]) {
      *tile = (int)order[pos];
      const int key = *tile * kTileKeys + (tid % kTileKeys);
      if (key < n_cand) return cand_entry(okc[pos * kTileKeys + tid % kTileKeys], (uint32_t)key);
    }
    return 0ull;
  };
  const uint64_t below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
  for (int p0 = 0; p0 < n_pos; p0 += NT / kTileKeys) {
    int tile;
    const uint64_t e = entry_at(p0, &tile);
    const bool in = e != 0ull && (e >> (64 - pbits)) == (prefix >> (64 - pbits));
    const uint64_t m = __ballot(in);
    if (m) {
      const int leader = __ffsll((unsigned long long)m) - 1;
      uint32_t base = 0;
      if (lane == leader) base = atomicAdd(&n_eval, (uint32_t)__popcll(m));
      base = __builtin_amdgcn_readlane(base, leader);
      const uint32_t at_ = base + (uint32_t)__popcll(m & below);
      if (in && at_ < (uint32_t)kRankDirect) gb[at_] = e;
    }
  }
  __syncthreads();
  const int n_grp = min((int)n_eval, kRankDirect);
  {
    // member i against a share of the group: thread t takes member t % n_grp and share t / n_grp
    const int parts = n_grp > 0 ? max(1, NT / n_grp) : 1;
    if (tid < parts * n_grp) {
      const int i = tid % n_grp, part = tid / n_grp;
      const int j0 = part * n_grp / parts, j1 = (part + 1) * n_grp / parts;
      const uint64_t e = gb[i];
      uint32_t larger = 0;
      for (int j = j0; j < j1; ++j) larger += gb[j] > e ? 1u : 0u;
      if (larger) atomicAdd(&gcnt[i], larger);
    }
  }
  __syncthreads();
  for (int i = tid; i < n_grp; i += NT)
    if (gcnt[i] == (uint32_t)(need - 1)) cut_entry = gb[i];
  __syncthreads();
  const uint64_t t_entry = cut_entry;
  for (int p0 = 0; p0 < n_pos; p0 += NT / kTileKeys) {
    int tile;
    const uint64_t e = entry_at(p0, &tile);
    const uint64_t m = __ballot(e != 0ull && e >= t_entry);
    if ((tid & (kTileKeys - 1)) == 0 && tile >= 0) bm[tile] = (uint32_t)(m >> (lane & 32));
  }
  __syncthreads();
  uint32_t* wpre = red_hist;  // candidates in the bitmap words before each word
  if (wave == 0) {
    constexpr int PW = kBitmapWords / 64;
    uint32_t v[PW];
    uint32_t sum = 0;
#pragma unroll
    for (int k = 0; k < PW; ++k) {
      const int w = lane * PW + k;
      v[k] = w < n_words ? (uint32_t)__popc(bm[w]) : 0u;
      sum += v[k];
    }
    uint32_t run = wave_inclusive_sum(sum) - sum;
#pragma unroll
    for (int k = 0; k < PW; ++k) {
      wpre[lane * PW + k] = run;
      run += v[k];
    }
  }
  __syncthreads();
  uint64_t* dst = a.cand_out + ((size_t)p * a.h_kv + g) * a.cand_stride;
  // with the selection: the candidates' positions and scores by slot, their 1 / |k|, the greedy's
  // trace (the bounds are dead after pass 2; the ranked group's space after the cut)
  int32_t* cpos_l = reinterpret_cast<int32_t*>(ub);
  float* cst_l = ub + gram::kMaxCand;
  float* cinv_l = ub + 2 * gram::kMaxCand;
  uint32_t* trace_slot = reinterpret_cast<uint32_t*>(ub + 3 * gram::kMaxCand);
  uint32_t* trace_key = bins + kBitmapWords;
  for_each_entry([&](uint64_t e, int key) {
    if (e >= t_entry) {
      const uint32_t below = bm[key >> 5] & ((1u << (key & 31)) - 1u);
      const uint32_t rank = wpre[key >> 5] + (uint32_t)__popc(below);
      if (rank < (uint32_t)C) {  // exactly C entries are >= t_entry
        dst[rank] = e;
        if constexpr (SEL) {
          cpos_l[rank] = key;
          cst_l[rank] = key_float((uint32_t)(e >> 32));
        }
      }
    }
  });
  for (int i = C + tid; i < a.cand_stride; i += NT) dst[i] = 0ull;
  float den = c_max[0];
#pragma unroll
  for (int w = 1; w < NW; ++w) den = fmaxf(den, c_max[w]);
  den = fmaxf(den, 1e-12f);
  if (tid == 0) a.cand_max[(size_t)p * a.h_kv + g] = den;
  if constexpr (SEL) {
    // ---- the selection of the unit (section 3.2, Eq. (2), (4)) from its C candidates, as the
    //      selection kernel runs it on the list just written: s~ = score / normaliser, the cosine
    //      triangle in the ring, the greedy on wave 0, then the outputs and the compaction
    __syncthreads();  // the slot arrays are complete; the ring's score keys are dead
    for (int c2 = tid; c2 < C; c2 += NT) cst_l[c2] = cst_l[c2] / den;
    gram::cosines<D, NW>(kg, cpos_l, C, cinv_l, reinterpret_cast<unsigned char*>(ring), tid);
    const float* tri = reinterpret_cast<const float*>(ring) + 1;
    constexpr int kRowVecs = D * 2 / 16;  // 16-byte vectors of a key row
    const uint4* k4 = reinterpret_cast<const uint4*>(a.k);
    const uint4* v4 = reinterpret_cast<const uint4*>(a.v);
    const size_t src0 = stat_base * kRowVecs;
    const size_t dst0 = ((size_t)p * a.h_kv + g) * a.out_rows * kRowVecs;
    if (wave == 0) {
      gram::Greedy gr;
      gr.init(cst_l, C, lane);
      if (a.sel_score) gr.run_for<true>(tri, C, bp, a.lambda2[p], lane, trace_slot, trace_key);
      else gr.run_for<false>(tri, C, bp, a.lambda2[p], lane, trace_slot, trace_key);
    } else if (a.k_out) {
      // meanwhile the other waves copy the kept tail (rows bp .. bp + keep_tail - 1 of the block)
      // and fetch the candidates' value rows into the caches for the compaction below
      const int t1 = tid - 64, nt1 = NT - 64;
      for (int e = t1; e < a.keep_tail * kRowVecs; e += nt1) {
        const int r = e / kRowVecs, cv = e % kRowVecs;
        const size_t sidx = src0 + (size_t)(L - a.keep_tail + r) * kRowVecs + cv;
        const size_t didx = dst0 + (size_t)(bp + r) * kRowVecs + cv;
        reinterpret_cast<uint4*>(a.k_out)[didx] = k4[sidx];
        reinterpret_cast<uint4*>(a.v_out)[didx] = v4[sidx];
      }
      // one dword per 128-byte line of each row, loaded straight into LDS words that nothing
      // reads (the histogram, cleared before its next use below)
      uint32_t* sink = red_hist + 64 * (wave & 7);
      for (int c2 = t1; c2 < C; c2 += nt1) {
        const uint4* row = v4 + src0 + (size_t)cpos_l[c2] * kRowVecs;
#pragma unroll
        for (int l = 0; l < kRowVecs; l += 8)
          __builtin_amdgcn_global_load_lds((gptr_t)(row + l), (lptr_t)sink, 4, 0, 0);
      }
      wait_vmem<0>();
    }
    __syncthreads();
    const size_t so0 = ((size_t)p * a.h_kv + g) * a.budget;
    for (int t = tid; t < a.budget; t += NT) {
      a.sel_idx[so0 + t] = t < bp ? cpos_l[trace_slot[t]] : -1;
      if (a.sel_score) a.sel_score[so0 + t] = t < bp ? key_float(trace_key[t]) : 0.f;
    }
    if (a.k_out) {
      // the admitted rows (the tail is copied)
      int32_t* srt = reinterpret_cast<int32_t*>(ring);  // the triangle is dead
      gram::admitted_in_order(trace_slot, cpos_l, bp, red_hist, srt, tid, NT);
      copy_kept_rows(k4, v4, srt, bp, 0, L, kRowVecs, src0, dst0,
                     reinterpret_cast<uint4*>(a.k_out), reinterpret_cast<uint4*>(a.v_out), tid, NT);
    }
  }
}

template <int D, int NB, int W> struct PruneLaunch {
  static hipError_t run(const Shape& s, const StreamArgs& args, hipStream_t st) {
    if constexpr (W != 32) return hipErrorInvalidValue;  // the tile codes hold 32 window rows
    else return run32(s, args, st);
  }
  static hipError_t run32(const Shape& s, const StreamArgs& args, hipStream_t st) {
    const dim3 grid(1, s.h_kv, s.n_prob);
    const bool all = args.sigma_all != 0, prune = args.prune != 0;
    auto launch = [&](auto al, auto pr) {
      constexpr bool A = decltype(al)::value, P = decltype(pr)::value;
      if (args.sel_idx) window_prune_kernel<D, NB, A, kWaves, 2, true, P><<<grid, kThreads, 0, st>>>(args);
      else window_prune_kernel<D, NB, A, kWaves, 2, false, P><<<grid, kThreads, 0, st>>>(args);
    };
    if (all && prune) launch(std::true_type{}, std::true_type{});
    else if (all) launch(std::true_type{}, std::false_type{});
    else if (prune) launch(std::false_type{}, std::true_type{});
    else launch(std::false_type{}, std::false_type{});
    return hipGetLastError();
  }
};

}  // namespace
}  // namespace stream

int cand_code_stride(const Shape& s) {
  return (s.max_len + stream::kTileKeys - 1) / stream::kTileKeys * 32;
}

hipError_t launch_stream_window_cands(const Shape& s, const StreamPlan& plan, const void* q_win,
                                      const void* k, float scale, const float* lambda1, float w_mu,
                                      int budget, const int32_t* budgets, int cand_mult,
                                      int keep_tail, float* row_max, float* row_sum,
                                      uint64_t* cand_out, float* cand_max, int cand_stride,
                                      uint32_t* codes, bool sigma_all, const CandSelect* sel,
                                      hipStream_t stream) {
  if (!plan.one_wg() || !cand_out || !cand_max || !codes || s.max_len > kCandMaxLen)
    return hipErrorInvalidValue;
  if (sel && (!sel->lambda2 || !sel->sel_idx || (sel->k_out && (!sel->v || !sel->v_out))))
    return hipErrorInvalidValue;
  stream::StreamArgs a = stream::base_args(s, plan, q_win, k, scale);
  a.row_max_out = row_max;
  a.row_sum_out = row_sum;
  a.sigma_all = sigma_all ? 1 : 0;
  a.lambda1 = lambda1;
  a.w_mu = w_mu;
  a.cand_out = cand_out;
  a.cand_max = cand_max;
  a.cand_stride = cand_stride;
  a.budget = budget;
  a.budgets = budgets;
  a.cand_mult = cand_mult;
  a.keep_tail = keep_tail;
  a.codes = codes;
  a.code_stride = cand_code_stride(s);
  // Bounds pay where tiles outnumber candidates and few tiles hold the best keys: with at most as many
  // tiles as candidates, a cut that is not confined to few clusters has one in almost every tile (256
  // units of 8000 keys, C = 256: 287 us with bounds, 267 without; of 2000 keys 129 and 117).  Above the
  // line salient keys gain much (16000 keys, C = 256: 257 and 442; 8000 keys, C = 128: 139 and 232)
  // and flat scores lose a tenth (10000 keys, C = 256: 346 and 317); the line is where the gain can
  // first outweigh the loss, not where it always does.
  a.prune = s.max_len / stream::kTileKeys > cand_stride ? 1 : 0;
  if (sel) {
    a.lambda2 = sel->lambda2;
    a.sel_idx = sel->sel_idx;
    a.sel_score = sel->sel_score;
    a.v = static_cast<const uint16_t*>(sel->v);
    a.k_out = static_cast<uint16_t*>(sel->k_out);
    a.v_out = static_cast<uint16_t*>(sel->v_out);
    a.out_rows = sel->out_rows;
  }
  return stream::launch_for_shape<stream::PruneLaunch>(s, a, stream);
}

}  // namespace kv
