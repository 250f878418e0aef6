// Score bounds of key tiles and the order they are revisited in (section 3.2, Eq. (5) and the top-4B
// restriction), shared by the kernel that takes whole units (stream_prune.hip) and the two launches
// for units of several workgroups (stream_prune_segs.hip): what pass 1 records per tile (TileCodes),
// and the bounds and the order from it (order_tiles).
#pragma once

#include "stream_passes.h"

namespace kv {
namespace stream {
namespace {

constexpr int kPruneMaxTiles = kCandMaxLen / kTileKeys;
// Order of the tiles for pass 2: bin 0 holds the tiles with a masked key (bound +inf), bin k >= 1
// the tiles whose bound lies within ((k - 1) / 16, k / 16] octaves below the largest finite bound
// (the last bin: everything further below).
constexpr int kOrderBins = 1024;
constexpr float kBinsPerOctave = 16.f;
// Bounds are widened by kBoundSlack for the rounding of both passes (logits formed in another
// MFMA operand order, approximate exp2 / log2) and kept above kBoundFloor.
constexpr float kBoundSlack = 1.00390625f;  // 1 + 2^-8
constexpr float kBoundFloor = 0x1p-100f;
constexpr float kCodeStep = 0.125f;          // code units: 1/8 of a factor of two

// Pass-1 hook of candidate mode: per tile, the largest t = logit * c of every (head, window row) as
// the number of 1/8-steps it lies below the tile's largest t (rounded down, one less where the
// exact number is an odd integer; at most 255), one byte per head of the row's word in the unit's
// code rows, and the tile's largest t into ref[tile] (LDS); a tile with a masked key gets
// ref = +inf and a tile with a NaN logit ref = NaN (both always revisited).  The row maxima of two
// heads are merged across the wave's halves in one exchange, leaving head k in lanes 0-31 and head
// k + NB / 2 in lanes 32-63, so each lane stores the bytes of its row's word that belong to its
// heads (one store per tile).
// With GREF the tiles' references go to memory (a second store per tile), for a later launch.
template <int NBH, bool GREF = false> struct TileCodes {
  static constexpr int kStores = GREF ? 2 : 1;
  static_assert(NBH == 1 || NBH == 2 || NBH == 4, "one, two or four query heads per key head");
  uint32_t* codes;  // tile i at codes + 32 i: word r = window row r, byte b < NB = head b
  float* ref;       // [n_tiles], LDS or (GREF) memory
  float c;          // softmax scale * log2(e)
  int l32, lane;

  template <int NB>
  __device__ __forceinline__ void interior(int tile, const float (&tmax)[NB]) const {
    static_assert(NB == NBH, "head count");
    constexpr int NP = NB == 4 ? 2 : 1;  // heads per lane after the exchange
    float tm[NP];  // row maxima of t over the tile's 32 keys
    if constexpr (NB == 1) {
      tm[0] = max_halves(tmax[0]) * c;
    } else {
#pragma unroll
      for (int k = 0; k < NP; ++k) {
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(tmax[k]),
                                                        __float_as_uint(tmax[k + NB / 2]), false, false);
        tm[k] = __builtin_elementwise_maximum(__uint_as_float(r[0]), __uint_as_float(r[1])) * c;
      }
    }
    const float m = NP == 2 ? __builtin_elementwise_maximum(tm[0], tm[NP - 1]) : tm[0];
    float r = wave_max_uniform(m);  // the tile's largest t
    if (__ballot(m != m)) r = __builtin_nanf("");
    // code: the steps (r - t) * 8 less half a step, rounded to nearest (even) and saturated to
    // [0, 255] by v_cvt_pk_u8_f32: never above the exact number of steps (NaN gives 0)
    uint32_t w = 0u;
#pragma unroll
    for (int k = 0; k < NP; ++k)
      w = __builtin_amdgcn_cvt_pk_u8_f32(fmaf(r - tm[k], 1.f / kCodeStep, -0.5f), (uint32_t)k, w);
    char* dst = reinterpret_cast<char*>(codes + 32 * tile + l32);
    if constexpr (NB == 4) store_u16(dst + 2 * (lane >> 5), w);
    else if constexpr (NB == 2) store_u8(dst + (lane >> 5), w);
    else store_u8(dst, w);
    put_ref(tile, r);
  }
  __device__ __forceinline__ void guarded(int tile) const {
    store_word(codes + 32 * tile + l32, 0xFFFFFFFFu);
    put_ref(tile, INFINITY);
  }
  __device__ __forceinline__ void put_ref(int tile, float r) const {
    if (lane == 0) {
      if constexpr (GREF) store_word(reinterpret_cast<uint32_t*>(ref + tile), __float_as_uint(r));
      else ref[tile] = r;
    }
  }
  __device__ __forceinline__ static void store_word(uint32_t* dst, uint32_t v) {
    asm volatile("global_store_dword %0, %1, off sc1" ::"v"(dst), "v"(v) : "memory");
  }
  __device__ __forceinline__ static void store_u16(char* dst, uint32_t v) {
    asm volatile("global_store_short %0, %1, off sc1" ::"v"(dst), "v"(v) : "memory");
  }
  __device__ __forceinline__ static void store_u8(char* dst, uint32_t v) {
    asm volatile("global_store_byte %0, %1, off sc1" ::"v"(dst), "v"(v) : "memory");
  }
};

// Upper bound of the base score s = w_mu mu + lambda1 sigma (section 3.2, Eq. (5)) of every key of
// a tile from its codes (row r of head h: t <= ref - code / 8) and the final row normalisers b:
// a[h][r] = 2^(t - b[h][r]) <= a'[h][r], hence mu <= (1 / 32) sum_r abar'[r] (abar': mean over the
// G heads) and, since a variance is at most the mean square, sigma <= sqrt(sum_r abar'[r]^2 / 31)
// (sum_{h,r} a'^2 / (32 G - 1) for the dispersion over all rows).  The positive parts of w_mu and
// lambda1 enter.
// A thread takes whole tiles: bound by its 128 exponentials per tile.  Eight lanes per tile, four rows
// each, read a wave's codes in one coalesced load, but 32 layers of 32768 keys (C = 256) then take
// 433 us instead of 430 (kv_window_candidates) and 458 instead of 455.5 (kv_evict_pass).
template <int NB, bool ALL>
__device__ __forceinline__ float tile_bound(const uint32_t* codes_t, float ref, const float* bsh,
                                            float wmu_p, float lam1_p, float inv_g) {
  const uint4* src = reinterpret_cast<const uint4*>(codes_t);
  float p1 = 0.f, p2 = 0.f;
#pragma unroll 2
  for (int v = 0; v < 8; ++v) {
    const uint4 w4 = src[v];
    const uint32_t ws[4] = {w4.x, w4.y, w4.z, w4.w};
    float arow[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const float4 bv = *reinterpret_cast<const float4*>(bsh + b * 32 + 4 * v);
      const float bb[4] = {bv.x, bv.y, bv.z, bv.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float code = (float)((ws[e] >> (8 * b)) & 0xFFu);
        const float a = __builtin_amdgcn_exp2f(fmaf(code, -kCodeStep, ref) - bb[e]);
        arow[e] += a;
        if constexpr (ALL) p2 = fmaf(a, a, p2);
      }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      p1 += arow[e];
      if constexpr (!ALL) {
        const float ab = arow[e] * inv_g;
        p2 = fmaf(ab, ab, p2);
      }
    }
  }
  constexpr float inv_n1 = ALL ? 1.f / (float)(NB * 32 - 1) : 1.f / 31.f;
  const float mu_b = p1 * inv_g * (1.f / 32.f);
  return fmaf(fmaf(lam1_p, __builtin_sqrtf(p2 * inv_n1), wmu_p * mu_b), kBoundSlack, kBoundFloor);
}

// The tiles of the workgroup (local tile i: keys from key0 + 32 i on, codes at codes_w + 32 i, ref in
// ub[i]) in decreasing order of their bounds: a counting sort into bins of 1/16 of an octave below
// the largest bound, each tile standing for its bin's upper edge.  Out: order[j], ub[j] (the bound)
// of the j-th tile, *n_eval tiles in all (those with a candidate key), and the largest finite bound
// (returned; also in *bmax_bits, which starts at 0).  bins: 2 kOrderBins words.  Ends synchronised.
template <int NB, bool ALL, int NT>
__device__ __forceinline__ float order_tiles(const uint32_t* codes_w, int n_tiles, int key0, int n_cand,
                                             const float* bsh, float w_mu, float lam1, float inv_g,
                                             float* ub, uint16_t* order, uint32_t* bins,
                                             uint32_t* bmax_bits, uint32_t* n_eval, int tid) {
  constexpr int kTilesPerThread = kPruneMaxTiles / NT;
  static_assert(kPruneMaxTiles % NT == 0, "whole tiles per thread");
  const int lane = tid & 63, wave = tid >> 6;
  uint32_t* cnt = bins;                  // [kOrderBins] tiles per bin
  uint32_t* off = bins + kOrderBins;     // [kOrderBins] first position of each bin, then a cursor
  for (int i = tid; i < kOrderBins; i += NT) cnt[i] = 0u;
  const float wmu_p = fmaxf(w_mu, 0.f), lam1_p = fmaxf(lam1, 0.f);
  // the bounds of the thread's tiles tid + u NT (-inf: no candidate key, never revisited)
  float bnd[kTilesPerThread];
  float lmax = 0.f;  // largest finite bound (bounds are positive)
#pragma unroll
  for (int u = 0; u < kTilesPerThread; ++u) {
    const int i = tid + u * NT;
    bnd[u] = -INFINITY;
    if (i < n_tiles && key0 + i * kTileKeys < n_cand) {
      const float r = ub[i];
      float bd = INFINITY;
      if (r < INFINITY) bd = tile_bound<NB, ALL>(codes_w + 32 * i, r, bsh, wmu_p, lam1_p, inv_g);
      if (!(bd == bd)) bd = INFINITY;  // NaN inputs: revisit
      bnd[u] = bd;
      if (bd < INFINITY) lmax = fmaxf(lmax, bd);
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) lmax = fmaxf(lmax, __shfl_xor(lmax, o, 64));
  if (lane == 0) atomicMax(bmax_bits, __float_as_uint(lmax));  // positive floats order as integers
  __syncthreads();
  const float bmax = __uint_as_float(*bmax_bits);
  const float lg_max = __builtin_amdgcn_logf(bmax);  // log2; only used when a finite bound exists
  int bin[kTilesPerThread];
#pragma unroll
  for (int u = 0; u < kTilesPerThread; ++u) {
    bin[u] = -1;
    if (bnd[u] == INFINITY) {
      bin[u] = 0;
    } else if (bnd[u] > 0.f) {
      // bins counted down from the largest bound, rounded towards the larger bound (the bin's
      // upper edge stays above every bound in it despite the rounding of log2)
      const float x = (lg_max - __builtin_amdgcn_logf(bnd[u])) * kBinsPerOctave - (1.f / 64.f);
      bin[u] = 1 + (int)fminf(fmaxf(x, 0.f), (float)(kOrderBins - 2));
    }
    if (bin[u] >= 0) atomicAdd(&cnt[bin[u]], 1u);
  }
  __syncthreads();
  if (wave == 0) {
    // exclusive scan of the counts: lane l holds bins 16 l .. 16 l + 15
    constexpr int PB = kOrderBins / 64;
    uint32_t v[PB];
    uint32_t s = 0;
#pragma unroll
    for (int k = 0; k < PB; ++k) {
      v[k] = cnt[lane * PB + k];
      s += v[k];
    }
    uint32_t incl = s;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t t = (uint32_t)__shfl_up((int)incl, o, 64);
      if (lane >= o) incl += t;
    }
    uint32_t run = incl - s;
#pragma unroll
    for (int k = 0; k < PB; ++k) {
      off[lane * PB + k] = run;
      run += v[k];
    }
    if (lane == 63) *n_eval = incl;
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < kTilesPerThread; ++u) {
    if (bin[u] >= 0) {
      const uint32_t pos = atomicAdd(&off[bin[u]], 1u);
      order[pos] = (uint16_t)(tid + u * NT);
      ub[pos] = bin[u] == 0 ? INFINITY
                            : bmax * __builtin_amdgcn_exp2f(-(float)(bin[u] - 1) * (1.f / kBinsPerOctave));
    }
  }
  __syncthreads();
  return bmax;
}

}  // namespace
}  // namespace stream
}  // namespace kv
