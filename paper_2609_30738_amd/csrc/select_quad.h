// The greedy selection over more candidates than the Gram triangle takes (bf16, C > 256) and over
// fp32 keys (section 3.2, Eq. (2), (4)): the cosines to the last admitted key are formed in every
// step.
//
// A dot product is the sum of four chains, chain u over the u-th dwords of the row's 16-byte chunks,
// (a0 + a1) + (a2 + a3).  The four lanes of a quad take one chain each of the quad's 4 J candidates
// and keep those chains in registers, so a step reads each dword of the last admitted row once per
// lane instead of once per candidate; the chains are added with two DPP steps, after which lane u
// goes on with candidate 4 quad + u (slots tid, tid + QT: as many candidates as lanes).
//
// Bound by the latency of a step (its barrier and the exchanges around it), then by the chains'
// arithmetic.  The last admitted row is read either from a copy of all rows in LDS (LDS_ROWS), or
// from where the quad that holds a wave's best candidate has put it before the step's barrier, which
// takes longer but lets two workgroups share a CU.  With a candidate per lane, every lane reading the
// whole row from the LDS copy (128 broadcast 16-byte reads per step), a step at C = 512 took
// 0.95 us; from the copy chain by chain 0.73 us (0.58 without the chains); 2048 units of C = 512,
// B = 128 take 860 us by the second form, 1349 us before.
#pragma once

#include <float.h>

#include "common.h"
#include "compact_rows.h"

namespace kv {
namespace quad {

typedef uint32_t __attribute__((ext_vector_type(4))) u32x4;

template <int DT, int D> struct Geo {
  static constexpr int kDwords = D * (int)sizeof(typename Elem<DT>::T) / 4;  // dwords of a row
  static constexpr int kLen = kDwords / 4;                                   // dwords of a chain
  static constexpr int kGroups = kLen / 4;                                   // 16-byte reads of a chain
};

// A wave's best candidate of a step: its row, chain by chain, and 1 / |k|.
template <int DT, int D> struct alignas(16) Row {
  uint32_t chain[4][Geo<DT, D>::kLen];
  float inv;
  uint32_t pad[3];
};

// One dword of a chain: two bf16 products or one fp32 product, added to acc.
template <int DT> __device__ __forceinline__ float chain_step(uint32_t a, uint32_t b, float acc) {
  if constexpr (DT == kDtBf16) {
    typedef __bf16 __attribute__((ext_vector_type(2))) bf2;
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf2, a), __builtin_bit_cast(bf2, b), acc, false);
  } else {
    return fmaf(__uint_as_float(a), __uint_as_float(b), acc);
  }
}

template <int CTRL> __device__ __forceinline__ uint32_t dpp(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, false);
}

// (a0 + a1) + (a2 + a3) over the four lanes of a quad, in each of them.
__device__ __forceinline__ float quad_sum(float v) {
  v += __uint_as_float(dpp<0xB1>(__float_as_uint(v)));
  v += __uint_as_float(dpp<0x4E>(__float_as_uint(v)));
  return v;
}

// The value of index u (0 .. 3).
template <typename V> __device__ __forceinline__ V pick(V a, V b, V c, V d, int u) {
  return (u & 2) ? ((u & 1) ? d : c) : ((u & 1) ? b : a);
}

// Dword u of each of the four chunks that the lanes of the quad hold (lane e: chunk x).
__device__ __forceinline__ void transpose(const u32x4& x, uint32_t (&out)[4], int u) {
  out[0] = pick(dpp<0x00>(x[0]), dpp<0x00>(x[1]), dpp<0x00>(x[2]), dpp<0x00>(x[3]), u);
  out[1] = pick(dpp<0x55>(x[0]), dpp<0x55>(x[1]), dpp<0x55>(x[2]), dpp<0x55>(x[3]), u);
  out[2] = pick(dpp<0xAA>(x[0]), dpp<0xAA>(x[1]), dpp<0xAA>(x[2]), dpp<0xAA>(x[3]), u);
  out[3] = pick(dpp<0xFF>(x[0]), dpp<0xFF>(x[1]), dpp<0xFF>(x[2]), dpp<0xFF>(x[3]), u);
}

// LDS of the greedy: per step parity the waves' best candidates, their scores' order keys and slots
// and (without LDS_ROWS) their rows; with LDS_ROWS the rows of all candidates follow.
template <int DT, int D, int QT, bool LDS_ROWS> struct Shared {
  Row<DT, D> row[2][LDS_ROWS ? 0 : QT / 64];
  uint2 best[2][QT / 64];
  __device__ uint32_t* rows() { return reinterpret_cast<uint32_t*>(this + 1); }
  static constexpr size_t bytes(int max_cand) {
    return sizeof(Shared) + (LDS_ROWS ? (size_t)max_cand * Geo<DT, D>::kDwords * 4 : 0);
  }
};

typedef const __attribute__((address_space(1))) void* gptr;
typedef __attribute__((address_space(3))) void* lptr;

// The greedy by the first QT threads of the workgroup (the others keep step with the barriers) over
// the C candidates at positions cpos of the unit's keys kg: cst[c] = s~ of candidate c, cinv[c]
// receives 1 / |k| (LDS);
// trace_slot / trace_key [bp] out (LDS).  With want_corr, corr[j] afterwards holds the corr of the
// lane's slot tid + j QT when it was admitted or, if never, after the last step.  Every thread calls
// run after cpos and cst are visible; it ends unsynchronised.
template <int DT, int D, int QT, int J, bool LDS_ROWS> struct Greedy {
  using G = Geo<DT, D>;
  static constexpr int kWaves = QT / 64;
  static_assert(kWaves == 4 || kWaves == 8, "a record per lane of a quad or of half a DPP row");
  uint32_t key[J][4][G::kLen];
  float st[J], corr[J], inv[J];
  bool admitted[J];

  __device__ __forceinline__ void init(const typename Elem<DT>::T* __restrict__ kg, const int32_t* cpos,
                                       const float* cst, float* cinv, int C, int tid) {
    const int u = tid & 3;
    u32x4 x[J][4][G::kGroups];
#pragma unroll
    for (int j = 0; j < J; ++j)
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        // slots past C read the last candidate's row (never used)
        const int c = min((tid & ~3) + k + j * QT, C - 1);
        const u32x4* src = reinterpret_cast<const u32x4*>(kg + (size_t)cpos[c] * D);
#pragma unroll
        for (int i = 0; i < G::kGroups; ++i) x[j][k][i] = src[4 * i + u];
      }
#pragma unroll
    for (int j = 0; j < J; ++j) {
      float n2 = 0.f;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
#pragma unroll
        for (int i = 0; i < G::kGroups; ++i) {
          uint32_t o[4];
          transpose(x[j][k][i], o, u);
#pragma unroll
          for (int e = 0; e < 4; ++e) key[j][k][4 * i + e] = o[e];
        }
        float a = 0.f;
#pragma unroll
        for (int i = 0; i < G::kLen; ++i) a = chain_step<DT>(key[j][k][i], key[j][k][i], a);
        a = quad_sum(a);
        n2 = u == k ? a : n2;
      }
      const int c = tid + j * QT;
      admitted[j] = c >= C;  // slots past C never compete
      inv[j] = n2 > 0.f ? 1.f / sqrtf(n2) : 0.f;  // a zero key has cosine 0 to everything
      st[j] = c < C ? cst[c] : 0.f;
      corr[j] = 0.f;
      if (LDS_ROWS && c < C) cinv[c] = inv[j];
    }
  }
  // the rows of the C candidates chain by chain into LDS by nt threads: each load instruction of a
  // wave fills 64 dwords
  __device__ __forceinline__ static void stage_rows(const typename Elem<DT>::T* __restrict__ kg,
                                                    const int32_t* cpos, int C, uint32_t* rows, int tid, int nt) {
    const int lane = tid & 63;
    for (int s0 = tid - lane; s0 < C * G::kDwords; s0 += nt) {
      const int c = (s0 + lane) / G::kDwords, in = (s0 + lane) % G::kDwords;
      if (c < C)
        __builtin_amdgcn_global_load_lds(
            (gptr)(reinterpret_cast<const uint32_t*>(kg + (size_t)cpos[c] * D) + 4 * (in % G::kLen) + in / G::kLen),
            (lptr)(rows + s0), 4, 0, 0);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  }
  // corr against a row (its chain u at `chain`) with 1 / |k| last_inv
  __device__ __forceinline__ void update(const uint32_t* chain, float last_inv, int u) {
    uint32_t row[G::kLen];
#pragma unroll
    for (int i = 0; i < G::kGroups; ++i) {
      const u32x4 x = *reinterpret_cast<const u32x4*>(chain + 4 * i);
#pragma unroll
      for (int e = 0; e < 4; ++e) row[4 * i + e] = x[e];
    }
#pragma unroll
    for (int j = 0; j < J; ++j) {
      float a[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        a[k] = 0.f;
#pragma unroll
        for (int i = 0; i < G::kLen; ++i) a[k] = chain_step<DT>(key[j][k][i], row[i], a[k]);
        a[k] = quad_sum(a[k]);
      }
      const float cs = pick(a[0], a[1], a[2], a[3], u) * inv[j] * last_inv;
      if (!admitted[j]) corr[j] = fmaxf(corr[j], cs);
    }
  }
  // the row and 1 / |k| of the candidate that lane l of the wave owns in group j
  template <int JJ> __device__ __forceinline__ void put_row(Row<DT, D>& dst, int l, int lane) const {
    const int u = lane & 3;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if ((l & 3) == k && (lane >> 2) == (l >> 2)) {
#pragma unroll
        for (int i = 0; i < G::kGroups; ++i)
          *reinterpret_cast<u32x4*>(&dst.chain[u][4 * i]) =
              u32x4{key[JJ][k][4 * i], key[JJ][k][4 * i + 1], key[JJ][k][4 * i + 2], key[JJ][k][4 * i + 3]};
        if (u == k) dst.inv = inv[JJ];
      }
    }
  }

  __device__ __forceinline__ void run(const typename Elem<DT>::T* __restrict__ kg, const int32_t* cpos,
                                      const float* cst, float* cinv, int C, int bp, float lam2,
                                      Shared<DT, D, QT, LDS_ROWS>& sh, uint32_t* trace_slot,
                                      uint32_t* trace_key, int tid, int nt, bool want_corr) {
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), u = tid & 3;
    const bool live = wave < QT / 64;
    if (live) init(kg, cpos, cst, cinv, C, tid);
    if constexpr (LDS_ROWS) {
      stage_rows(kg, cpos, C, sh.rows(), tid, nt);
      __syncthreads();
    }
    auto update_last = [&](int t, int last) __attribute__((always_inline)) {  // admitted at step t
      if constexpr (LDS_ROWS) {
        update(sh.rows() + last * G::kDwords + u * G::kLen, cinv[last], u);
      } else {
        const Row<DT, D>& r = sh.row[t & 1][(last % QT) >> 6];
        update(r.chain[u], r.inv, u);
      }
    };
    int last = -1;
    for (int t = 0; t < bp; ++t) {
      if (live) {
        if (last >= 0) update_last(t - 1, last);
        float sc[J];
#pragma unroll
        for (int j = 0; j < J; ++j) {
          sc[j] = fmaf(lam2, corr[j], st[j]);
          if (!(sc[j] > -INFINITY)) sc[j] = -FLT_MAX;  // NaN or -inf still ranks above admitted slots
          if (admitted[j]) sc[j] = -INFINITY;
        }
        float lm = sc[0];
        if constexpr (J == 2) lm = fmaxf(sc[0], sc[J - 1]);
        const float wm = wave_max_uniform(lm);
        // the wave's lowest slot that holds it (slots ascend with the lane, group 1 after group 0)
        const uint64_t m0 = __ballot(sc[0] == wm);
        uint32_t slot;
        if (J == 1 || m0 != 0) {
          const int l = __ffsll((unsigned long long)m0) - 1;
          slot = 64u * (uint32_t)wave + (uint32_t)l;
          if constexpr (!LDS_ROWS) put_row<0>(sh.row[t & 1][wave], l, lane);
        } else {
          const int l = __ffsll((unsigned long long)__ballot(sc[J - 1] == wm)) - 1;
          slot = (uint32_t)QT + 64u * (uint32_t)wave + (uint32_t)l;
          if constexpr (!LDS_ROWS) put_row<J - 1>(sh.row[t & 1][wave], l, lane);
        }
        if (lane == 0) sh.best[t & 1][wave] = make_uint2(order_key(wm), slot);
      }
      __syncthreads();
      if (live) {
        // the waves' records, one per lane of each group of kWaves: the largest score, then the
        // lowest slot
        const uint2 r = sh.best[t & 1][lane & (kWaves - 1)];
        uint32_t km = r.x;
        km = max(km, dpp<0xB1>(km));
        km = max(km, dpp<0x4E>(km));
        if constexpr (kWaves > 4) km = max(km, dpp<0x141>(km));
        uint32_t sl = r.x == km ? r.y : ~0u;
        sl = min(sl, dpp<0xB1>(sl));
        sl = min(sl, dpp<0x4E>(sl));
        if constexpr (kWaves > 4) sl = min(sl, dpp<0x141>(sl));
        last = min((int)__builtin_amdgcn_readfirstlane(sl), C - 1);  // always a live slot: bp <= C
#pragma unroll
        for (int j = 0; j < J; ++j)
          if (tid + j * QT == last) admitted[j] = true;
        if (tid == 0) {
          // the step's record; written out after the last step
          trace_slot[t] = (uint32_t)last;
          trace_key[t] = km;
        }
      }
    }
    if (live && want_corr) update_last(bp - 1, last);
  }
};

}  // namespace quad
}  // namespace kv
