// Attention of one generated token per (sequence, layer) over its compacted cache (section 4.3:
// after eviction the model generates against the kept B + W rows of every layer).
//
// decode_kernel: one workgroup of 256 threads per (split of the rows, kv head, problem).  A row of
//   d elements is CH 16-byte chunks; thread t takes chunk t % CH of rows t / CH, t / CH + RPP, ...
//   (RPP = 256 / CH rows per pass), so a pass reads RPP whole consecutive rows of K and of V.  The
//   G query heads of the kv head share every loaded row.  The chunk dot products of a row are summed
//   over its CH lanes with DPP adds (a row of 128 bf16 is one DPP row of 16 lanes); every lane keeps,
//   per head, the sum of the weights 2^(t - m) and the weighted sum of its value chunk.  The
//   reference m is one value per wave and head, raised (and the sums rescaled) only when a logit
//   exceeds it by more than kSlack octaves, so an ordinary row costs one exponential per head and
//   no rescaling; weights are 2^(t - m - kSlack), exactly scaled after the exponential, so that none
//   exceeds 1 and large values keep finite sums (raised with every larger logit instead, splits of a
//   few steps pay: 2 problems of 9000 rows, G = 8: 46 us against 38).  The next rows load while the current ones are computed.  At the end the row
//   groups of a wave are added with lane swaps and the four waves merged through LDS.  With one
//   split the normalised output is written; with several, a partial (m, sum, weighted values) per
//   (head, split) goes to the workspace and decode_combine_kernel merges the splits.
//   If the token's own key / value are given, the split that holds row `len` attends to them from
//   the inputs and also writes them into row `len` of the cache block.
//   Bound by the cache reads for long caches: 256 units of 28672-32768 rows (4.03 GB, G = 4,
//   d = 128, bf16) take 704 us, 5.7 TB/s; with the row sums over ds_bpermute, two exponentials and
//   a rescale per row and head, and loads that waited for the step before, it was 1231 us
//   (3.3 TB/s).  Dot products by v_dot2_f32_bf16 instead of unpacked FMAs: 704 against 890 us at the
//   same error against 64 bits.  A kept cache of 96 rows is latency (9.6 us, before 12.3).
#include <math.h>

#include <algorithm>
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace kv {

namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;
constexpr int kMaxSplits = 2304;
// K and V of a launch from here on are read with the non-temporal bit: they outgrow the 256 MB
// last-level cache, so nothing of them is there at the next token (a smaller cache may be).
constexpr int64_t kNtBytes = (int64_t)256 << 20;
constexpr float kSlack = 8.f;           // octaves a logit may exceed its reference
constexpr float kSlackScale = 0x1p-8f;  // of the weights, so that none exceeds 1

typedef uint32_t __attribute__((ext_vector_type(4))) u32x4;
typedef __bf16 __attribute__((ext_vector_type(2))) bf16x2;

// One 16-byte chunk as fp32 values.
__device__ __forceinline__ void chunk_to_f32(const u32x4& u, float (&f)[8]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    f[2 * i] = __uint_as_float(u[i] << 16);
    f[2 * i + 1] = __uint_as_float(u[i] & 0xFFFF0000u);
  }
}
__device__ __forceinline__ void chunk_to_f32(const u32x4& u, float (&f)[4]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) f[i] = __uint_as_float(u[i]);
}

// Dot product of two chunks (fp32 accumulation).
template <int DT> __device__ __forceinline__ float chunk_dot(const u32x4& a, const u32x4& b) {
  float t = 0.f;
  if constexpr (DT == kDtBf16) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t x = a[i], y = b[i];
      t = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, x), __builtin_bit_cast(bf16x2, y), t, false);
    }
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) t = fmaf(__uint_as_float(a[i]), __uint_as_float(b[i]), t);
  }
  return t;
}

template <int CTRL> __device__ __forceinline__ float dpp_add(float v) {
  return v + __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(v), CTRL, 0xF, 0xF, false));
}
__device__ __forceinline__ float swap16_add(float v) {  // v + v of lane ^ 16
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float swap32_add(float v) {  // v + v of lane ^ 32
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Sum over the CH lanes of a row (CH = 8, 16 or 32 consecutive lanes), the same bits in each.
template <int CH> __device__ __forceinline__ float row_sum(float v) {
  static_assert(CH == 8 || CH == 16 || CH == 32, "lanes of a row");
  v = dpp_add<0xB1>(v);   // quad_perm [1,0,3,2]
  v = dpp_add<0x4E>(v);   // quad_perm [2,3,0,1]
  v = dpp_add<0x141>(v);  // row_half_mirror: the other quad of the 8 lanes
  if constexpr (CH >= 16) v = dpp_add<0x140>(v);  // row_mirror: the other 8 lanes
  if constexpr (CH >= 32) v = swap16_add(v);
  return v;
}

// Sum over the 64 / CH rows of a wave, per chunk position.
template <int CH> __device__ __forceinline__ float group_sum(float v) {
  if constexpr (CH <= 8) v = dpp_add<0x128>(v);  // row_ror:8
  if constexpr (CH <= 16) v = swap16_add(v);
  return swap32_add(v);
}

}  // namespace

// Rows per thread in a step and the wave count per SIMD that the registers are held to: the value
// sums take GM EPT registers, two steps of rows 16 kRows, and a spill costs more than the rows in
// flight give (G = 4 with kRows = 4 spilled at four waves: 2119 us against 704 at three and 2).
template <int GM, int EPT> constexpr int kRows = GM == 1 ? 4 : (GM * EPT <= 32 ? 2 : 1);
template <int GM> constexpr int kMinWaves = GM <= 2 ? 4 : (GM == 4 ? 3 : 2);

// NT: non-temporal cache reads (a cache too large to stay on the chip until the next token).
template <int DT, int D, int GM, bool NT>
__global__ __launch_bounds__(kThreads, kMinWaves<GM>) void decode_kernel(DecodeArgs a) {
  constexpr int EPT = 16 / (int)sizeof(typename Elem<DT>::T);  // elements of a 16-byte chunk
  constexpr int CH = D / EPT;                                  // chunks of a row
  constexpr int RPP = kThreads / CH;                           // rows per pass
  constexpr int U = kRows<GM, EPT>;  // rows per thread in a step (twice that in flight)
  __shared__ float sh_m[kWaves][GM];
  __shared__ float sh_s[kWaves][GM];
  __shared__ __align__(16) float sh_acc[kWaves][GM][D];

  const int split = blockIdx.x, g = blockIdx.y, p = blockIdx.z;
  const int G = a.h_q / a.h_kv;
  const int len = a.lens[p];
  const bool append = a.k_new != nullptr;
  const int total = len + (append ? 1 : 0);
  const int r0 = split * a.split_rows;
  const int r1 = min(total, r0 + a.split_rows);
  const int tid = threadIdx.x, rg = tid / CH, c = tid % CH, wave = tid / 64, lane = tid % 64;

  const size_t unit = (size_t)p * a.h_kv + g;
  const u32x4* kc = static_cast<const u32x4*>(a.k) + unit * a.row_stride * CH;
  const u32x4* vc = static_cast<const u32x4*>(a.v) + unit * a.row_stride * CH;

  // rows rb + u RPP + rg of this thread: a whole step of cache rows (the step's rows are contiguous,
  // thread t takes its chunk t), or, at the end of the split, row by row (r == len: the appended
  // row; rows past the split re-read its last one)
  struct Rows {
    u32x4 k[U], v[U];
  };
  const int r_in = min(r1, len);  // rows of the split that come from the cache
  auto load = [&](Rows& x, int rb) __attribute__((always_inline)) {
    if (rb + U * RPP <= r_in) {
      const u32x4* ks = kc + (size_t)rb * CH;
      const u32x4* vs = vc + (size_t)rb * CH;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        x.k[u] = NT ? __builtin_nontemporal_load(ks + u * kThreads + tid) : ks[u * kThreads + tid];
        x.v[u] = NT ? __builtin_nontemporal_load(vs + u * kThreads + tid) : vs[u * kThreads + tid];
      }
    } else {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int r = min(rb + u * RPP + rg, r1 - 1);
        x.k[u] = *(r < len ? kc + (size_t)r * CH + c : static_cast<const u32x4*>(a.k_new) + unit * CH + c);
        x.v[u] = *(r < len ? vc + (size_t)r * CH + c : static_cast<const u32x4*>(a.v_new) + unit * CH + c);
      }
    }
  };
  constexpr int kStep = U * RPP;
  Rows xa, xb;
  if (r0 < r1) load(xa, r0);
  if (r0 + kStep < r1) load(xb, r0 + kStep);

  // the query chunks of the group's heads
  u32x4 qu[GM];
#pragma unroll
  for (int h = 0; h < GM; ++h) {
    qu[h] = u32x4{0u, 0u, 0u, 0u};
    if (h < G) qu[h] = static_cast<const u32x4*>(a.q)[((size_t)p * a.h_q + (size_t)g * G + h) * CH + c];
  }

  float m[GM], s[GM], acc[GM][EPT];
#pragma unroll
  for (int h = 0; h < GM; ++h) {
    m[h] = -INFINITY;
    s[h] = 0.f;
#pragma unroll
    for (int e = 0; e < EPT; ++e) acc[h][e] = 0.f;
  }

  auto compute = [&](const Rows& x, int rb, auto masked) __attribute__((always_inline)) {
    constexpr bool kMasked = decltype(masked)::value;
    float t[U][GM];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int h = 0; h < GM; ++h) {
        t[u][h] = row_sum<CH>(chunk_dot<DT>(qu[h], x.k[u])) * a.c;  // base 2
        if (kMasked && rb + u * RPP + rg >= r1) t[u][h] = -INFINITY;
      }
    bool over = false;
#pragma unroll
    for (int h = 0; h < GM; ++h) {
      float tm = t[0][h];
#pragma unroll
      for (int u = 1; u < U; ++u) tm = fmaxf(tm, t[u][h]);
      over = over || tm > m[h] + kSlack;
    }
    if (__ballot(over)) {
#pragma unroll
      for (int h = 0; h < GM; ++h) {
        float tm = t[0][h];
#pragma unroll
        for (int u = 1; u < U; ++u) tm = fmaxf(tm, t[u][h]);
        const float mn = fmaxf(m[h], wave_max_uniform(tm));
        const float f = m[h] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m[h] - mn);
        s[h] *= f;
#pragma unroll
        for (int e = 0; e < EPT; ++e) acc[h][e] *= f;
        m[h] = mn;
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float vf[EPT];
      chunk_to_f32(x.v[u], vf);
#pragma unroll
      for (int h = 0; h < GM; ++h) {
        float w = __builtin_amdgcn_exp2f(t[u][h] - m[h]) * kSlackScale;
        if (kMasked && rb + u * RPP + rg >= r1) w = 0.f;
        s[h] += w;
#pragma unroll
        for (int e = 0; e < EPT; ++e) acc[h][e] = fmaf(w, vf[e], acc[h][e]);
      }
    }
  };
  auto step = [&](const Rows& x, int rb) __attribute__((always_inline)) {
    if (rb + kStep <= r1) compute(x, rb, std::false_type{});
    else compute(x, rb, std::true_type{});
  };
  for (int rb = r0; rb < r1; rb += 2 * kStep) {
    step(xa, rb);
    if (rb + 2 * kStep < r1) load(xa, rb + 2 * kStep);
    if (rb + kStep < r1) {
      step(xb, rb + kStep);
      if (rb + 3 * kStep < r1) load(xb, rb + 3 * kStep);
    }
  }
  if (append && len >= r0 && len < r1 && rg == 0) {  // the new row joins the cache
    static_cast<u32x4*>(a.k)[(unit * a.row_stride + len) * CH + c] =
        static_cast<const u32x4*>(a.k_new)[unit * CH + c];
    static_cast<u32x4*>(a.v)[(unit * a.row_stride + len) * CH + c] =
        static_cast<const u32x4*>(a.v_new)[unit * CH + c];
  }

  // the row groups of each wave (lanes c, c + CH, ... hold the same chunk; one m per wave)
#pragma unroll
  for (int h = 0; h < GM; ++h) {
    s[h] = group_sum<CH>(s[h]);
#pragma unroll
    for (int e = 0; e < EPT; ++e) acc[h][e] = group_sum<CH>(acc[h][e]);
  }
  if (lane < CH) {
#pragma unroll
    for (int h = 0; h < GM; ++h) {
      if (c == 0) {
        sh_m[wave][h] = m[h];
        sh_s[wave][h] = s[h];
      }
#pragma unroll
      for (int e = 0; e < EPT; e += 4)
        *reinterpret_cast<float4*>(&sh_acc[wave][h][c * EPT + e]) =
            make_float4(acc[h][e], acc[h][e + 1], acc[h][e + 2], acc[h][e + 3]);
    }
  }
  __syncthreads();
  for (int idx = tid; idx < G * D; idx += kThreads) {
    const int h = idx / D, e = idx % D;
    float M = -INFINITY;
#pragma unroll
    for (int i = 0; i < kWaves; ++i) M = fmaxf(M, sh_m[i][h]);
    float S = 0.f, A = 0.f;
#pragma unroll
    for (int i = 0; i < kWaves; ++i) {
      const float mi = sh_m[i][h];
      const float f = mi == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mi - M);
      S = fmaf(sh_s[i][h], f, S);
      A = fmaf(sh_acc[i][h][e], f, A);
    }
    const size_t row = (size_t)p * a.h_q + (size_t)g * G + h;
    if (a.n_split == 1) {
      a.out[row * D + e] = A / S;
    } else {
      float* pt = a.part + (row * a.n_split + split) * (D + 2);
      if (e == 0) {
        pt[0] = M;
        pt[1] = S;
      }
      pt[2 + e] = A;
    }
  }
}

// One workgroup per (problem, q head): the splits' weights 2^(m_i - M) in LDS, then every thread
// sums one element over a share of the splits.
template <int D>
__global__ __launch_bounds__(kThreads) void decode_combine_kernel(const float* __restrict__ part,
                                                                  int n_split,
                                                                  float* __restrict__ out) {
  constexpr int PARTS = kThreads / D;
  __shared__ float f[kMaxSplits];
  __shared__ float red[kWaves];
  __shared__ float sum[PARTS][D + 1];
  const int tid = threadIdx.x, e = tid % D, pt = tid / D;
  const float* row = part + (size_t)blockIdx.x * n_split * (D + 2);
  float m = -INFINITY;
  for (int i = tid; i < n_split; i += kThreads) {
    f[i] = row[(size_t)i * (D + 2)];
    m = fmaxf(m, f[i]);
  }
  m = wave_max_uniform(m);
  if ((tid & 63) == 0) red[tid >> 6] = m;
  __syncthreads();
  const float M = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
  static_assert(kWaves == 4, "four waves");
  float A = 0.f, S = 0.f;
#pragma unroll 4
  for (int i = pt; i < n_split; i += PARTS) {
    const float w = f[i] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(f[i] - M);
    S = fmaf(row[(size_t)i * (D + 2) + 1], w, S);
    A = fmaf(row[(size_t)i * (D + 2) + 2 + e], w, A);
  }
  sum[pt][e] = A;
  if (e == 0) sum[pt][D] = S;
  __syncthreads();
  if (pt == 0) {
#pragma unroll
    for (int q = 1; q < PARTS; ++q) {
      A += sum[q][e];
      S += sum[q][D];
    }
    // every thread of part 0 holds the same S
    out[(size_t)blockIdx.x * D + e] = A / S;
  }
}

namespace {

template <int DT, int D, bool NT>
void decode_groups(const DecodeArgs& a, const dim3& grid, hipStream_t st) {
  const int G = a.h_q / a.h_kv;
  if (G == 1) decode_kernel<DT, D, 1, NT><<<grid, kThreads, 0, st>>>(a);
  else if (G == 2) decode_kernel<DT, D, 2, NT><<<grid, kThreads, 0, st>>>(a);
  else if (G <= 4) decode_kernel<DT, D, 4, NT><<<grid, kThreads, 0, st>>>(a);
  else decode_kernel<DT, D, 8, NT><<<grid, kThreads, 0, st>>>(a);
}

template <int DT, int D>
hipError_t decode_dispatch(const DecodeArgs& a, int n_prob, hipStream_t st) {
  const dim3 grid((unsigned)a.n_split, (unsigned)a.h_kv, (unsigned)n_prob);
  // K and V of the launch (rows up to the longest cache)
  const int64_t bytes = (int64_t)n_prob * a.h_kv * a.n_split * a.split_rows * D * 2 *
                        (int64_t)sizeof(typename Elem<DT>::T);
  if (bytes >= kNtBytes) decode_groups<DT, D, true>(a, grid, st);
  else decode_groups<DT, D, false>(a, grid, st);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || a.n_split == 1) return e;
  decode_combine_kernel<D><<<(unsigned)(n_prob * a.h_q), kThreads, 0, st>>>(a.part, a.n_split, a.out);
  return hipGetLastError();
}

}  // namespace

DecodePlan decode_plan(int n_prob, int h_kv, int max_len, int group, int row_bytes) {
  // Up to one_split rows a unit stays whole, a launch less: 300 rows of 64 units (G = 4, d = 128, bf16)
  // take 12.0 us whole and 12.8 us split and merged, 500 rows of 8 units 15.8 and 12.8 us.  A row costs
  // about its bytes times the heads: where these are at most kLightRow, 500 rows of 8 to 256 units take
  // 9.6 to 13.5 us whole and 11.9 to 15.4 split (G = 1 at 128 to 512 bytes a row, G = 2 at 128 and 256,
  // G = 4 at 128); G = 4 at 256 bytes (d = 64, fp32) 13.2 to 16.3 and 11.9 to 15.9.  Long caches get about three rounds of
  // the 768 workgroups that fit the chip at once (three per CU), so that caches of unequal length
  // even out (768 workgroups 717 us, 1536 703, 2304 706, 6144 729 at 256 units of 32768 rows);
  // where that leaves fewer than 1024 rows to a split, one round of splits of at least kMinSplit
  // rows (2000 rows of 8 units: 11.4 us, at least 256 rows 12.6 us).
  constexpr int64_t kMinSplit = 128, kStep = 64, kRound = 768;
  constexpr int kLightRow = 512;
  const int64_t one_split = group * row_bytes <= kLightRow ? 512 : 384;
  static_assert(3 * kRound <= kMaxSplits, "the merge holds every split's weight");
  const int64_t units = (int64_t)n_prob * h_kv;
  const int64_t rows = (int64_t)max_len + 1;  // room for an appended row
  auto splits = [&](int64_t groups) { return std::max<int64_t>(1, groups / units); };
  int64_t n_split = 1;
  if (rows > one_split) {
    n_split = splits(3 * kRound);
    if (rows < 1024 * n_split) n_split = std::min(splits(kRound), (rows + kMinSplit - 1) / kMinSplit);
  }
  DecodePlan plan;
  plan.ws_splits = (int)n_split;
  int64_t split_rows = (rows + n_split - 1) / n_split;
  split_rows = (split_rows + kStep - 1) / kStep * kStep;
  n_split = (rows + split_rows - 1) / split_rows;
  plan.n_split = (int)n_split;
  plan.split_rows = (int)split_rows;
  return plan;
}

size_t decode_ws_bytes(int n_prob, int h_q, int d, const DecodePlan& plan) {
  if (plan.ws_splits == 1) return 0;
  return (size_t)n_prob * h_q * plan.ws_splits * (d + 2) * sizeof(float);
}

hipError_t launch_decode(int dtype, int d, int n_prob, const DecodeArgs& a, hipStream_t stream) {
  if (dtype == kDtBf16)
    return d == 64 ? decode_dispatch<kDtBf16, 64>(a, n_prob, stream)
                   : decode_dispatch<kDtBf16, 128>(a, n_prob, stream);
  return d == 64 ? decode_dispatch<kDtF32, 64>(a, n_prob, stream)
                 : decode_dispatch<kDtF32, 128>(a, n_prob, stream);
}

}  // namespace kv
