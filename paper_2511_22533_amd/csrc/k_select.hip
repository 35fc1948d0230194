// Spatiotemporal Stability Criterion scoring and lowest-score selection
// (Sec. 4.2, Eqs. 2, 6, 7; Algorithm 1, SSC).
//
// k_score_stats streams the two velocity caches over the whole chip (one
// 256-thread workgroup per 1024 tokens of a sample): V_i = ||v_cache_i|| and
// A_i = ||v_cache_i - v_prev_i|| with a sequential float32 sum of squares (no
// fused multiply-add, correctly rounded sqrt), written as (V_i, A_i) pairs,
// and each workgroup's min/max of both. min/max are exact and order-free
// (the magnitudes are never -0; NaN is ignored), so the per-sample extremes do
// not depend on how the tokens are split.
//
// The score C_i = w_a * norm(A_i) + w_v * norm(V_i) gives an order-preserving
// 32-bit key (NaN -> largest). From 8193 tokens a second grid-wide kernel
// (k_keys) forms the keys and a 4096-bin histogram of the scores; below, the
// selecting workgroup does both itself.
//
// k_select runs one 1024-thread workgroup per sample with the keys in
// registers, each wave owning one contiguous run of tokens. The score bin that
// holds rank c-1 comes from the histogram; while a bin holds many keys (crowded
// or equal scores), its key range is cut into 4096 bins again. The few keys left
// are ranked against each other, which gives the key of rank c-1. A token is
// cached if its key is smaller, or equal and among the first r equal keys in token
// order, which reproduces a stable ascending sort truncated at c.
#include <mutex>
#include <type_traits>
#include <vector>

#include "common.h"
#include "kernels.h"

#pragma clang fp contract(off)

namespace f3c {

namespace {

constexpr int kThreads = 1024;       // select: one workgroup per sample
constexpr int kWaves = kThreads / 64;
static_assert(kWaves == 16, "the waves' values are reduced in a row of 16 lanes");
constexpr int kStatThreads = 256;    // score statistics: tokens streamed over the chip
constexpr int kStatPer = 4;
constexpr int kChunk = kStatThreads * kStatPer;
constexpr int kMaxChunks = kMaxTokens / kChunk;
static_assert(kMaxChunks <= 64, "the partial extremes are reduced in one wave");
constexpr int kBins = 4096;          // score bins: [0, 1) in steps of 2^-12, NaN and 1 in the last
constexpr int kCandidates = 128;     // keys of one bin that are ranked against each other (a power of two)
// One workgroup issues an instruction for 32768 tokens in 0.2 us, so for many
// tokens the keys (two correctly rounded divisions each) and their histogram
// are worth a grid-wide kernel of their own. Measured on MI355X, batch 1, all
// kernels, keys in k_select / in k_keys: 8193 tokens 16.2 / 16.1 us, 16384
// 17.6 / 17.0, 32768 35.0 / 24.8 (before the scans left the LDS pipe, which takes
// 0.6 us off either). Against four radix passes over keys in LDS: 512 tokens 9.8
// -> 6.0 us, 4096 16.4 -> 8.9, 32768 67.2 -> 23.9; scores crowded around one value
// 9.9 -> 7.7, 17.0 -> 12.5, 68.4 -> 42.2; all equal 9.4 -> 7.6, 16.0 -> 11.0, 64.5
// -> 35.1.
constexpr int kFusedTokens = 8192;
static_assert(kBins <= kFusedTokens, "the histogram lives in the sample's pos rows");

__device__ __forceinline__ float sumsq8(const float4& a, const float4& b) {
  float s = 0.0f;
  s = __fadd_rn(s, __fmul_rn(a.x, a.x));
  s = __fadd_rn(s, __fmul_rn(a.y, a.y));
  s = __fadd_rn(s, __fmul_rn(a.z, a.z));
  s = __fadd_rn(s, __fmul_rn(a.w, a.w));
  s = __fadd_rn(s, __fmul_rn(b.x, b.x));
  s = __fadd_rn(s, __fmul_rn(b.y, b.y));
  s = __fadd_rn(s, __fmul_rn(b.z, b.z));
  s = __fadd_rn(s, __fmul_rn(b.w, b.w));
  return s;
}

__device__ __forceinline__ float4 sub4(const float4& a, const float4& b) {
  return make_float4(__fsub_rn(a.x, b.x), __fsub_rn(a.y, b.y), __fsub_rn(a.z, b.z), __fsub_rn(a.w, b.w));
}

__device__ __forceinline__ uint32_t order_key(float c) {
  if (c != c) return 0xFFFFFFFFu;
  if (c == 0.0f) c = 0.0f;                          // -0 orders with +0
  uint32_t u = __float_as_uint(c);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Correctly rounded float32 square root and quotient. (The library is built
// with -fhip-fp32-correctly-rounded-divide-sqrt; the __fsqrt_rn intrinsic maps to
// the approximate native instruction and is not used.)
__device__ __forceinline__ float sqrt_rn(float x) { return __builtin_sqrtf(x); }
__device__ __forceinline__ float div_rn(float a, float b) { return a / b; }

__device__ __forceinline__ float norm_term(float a, float lo, float hi) {
  if (!(hi > lo)) return 0.0f;
  return div_rn(__fsub_rn(a, lo), __fsub_rn(hi, lo));
}

__device__ __forceinline__ float score_of(const float2& va, const float4& ext, float w_a, float w_v) {
  return __fadd_rn(__fmul_rn(w_a, norm_term(va.y, ext.z, ext.w)), __fmul_rn(w_v, norm_term(va.x, ext.x, ext.y)));
}

// Bin of a score's key. Scores are >= 0 (or NaN), so the key is the score's
// bits with the sign bit set; the product is exact and both steps are
// monotonic, so a smaller key never has a larger bin. fminf drops NaN.
__device__ __forceinline__ int bin_of(uint32_t key) {
  return (int)fminf(__uint_as_float(key & 0x7FFFFFFFu) * (float)kBins, (float)(kBins - 1));
}

// Smallest key of a bin: its score is exact.
__device__ __forceinline__ uint32_t bin_start(int bin) {
  return __float_as_uint((float)bin * (1.0f / (float)kBins)) | 0x80000000u;
}

// bins[bin] += 1 over the active lanes. Same-address atomics of one instruction
// serialise, and scores may crowd into one bin (8192 such tokens: 20.4 us, 24.6
// with an atomic per lane; spread ones 11.8 and 11.6).
__device__ __forceinline__ void count_one(int* bins, int bin) {
  const int b0 = __builtin_amdgcn_readfirstlane(bin);
  const uint64_t m = __ballot(1);
  if (__ballot(bin != b0) != 0) atomicAdd(&bins[bin], 1);
  else if ((int)(threadIdx.x & 63) == __ffsll((unsigned long long)m) - 1) atomicAdd(&bins[b0], (int)__popcll(m));
}

// The same over the lanes with `in`, where a few bins may hold most: the lanes that
// share the first one's bin add their number at once.
__device__ __forceinline__ void count_in(int* bins, bool in, int bin) {
  const uint64_t m = __ballot(in);
  if (!m) return;
  const int leader = __ffsll((unsigned long long)m) - 1;
  const uint64_t same = __ballot(in && bin == __builtin_amdgcn_readlane(bin, leader));
  const int lane = threadIdx.x & 63;
  if (in && (lane == leader || !((same >> lane) & 1ull)))
    atomicAdd(&bins[bin], lane == leader ? (int)__popcll(same) : 1);
}

// The smallest value in each row of 16 lanes, in all of them.
__device__ __forceinline__ uint32_t row_min(uint32_t v) {
  auto with = [&](auto ctrl) {
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, decltype(ctrl)::value, 0xf, 0xf, false));
  };
  with(std::integral_constant<int, kDppXor8>{});
  with(std::integral_constant<int, kDppMirror8>{});
  with(std::integral_constant<int, kDppXor2>{});
  with(std::integral_constant<int, kDppXor1>{});
  return v;
}
// Inclusive sums over the lanes of a wave (the LDS pipe's __shfl_up takes six
// round trips of its latency).
__device__ __forceinline__ int wave_scan(int x) {
  auto with = [&](auto ctrl) {
    x += __builtin_amdgcn_update_dpp(0, x, decltype(ctrl)::value, 0xf, 0xf, false);
  };
  with(std::integral_constant<int, 0x111>{});       // row_shr: from 1, 2, 4, 8 lanes before, or 0
  with(std::integral_constant<int, 0x112>{});
  with(std::integral_constant<int, 0x114>{});
  with(std::integral_constant<int, 0x118>{});
  const int r0 = __builtin_amdgcn_readlane(x, 15), r1 = __builtin_amdgcn_readlane(x, 31);
  const int r2 = __builtin_amdgcn_readlane(x, 47), row = (threadIdx.x >> 4) & 3;
  return x + (row == 0 ? 0 : row == 1 ? r0 : row == 2 ? r0 + r1 : r0 + r1 + r2);
}
// Sum of cnt over the waves before this one, the same in every lane.
__device__ __forceinline__ int waves_before(const int* cnt, int wave) {
  const int w = threadIdx.x & (kWaves - 1);
  int v = cnt[w];
  v = w < wave ? v : 0;
  auto with = [&](auto ctrl) {
    v += __builtin_amdgcn_update_dpp(0, v, decltype(ctrl)::value, 0xf, 0xf, false);
  };
  with(std::integral_constant<int, kDppXor8>{});
  with(std::integral_constant<int, kDppMirror8>{});
  with(std::integral_constant<int, kDppXor2>{});
  with(std::integral_constant<int, kDppXor1>{});
  return __builtin_amdgcn_readfirstlane(v);
}
// Smallest value in the wave.
__device__ __forceinline__ uint32_t wave_min(uint32_t v) {
  v = row_min(v);
  auto row = [&](int l) { return (uint32_t)__builtin_amdgcn_readlane((int)v, l); };
  return min(min(row(0), row(16)), min(row(32), row(48)));
}

// The sample's extremes (loV, hiV, loA, hiA) from its partials, by one wave.
__device__ __forceinline__ float4 reduce_extremes(const float4* partial, int chunks, int lane) {
  float4 m = lane < chunks ? partial[lane] : make_float4(INFINITY, -INFINITY, INFINITY, -INFINITY);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    m.x = fminf(m.x, __shfl_xor(m.x, o));
    m.y = fmaxf(m.y, __shfl_xor(m.y, o));
    m.z = fminf(m.z, __shfl_xor(m.z, o));
    m.w = fmaxf(m.w, __shfl_xor(m.w, o));
  }
  return m;
}

// (V_i, A_i) of every token of the samples with c_b > 0, and each
// workgroup's extremes (loV, hiV, loA, hiA) at partial[b * chunks + chunk].
// hist (may be null): [B][N] ints whose first kBins per sample are zeroed for
// k_keys.
__global__ __launch_bounds__(kStatThreads) void k_score_stats(const float* __restrict__ v_cache,
                                                             const float* __restrict__ v_prev, int N, Segs n_cache,
                                                             float2* __restrict__ va, float4* __restrict__ partial,
                                                             int chunks, int32_t* __restrict__ hist) {
  __shared__ float4 red[kStatThreads / 64];
  const int b = blockIdx.y, chunk = blockIdx.x;
  if (n_cache.off[b] == 0) return;
  const int tid = threadIdx.x;
  const size_t base = (size_t)b * N;
  float4 c0[kStatPer], c1[kStatPer], p0[kStatPer], p1[kStatPer];
#pragma unroll
  for (int j = 0; j < kStatPer; ++j) {
    const int i = min(chunk * kChunk + j * kStatThreads + tid, N - 1);   // clamped: loads stay in bounds
    const float4* pc = reinterpret_cast<const float4*>(v_cache + (base + i) * 8);
    const float4* pp = reinterpret_cast<const float4*>(v_prev + (base + i) * 8);
    c0[j] = pc[0];
    c1[j] = pc[1];
    p0[j] = pp[0];
    p1[j] = pp[1];
  }
  if (hist && chunk * kChunk < kBins) {
#pragma unroll
    for (int j = 0; j < kStatPer; ++j) hist[base + chunk * kChunk + j * kStatThreads + tid] = 0;
  }
  float loV = INFINITY, hiV = -INFINITY, loA = INFINITY, hiA = -INFINITY;
#pragma unroll
  for (int j = 0; j < kStatPer; ++j) {
    const int i = chunk * kChunk + j * kStatThreads + tid;
    if (i < N) {
      const float V = sqrt_rn(sumsq8(c0[j], c1[j]));
      const float A = sqrt_rn(sumsq8(sub4(c0[j], p0[j]), sub4(c1[j], p1[j])));
      va[base + i] = make_float2(V, A);
      loV = fminf(loV, V);
      hiV = fmaxf(hiV, V);
      loA = fminf(loA, A);
      hiA = fmaxf(hiA, A);
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    loV = fminf(loV, __shfl_xor(loV, o));
    hiV = fmaxf(hiV, __shfl_xor(hiV, o));
    loA = fminf(loA, __shfl_xor(loA, o));
    hiA = fmaxf(hiA, __shfl_xor(hiA, o));
  }
  if ((tid & 63) == 0) red[tid >> 6] = make_float4(loV, hiV, loA, hiA);
  __syncthreads();
  if (tid == 0) {
    float4 m = red[0];
#pragma unroll
    for (int w = 1; w < kStatThreads / 64; ++w) {
      m.x = fminf(m.x, red[w].x);
      m.y = fmaxf(m.y, red[w].y);
      m.z = fminf(m.z, red[w].z);
      m.w = fmaxf(m.w, red[w].w);
    }
    partial[(size_t)b * chunks + chunk] = m;
  }
}

// Score (when asked for), key and histogram of every token of the samples with
// c_b > 0, one workgroup per chunk as in k_score_stats. A chunk's keys replace
// its magnitude pairs: chunk c's 1024 keys start where its pairs did.
__global__ __launch_bounds__(kStatThreads) void k_keys(float2* __restrict__ va, const float4* __restrict__ partial,
                                                       int chunks, int N, float w_a, float w_v, Segs n_cache,
                                                       int32_t* __restrict__ hist, float* __restrict__ score) {
  __shared__ int bins[kBins];
  __shared__ float4 ext_s;
  const int b = blockIdx.y, chunk = blockIdx.x;
  if (n_cache.off[b] == 0) return;
  const int tid = threadIdx.x;
  const size_t base = (size_t)b * N;
  float2 p[kStatPer];
#pragma unroll
  for (int j = 0; j < kStatPer; ++j) p[j] = va[base + min(chunk * kChunk + j * kStatThreads + tid, N - 1)];
  for (int i = tid; i < kBins; i += kStatThreads) bins[i] = 0;
  if (tid < 64) {
    const float4 m = reduce_extremes(partial + (size_t)b * chunks, chunks, tid);
    if (tid == 0) ext_s = m;
  }
  wait_vm<0>();                                     // every pair of the chunk read before keys replace them
  __syncthreads();
  const float4 ext = ext_s;
  uint32_t* keys = reinterpret_cast<uint32_t*>(va + base + (size_t)chunk * kChunk);
#pragma unroll
  for (int j = 0; j < kStatPer; ++j) {
    const int l = j * kStatThreads + tid, i = chunk * kChunk + l;
    const float cs = score_of(p[j], ext, w_a, w_v);
    const uint32_t k = order_key(cs);
    if (i < N) {
      keys[l] = k;
      if (score) score[base + i] = cs;
    }
    if (i < N) count_one(bins, bin_of(k));
  }
  __syncthreads();
  for (int i = tid; i < kBins; i += kStatThreads)
    if (bins[i]) atomicAdd(&hist[base + i], bins[i]);
}

enum KeySource { KEYS_READY, KEYS_FROM_STATS, KEYS_FROM_SCORES };

// The selection. Wave w owns tokens w * 64 R .. (w + 1) * 64 R - 1 (R rounds
// of 64, at most KR), so ranks in token order need only per-wave counts.
//   KEYS_READY: k_keys left the keys in the workspace and the histogram in pos.
//   KEYS_FROM_STATS: keys and histogram are formed here from the pairs.
//   KEYS_FROM_SCORES: any float32 scores given; the first bins cut the range of
//     all keys.
template <int SRC, int KR>
__global__ __launch_bounds__(kThreads) void k_select(const float2* __restrict__ va, const float4* __restrict__ partial,
                                                     int chunks, int N, float w_a, float w_v, Segs n_cache, Segs act,
                                                     int32_t* __restrict__ idx_active, int32_t* __restrict__ pos,
                                                     float* __restrict__ score, const float* __restrict__ given) {
  __shared__ int bins[kBins];
  __shared__ uint32_t cand[kCandidates];
  __shared__ int wave_cnt[2][kWaves];
  __shared__ uint32_t wave_range[2][kWaves], own_keys[KR][kThreads];
  __shared__ int sel[3], n_cand;
  __shared__ float4 ext_s;

  const int b = blockIdx.x;
  const int tid = threadIdx.x;
  const int c = n_cache.off[b];
  const int row0 = act.off[b];
  const size_t base = (size_t)b * N;
  const int lane = tid & 63, wave = tid >> 6;

  if (c == 0) {  // full step for this sample: identity selection, no scoring
    for (int i = tid; i < N; i += kThreads) {
      idx_active[row0 + i] = i;
      pos[base + i] = row0 + i;
    }
    return;
  }

  const int R = (N + kThreads - 1) / kThreads;
  const int i0 = wave * 64 * R + lane;              // this lane's token of round j: i0 + 64 j
  uint32_t key[KR];                                 // past the end the last token's again: see holds
  if (tid == 0) n_cand = 0;
  if constexpr (SRC == KEYS_READY) {
#pragma unroll
    for (int j = 0; j < KR; ++j) {
      const int i = min(i0 + 64 * j, N - 1), ch = i / kChunk;
      key[j] = reinterpret_cast<const uint32_t*>(va + base + (size_t)ch * kChunk)[i - ch * kChunk];
    }
  } else if constexpr (SRC == KEYS_FROM_SCORES) {
#pragma unroll
    for (int j = 0; j < KR; ++j) key[j] = order_key(given[base + min(i0 + 64 * j, N - 1)]);
  } else {
    float2 p[KR];
#pragma unroll
    for (int j = 0; j < KR; ++j) p[j] = va[base + min(i0 + 64 * j, N - 1)];
    for (int i = tid; i < kBins; i += kThreads) bins[i] = 0;
    if (wave == 0) {
      const float4 m = reduce_extremes(partial + (size_t)b * chunks, chunks, lane);
      if (lane == 0) ext_s = m;
    }
    __syncthreads();
    const float4 ext = ext_s;
#pragma unroll
    for (int j = 0; j < KR; ++j) {
      const int i = i0 + 64 * j;
      const float cs = score_of(p[j], ext, w_a, w_v);
      key[j] = order_key(cs);
      const bool in = j < R && i < N;
      if (score && in) score[base + i] = cs;
      if (in) count_one(bins, bin_of(key[j]));
    }
  }
  __syncthreads();
  // whether this lane holds a token in round j
  auto holds = [&](int j) { return j < R && i0 + 64 * j < N; };

  // The bin that holds rank r (1-based), given four consecutive bins per thread:
  // a scan over the wave, the waves before it added up. sel: bin, rank in it, its count.
  auto locate = [&](const int (&h)[4], int r) {
    const int tot = h[0] + h[1] + h[2] + h[3];
    const int x = wave_scan(tot);
    if (lane == 63) wave_cnt[0][wave] = x;
    __syncthreads();
    int before = x - tot + waves_before(wave_cnt[0], wave);
    if (before < r && r <= before + tot) {
      int d = 0;
#pragma unroll
      for (int e = 0; e < 3; ++e)
        if (d == e && before + h[e] < r) {
          before += h[e];
          d = e + 1;
        }
      sel[0] = 4 * tid + d;
      sel[1] = r - before;
      sel[2] = d == 0 ? h[0] : d == 1 ? h[1] : d == 2 ? h[2] : h[3];
    }
    __syncthreads();
  };
  // The key of rank c-1 and how many of the keys equal to it are cached: it is the
  // r-th smallest of the m keys in lo .. hi.
  auto first = [](int x) { return __builtin_amdgcn_readfirstlane(x); };   // the same in every lane
  uint32_t lo = 0, hi = 0xFFFFFFFFu;
  int r = c, m = N;
  if constexpr (SRC != KEYS_FROM_SCORES) {
    int h[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) h[e] = SRC == KEYS_READY ? pos[base + 4 * tid + e] : bins[4 * tid + e];
    locate(h, c);
    const int bin = first(sel[0]);
    lo = bin_start(bin);
    if (bin < kBins - 1) hi = bin_start(bin + 1) - 1;
    r = first(sel[1]);
    m = first(sel[2]);
  }
  if (__builtin_expect(m > kCandidates && lo != hi, 0)) {
    // Crowded or equal scores. From here on the keys are read from LDS, each thread
    // its own, in rolled loops: over the registers they cost the ordinary path 1 to
    // 2 us (masks and spills of KR rounds).
#pragma unroll
    for (int j = 0; j < KR; ++j) own_keys[j][tid] = key[j];
    // A pass leaves 2^20, then 2^8, then one of the 2^32 keys at most.
    for (int pass = 0; pass < 3 && m > kCandidates && lo != hi; ++pass) {
      if (pass > 0) {
        // still many: the range that they span (equal ones are found here)
        uint32_t least = 0xFFFFFFFFu, most = 0xFFFFFFFFu;   // most: of the complements
        for (int j = 0; j < R; ++j) {
          const uint32_t k = own_keys[j][tid];
          if ((i0 + 64 * j < N) & (k - lo <= hi - lo)) {
            least = min(least, k);
            most = min(most, ~k);
          }
        }
        least = wave_min(least);
        most = wave_min(most);
        if (lane == 0) {
          wave_range[0][wave] = least;
          wave_range[1][wave] = most;
        }
      }
      __syncthreads();
      for (int i = tid; i < kBins; i += kThreads) bins[i] = 0;
      if (pass > 0) {
        lo = (uint32_t)first((int)row_min(wave_range[0][lane & (kWaves - 1)]));
        hi = ~(uint32_t)first((int)row_min(wave_range[1][lane & (kWaves - 1)]));
        if (lo == hi) break;
      }
      __syncthreads();
      const int bits = 32 - __builtin_clz(hi - lo), shift = max(bits - 12, 0);
      for (int j = 0; j < R; ++j) {
        const uint32_t k = own_keys[j][tid];
        count_in(bins, (i0 + 64 * j < N) & (k - lo <= hi - lo), (int)((k - lo) >> shift) & (kBins - 1));
      }
      __syncthreads();
      int h[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) h[e] = bins[4 * tid + e];
      locate(h, r);
      lo += (uint32_t)first(sel[0]) << shift;
      hi = lo + min(hi - lo, (1u << shift) - 1);      // (the bin of the largest key may end past 2^32)
      r = first(sel[1]);
      m = first(sel[2]);
    }
  }
  uint32_t kstar = lo;
  if (lo != hi) {
#pragma unroll
    for (int j = 0; j < KR; ++j)
      if (holds(j) & (key[j] - lo <= hi - lo)) cand[atomicAdd(&n_cand, 1) & (kCandidates - 1)] = key[j];
    __syncthreads();
    if (tid < m) {
      const uint32_t k = cand[tid];
      int less = 0, same = 0;
      for (int i = 0; i < m; ++i) {
        less += cand[i] < k;
        same += cand[i] == k;
      }
      if (less < r && r <= less + same) {             // equal keys write the same values
        sel[0] = (int)k;
        sel[1] = r - less;
      }
    }
    __syncthreads();
    kstar = (uint32_t)first(sel[0]);
    r = first(sel[1]);
  }

  // Token-order ranks. Per wave the counts of smaller and of equal keys; the
  // waves before this one then give the equal keys and active tokens ahead of
  // its run, and within the run both follow from ballots round by round.
  int n_less = 0, n_eq = 0;
#pragma unroll
  for (int j = 0; j < KR; ++j) {
    n_less += __popcll(__ballot(holds(j) && key[j] < kstar));
    n_eq += __popcll(__ballot(holds(j) && key[j] == kstar));
  }
  if (lane == 0) {
    wave_cnt[0][wave] = n_less;
    wave_cnt[1][wave] = n_eq;
  }
  __syncthreads();
  const int less0 = waves_before(wave_cnt[0], wave);
  int eq0 = waves_before(wave_cnt[1], wave);
  int next = row0 + min(wave * 64 * R, N) - less0 - min(eq0, r);   // row of this wave's first active token
  const uint64_t below = (1ull << lane) - 1ull;
#pragma unroll
  for (int j = 0; j < KR; ++j) {
    const bool in = holds(j);
    bool cached = key[j] < kstar;
    const uint64_t eq = __ballot(in && key[j] == kstar);
    if (eq) {
      if ((eq >> lane) & 1ull) cached = eq0 + __popcll(eq & below) < r;
      eq0 += __popcll(eq);
    }
    const uint64_t am = __ballot(in && !cached);
    const int a = next + __popcll(am & below);
    next += __popcll(am);
    if (in) {
      pos[base + i0 + 64 * j] = cached ? -1 : a;
      if (!cached) idx_active[a] = i0 + 64 * j;
    }
  }
}

// Teacher-forced selection: pos of every token is -1 ...
__global__ __launch_bounds__(256) void k_pos_fill(int32_t* __restrict__ pos, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) pos[i] = -1;
}

// ... then every listed row r of sample b sets idx_active[r] = i and
// pos[b][i] = r, with i clamped into [0, N) so that no access leaves the
// arrays whatever the caller's buffer holds.
__global__ __launch_bounds__(256) void k_force_scatter(const int32_t* __restrict__ idx_in, Segs act, int N,
                                                       int32_t* __restrict__ idx_out, int32_t* __restrict__ pos) {
  const int r = blockIdx.x * 256 + threadIdx.x;
  if (r >= act.off[act.B]) return;
  const int b = find_segment(act.off, act.B, r);
  const int i = min(max(idx_in[r], 0), N - 1);
  idx_out[r] = i;
  pos[(size_t)b * N + i] = r;
}

}  // namespace

hipError_t launch_force_active(const int32_t* idx_in, const Segs& act, int N, int32_t* idx_out, int32_t* pos,
                               hipStream_t s) {
  const int64_t n = (int64_t)act.B * N;
  launch(k_pos_fill, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, pos, n);
  const int rows = act.off[act.B];
  if (rows > 0) launch(k_force_scatter, dim3((unsigned)((rows + 255) / 256)), dim3(256), 0, s, idx_in, act, N, idx_out, pos);
  return hipGetLastError();
}

// Static selection scratch for callers that cannot allocate (the no-alloc
// operator entry). Each device holds its own copy; its device address is
// looked up once per device and kept, since host code must never pass the
// symbol itself to a kernel.
constexpr size_t kStaticScratchBytes = (size_t(4) << 20) + (size_t(16) << 10);
static __device__ __align__(256) char scratch[kStaticScratchBytes];

hipError_t select_static_scratch(void** ptr, size_t* bytes) {
  static std::mutex mu;
  static std::vector<void*> by_device;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  std::lock_guard<std::mutex> lock(mu);
  if ((int)by_device.size() <= dev) by_device.resize(dev + 1, nullptr);
  if (!by_device[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    by_device[dev] = p;
  }
  *ptr = by_device[dev];
  *bytes = kStaticScratchBytes;
  return hipSuccess;
}

size_t select_workspace_bytes(int B, int N) {
  const int chunks = (N + kChunk - 1) / kChunk;
  return (((size_t)B * N * sizeof(float2) + 255) & ~(size_t)255) + (size_t)B * chunks * sizeof(float4);
}

hipError_t launch_select(const float* v_cache, const float* v_prev, int B, int N, float w_a, float w_v,
                         const Segs& n_cache, const Segs& act, int32_t* idx_active, int32_t* pos,
                         float* score, void* workspace, hipStream_t s) {
  const int chunks = (N + kChunk - 1) / kChunk;
  float2* va = static_cast<float2*>(workspace);
  float4* partial = reinterpret_cast<float4*>(static_cast<char*>(workspace) +
                                              (((size_t)B * N * sizeof(float2) + 255) & ~(size_t)255));
  const bool fused = N <= kFusedTokens;
  launch(k_score_stats, dim3(chunks, B), dim3(kStatThreads), 0, s, v_cache, v_prev, N, n_cache, va, partial, chunks,
         fused ? (int32_t*)nullptr : pos);
  if (!fused)
    launch(k_keys, dim3(chunks, B), dim3(kStatThreads), 0, s, va, (const float4*)partial, chunks, N, w_a, w_v, n_cache,
           pos, score);
  auto select = [&](auto kernel) {
    launch(kernel, dim3(B), dim3(kThreads), 0, s, (const float2*)va, (const float4*)partial, chunks, N, w_a, w_v,
           n_cache, act, idx_active, pos, score, (const float*)nullptr);
  };
  if (N <= kThreads) select(k_select<KEYS_FROM_STATS, 1>);
  else if (N <= 4 * kThreads) select(k_select<KEYS_FROM_STATS, 4>);
  else if (fused) select(k_select<KEYS_FROM_STATS, 8>);
  else if (N <= 16 * kThreads) select(k_select<KEYS_READY, 16>);
  else select(k_select<KEYS_READY, 32>);
  return hipGetLastError();
}

hipError_t launch_select_scores(const float* scores, int B, int N, const Segs& n_cache, const Segs& act,
                                int32_t* idx_active, int32_t* pos, hipStream_t s) {
  auto select = [&](auto kernel) {
    launch(kernel, dim3(B), dim3(kThreads), 0, s, (const float2*)nullptr, (const float4*)nullptr, 0, N, 0.0f, 0.0f,
           n_cache, act, idx_active, pos, (float*)nullptr, scores);
  };
  if (N <= kThreads) select(k_select<KEYS_FROM_SCORES, 1>);
  else if (N <= 4 * kThreads) select(k_select<KEYS_FROM_SCORES, 4>);
  else if (N <= 8 * kThreads) select(k_select<KEYS_FROM_SCORES, 8>);
  else if (N <= 16 * kThreads) select(k_select<KEYS_FROM_SCORES, 16>);
  else select(k_select<KEYS_FROM_SCORES, 32>);
  return hipGetLastError();
}

}  // namespace f3c
