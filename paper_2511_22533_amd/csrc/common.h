// Shared device-side definitions for the gfx950 kernels: element types, MFMA
// fragment traits for the 32x32 matrix-core family, and small helpers.
#pragma once

#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace f3c {

// Timing of one profiled library call. While it is set on this thread, every
// kernel launch goes through AMD's extended launch, which stamps the events
// with the kernels' own start and end: the first kernel of the call stamps
// start, each kernel re-stamps stop. The pair then spans the call's kernels
// without the host's dispatch gap in front of them.
struct LaunchTimer {
  hipEvent_t start = nullptr, stop = nullptr;
  bool used = false;
};

inline LaunchTimer& launch_timer() {
  static thread_local LaunchTimer t;
  return t;
}

// Kernel launch used by every kernel of the library (same arguments as
// hipLaunchKernelGGL).
template <typename F, typename... Args>
inline void launch(F kernel, dim3 grid, dim3 block, uint32_t shmem, hipStream_t s, Args... args) {
  LaunchTimer& t = launch_timer();
  if (!t.stop) {
    hipLaunchKernelGGL(kernel, grid, block, shmem, s, args...);
    return;
  }
  hipExtLaunchKernelGGL(kernel, grid, block, shmem, s, t.used ? nullptr : t.start, t.stop, 0u, args...);
  t.used = true;
}

typedef __bf16 bf16;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// 32x32 MFMA family. One instruction multiplies a 32xK by a Kx32 tile. Each
// lane l feeds E consecutive K-elements of row (A) / column (B) l % 32 for the
// K-group l / 32; the 16 accumulators of lane l hold column l % 32 and rows
// 8*(i/4) + 4*(l/32) + i%4, i = 0..15.
template <typename T> struct Mfma;

template <> struct Mfma<bf16> {
  static constexpr int E = 8;          // elements per lane per instruction (K = 16)
  typedef bf16x8 frag;
  static __device__ __forceinline__ f32x16 mma(const frag& a, const frag& b, const f32x16& c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
  }
};

template <> struct Mfma<float> {
  static constexpr int E = 1;          // K = 2
  typedef float frag;
  static __device__ __forceinline__ f32x16 mma(const frag& a, const frag& b, const f32x16& c) {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
  }
};

__device__ __forceinline__ float to_f32(float x) { return x; }
__device__ __forceinline__ float to_f32(bf16 x) { return static_cast<float>(x); }

template <typename T> __device__ __forceinline__ T from_f32(float x);
template <> __device__ __forceinline__ float from_f32<float>(float x) { return x; }
template <> __device__ __forceinline__ bf16 from_f32<bf16>(float x) { return static_cast<bf16>(x); }

// GELU in its tanh form, 0.5 x (1 + tanh(u)) with u = sqrt(2/pi) (x + 0.044715 x^3),
// evaluated as the identical x / (1 + e^(-2u)): one exponential and one
// reciprocal instead of the library tanhf (measured on MI355X: the MLP's first
// projection at 32768 rows, 485 -> 447 us; a plain store takes 440 us). For
// u far below zero e^(-2u) overflows to +inf and the result is -0.
__device__ __forceinline__ float gelu_tanh(float x) {
  const float k0 = 0.7978845608028654f;   // sqrt(2/pi)
  const float k1 = 0.044715f;
  const float u = k0 * (x + k1 * x * x * x);
  const float e = __builtin_amdgcn_exp2f(u * -2.8853900817779268f);   // 2^(-2u log2(e)) = e^(-2u)
  return x * __builtin_amdgcn_rcpf(1.0f + e);
}

__device__ __forceinline__ float silu(float x) { return x / (1.0f + expf(-x)); }

// The value of the lane that a DPP pattern within rows of 16 lanes names:
// kDppXor8 (rotate by 8), kDppMirror8 (lane ^ 7), kDppXor2, kDppXor1.
enum { kDppXor8 = 0x128, kDppMirror8 = 0x141, kDppXor2 = 0x4E, kDppXor1 = 0xB1 };
template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, false));
}

// Each lane's value added up over the four rows of 16 lanes (lanes l, l ^ 16,
// l ^ 32, l ^ 48), in all of them, with gfx950's half-row and half-wave swaps:
// two copies of v trade halves and are added. (Inline assembly: the builtin
// hands both results back in one register here. The nops cover a vector write
// read by the swap and the swap's result read by the add.)
__device__ __forceinline__ float rows_sum(float v) {
  float w = v;
  asm("s_nop 1\n\tv_permlane16_swap_b32 %0, %1\n\ts_nop 1" : "+v"(v), "+v"(w));
  v += w;
  w = v;
  asm("s_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\ts_nop 1" : "+v"(v), "+v"(w));
  return v + w;
}

// Sum over the wave, the same in every lane: six vector adds and two swaps
// (six __shfl_xor go through the LDS pipe at its latency each: with two of
// these per row, the output projection of 9831 rows of 1024 takes 3 us more).
__device__ __forceinline__ float wave_sum(float v) {
  v += dpp<kDppXor8>(v);
  v += dpp<kDppMirror8>(v);
  v += dpp<kDppXor2>(v);
  v += dpp<kDppXor1>(v);
  return rows_sum(v);
}

// Workgroups are dispatched round-robin over the 8 XCDs (each with its own
// L2). Map the hardware workgroup id to a logical id so that each XCD receives
// one contiguous range of logical ids (sizes differ by at most one).
__device__ __forceinline__ int xcd_logical_id(int hw, int total) {
  constexpr int kXcd = 8;
  const int x = hw % kXcd, i = hw / kXcd;
  const int q = total / kXcd, r = total % kXcd;
  return x * q + (x < r ? x : r) + i;
}

// 16 bytes per lane from global memory straight into LDS at lds_block + 16 *
// lane (gfx950 global_load_lds_dwordx4; the block base is wave-uniform and
// goes through M0). Written as inline assembly so that the compiler does not
// track it: it would otherwise wait for every outstanding LDS load of this
// kind before any LDS read. A kernel using it orders these loads itself (an
// s_waitcnt on the vector-memory counter and a barrier before a tile is
// read); waits the compiler places for its own loads only grow more
// conservative, since the counter retires in issue order.
__device__ __forceinline__ void dma16(const char* gptr, char* lds_block) {
  const uint32_t base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds_block;
  asm volatile("global_load_lds_dwordx4 %0, off" : : "v"(gptr), "{m0}"(__builtin_amdgcn_readfirstlane(base))
               : "memory");
}

// Wait until at most N vector-memory operations are outstanding (gfx9
// s_waitcnt encoding; expcnt and lgkmcnt left at their maxima).
template <int N>
__device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}

// Sample lookup in a segment table off[0..B] (off[B] = total rows).
__device__ __forceinline__ int find_segment(const int* off, int B, int row) {
  int b = 0;
  while (b + 1 < B && off[b + 1] <= row) ++b;
  return b;
}

// The same for a row that is uniform over the wave, all lanes active, B <= 64:
// many samples are looked at together (attention of 64 samples of 64 tokens, 16
// heads: 27 -> 18 us against the loop, whose scalar loads wait for each other).
__device__ __forceinline__ int find_segment_wave(const int* off, int B, int row) {
  if (B <= 4) return find_segment(off, B, row);
  const int b = (int)(threadIdx.x & 63) + 1;
  return __popcll(__ballot(off[b < B ? b : B] <= row && b < B));
}

}  // namespace f3c
