// Variable-length multi-head softmax attention on the 32x32 matrix cores, used
// for self-attention over the active tokens of each sample (Sec. 4.2: self
// attention runs on the active subset only) and for cross-attention from the
// active tokens to the image-condition tokens.
//
// Online softmax over key/value tiles of 64 staged in LDS. Each wavefront owns 32
// queries, or two blocks of 32, and computes S^T = K Q^T, so a lane holds one
// query's scores for 16 of every 32 keys of a block: the running max and sum are
// per-lane values combined with a single cross-half exchange (lane l with l ^ 32).
// The same accumulator layout feeds O^T = V^T P^T as the B operand without any
// data movement; the K-slot order of P (keys 8*(e/4) + 4*(l/32) + e%4) is matched
// when the V^T fragment is read: from row-major tiles by the LDS transpose read
// (bf16 with 64-wide heads), else from tiles stored transposed.
//
// Pipelining, bf16 with 64-wide heads (the transformer's case): K and V tiles
// go from global memory straight into five LDS buffers (four with key groups)
// with 16-byte DMA loads issued three tiles ahead (two with key groups). The
// step is cut into half tiles of 32 keys: while the vector unit takes the
// probabilities of one half, the matrix cores take the scores of the next and
// the PV product of the one before, interleaved instruction by instruction.
//
// What bounds it: at 32768 tokens the chip's power. With random operands the
// clock drops to 1.7-1.9 GHz under this kernel (2.4 GHz on zeros, with the same
// cycles), so work taken out counts for more than stalls taken out. Per 64
// keys and 256 queries of a CU: 1857 -> 1453 cycles against 1224 that the MFMAs
// alone take, from (a) the interleaving, (b) row sums on one small MFMA per
// eight probabilities instead of four v_dot2 (each of which holds the matrix
// pipe 16 cycles), (c) no wait on a tile's own sums, (d) 64 queries per wave,
// which halves the LDS fragment reads and, with 512 queries per workgroup, the
// DMA. 32768 tokens, 16 heads: 3797 -> 3388 us; 9831 tokens 414 -> 361 us.
//
// Other types and head sizes fetch the next tile into registers while the
// current one is consumed and write it to the other of two LDS buffers; the
// running max is updated lazily: the accumulators are rescaled only when some
// query's max grows by more than 2^8 (in base-2 units), which keeps every
// unnormalised probability below 2^8 and the result unchanged up to rounding.
// One barrier per tile either way. Only the last, ragged tile is masked.
//
// Few query tiles (late cached steps: a few hundred active tokens) cannot fill
// 256 CUs, so the key range may be split: each split writes its unnormalised
// output with its reference max and sum in f32, and a second kernel merges the
// splits in split order (the standard log-sum-exp combination; deterministic).
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace f3c {

namespace {

constexpr int kBKV = 64;             // keys per LDS tile

// f(std::integral_constant<int, I>) for I = 0 .. N - 1, unrolled.
template <typename F, int... I>
__device__ __forceinline__ void static_for_seq(F f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F f) {
  static_for_seq(f, std::make_integer_sequence<int, N>{});
}

// max(a, b, c) as one v_max3_f32. fmaxf on MFMA results costs three
// instructions each (both inputs are first quieted with v_max x, x, since the
// compiler cannot prove they are not signalling NaNs). A NaN score is passed over
// unless all three are; its query's probabilities and sum are NaN all the same,
// and a pass tests for sums that are not below its limit.
__device__ __forceinline__ float max3(float a, float b, float c) {
  float r;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}

// Max of the 16 accumulators of one 32 x 32 score tile: eight dependent
// v_max3_f32 in one block (one hazard boundary for the compiler instead of
// one per instruction; dependent VALU instructions need no wait states).
__device__ __forceinline__ float max16(const f32x16& v) {
  float r;
  asm("v_max3_f32 %0, %1, %2, %3\n\t"
      "v_max3_f32 %0, %0, %4, %5\n\t"
      "v_max3_f32 %0, %0, %6, %7\n\t"
      "v_max3_f32 %0, %0, %8, %9\n\t"
      "v_max3_f32 %0, %0, %10, %11\n\t"
      "v_max3_f32 %0, %0, %12, %13\n\t"
      "v_max3_f32 %0, %0, %14, %15\n\t"
      "v_max_f32 %0, %0, %16"
      : "=&v"(r)
      : "v"(v[0]), "v"(v[1]), "v"(v[2]), "v"(v[3]), "v"(v[4]), "v"(v[5]), "v"(v[6]), "v"(v[7]), "v"(v[8]),
        "v"(v[9]), "v"(v[10]), "v"(v[11]), "v"(v[12]), "v"(v[13]), "v"(v[14]), "v"(v[15]));
  return r;
}

typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) i16x4 lds_i16x4;
constexpr float kRescaleLog2 = 8.0f;
// DMA path: probabilities are taken against a reference max that moves only
// when a query's row sum passes kTileSumLimit times the number of key tiles; it
// then moves to leave the sum near 2^-kHeadroomLog2, since a move costs all of a
// wave's queries (1639 x 1639 keys with norms growing 30-fold, us: 25.4; moved to
// leave a sum near 1 30.2; with a limit of 2^16 31.5). Probabilities (bf16, the
// exponent range of f32) and sums stay finite, and their relative rounding does
// not depend on the reference. An unnormalised output is at most the row sum
// times the largest value: values of 2^100 cannot overflow it in 512 tiles (32768
// keys), and those of 2^-100 lose nothing that counts.
constexpr float kTileSumLimit = 0x1p17f, kHeadroomLog2 = 16.0f;
// Raw passes (see there): the first tile's max (base 2) that they take, and the
// row sum below which their outputs must be larger than kRawOutMin.
constexpr float kRawMin = -40.0f, kRawMax = 64.0f, kRawSumMin = 1.0f, kRawOutMin = 0x1p-100f;

struct AttnArgs {
  Segs qs, ks;
  int tile_off[kMaxBatch + 1];   // prefix of query tiles per sample
  const char* q;
  const char* k;
  const char* v;
  char* o;
  int ldq, ldk, ldv, ldo;        // elements
  int heads;
  float scale_log2;              // log2(e) / sqrt(hd), or 1 when the queries were stored scaled by it
  int splits;                    // key-range splits (1: normalised output straight to o)
  int rows;                      // query rows qs.off[B] - qs.off[0] (split partials)
  float* part_o;                 // [splits][rows][heads][hd] unnormalised outputs
  float* part_ml;                // [splits][rows][heads][2] (max * scale_log2, sum)
};

// KS key groups (matrix-core path only): the NW waves are NW/KS query waves
// times KS groups; group k takes key tiles t_begin + KS*i + k in lockstep
// with the others (one LDS stage holds the KS tiles of a step), and the
// groups' (max, sum, output) are merged through LDS at the end. Two groups
// double the waves per query tile where query tiles are too few to fill the
// chip.
// QB: blocks of 32 queries per wave.
// QS: the queries were stored multiplied by log2(e)/sqrt(hd) (scores come out
// in base-2 units).
template <typename T, int HD, int NW, int SITE, bool SPLIT, int KS = 1, bool QS = false, int QB = 1>
__global__ __launch_bounds__(64 * NW, QB) void k_attn(AttnArgs p) {
  constexpr int NT = 64 * NW;
  constexpr int QW = NW / KS;                // query waves
  constexpr int BQ = 32 * QB * QW;
  constexpr int ES = sizeof(T);
  constexpr int E = Mfma<T>::E;
  // bf16 with 64-wide heads: K and V tiles go global -> LDS directly (16-byte
  // DMA loads, no registers) into five buffers (four with key groups), row-major
  // with 128-byte rows
  // whose 16-byte chunks are XOR-swizzled by row (conflict-free fragment
  // reads); V^T fragments come from the row-major V tile through the LDS
  // transpose read. Other types and head sizes stage through registers, with
  // V transposed on its way into LDS.
  constexpr bool DMA = ES == 2 && HD == 64;
  static_assert(QB == 1 || (DMA && KS == 1 && !SPLIT), "query blocks need the matrix-core path");
  static_assert(KS == 1 || (KS == 2 && DMA && NW % 2 == 0 && !SPLIT),
                "key groups need the matrix-core path and the whole key range");
  constexpr int NBUF = DMA ? (KS == 1 ? 5 : 4) : 2;
  constexpr int KRS = DMA ? HD * ES : HD * ES + 16;   // K tile row stride (bytes)
  constexpr int VRS = kBKV * ES + 8;                 // V^T tile row stride (bytes), register path
  constexpr int NKS = HD * ES / 32;          // 32-byte K slices over the head dim
  constexpr int PER16 = 16 / ES;
  constexpr int MMA_PER_READ = PER16 / E;
  constexpr int HT = HD / 32;                // 32-row output tiles over the head dim
  constexpr int CPR = HD * ES / 16;          // 16-byte chunks per key row
  constexpr int KITEMS = kBKV * CPR;        // K chunks per tile
  constexpr int VITEMS = kBKV / 2 * CPR;    // V (key pair, chunk) items per tile
  constexpr int KCH = (KITEMS + NT - 1) / NT;
  constexpr int VPR = (VITEMS + NT - 1) / NT;
  constexpr int KBUF = kBKV * KRS, VBUF = DMA ? kBKV * HD * ES : HD * VRS;
  constexpr int TB = KBUF + VBUF, SB = KS * TB;      // bytes per tile, per stage
  // DMA path: the K tiles of all stages, then the V tiles (VREG on), so that a
  // fragment read's stage offset fits the 16-bit offset field of the LDS read.
  constexpr int VREG = NBUF * KS * KBUF;
  __shared__ __attribute__((aligned(16))) char lds[NBUF * SB];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int kgrp = wave / QW, qw = wave - kgrp * QW;
  const int g = lane >> 5, r32 = lane & 31;
  // 1-D grid over (head, query tile, split); all work of a head shares one XCD's L2.
  const int ntq = p.tile_off[p.qs.B];
  const int nsp = SPLIT ? p.splits : 1;
  const int logical = xcd_logical_id(blockIdx.x, ntq * p.heads * nsp);
  const int head = logical / (ntq * nsp);
  const int rem = logical - head * ntq * nsp;
  const int tq = rem / nsp, sp = rem - tq * nsp;
  const int b = find_segment_wave(p.tile_off, p.qs.B, tq);
  const int qt = tq - p.tile_off[b];
  const int q_begin = p.qs.off[b], nq = p.qs.off[b + 1] - q_begin;
  const int k_begin = p.ks.off[b], nk = p.ks.off[b + 1] - k_begin;
  const int qi = qt * BQ + qw * 32 * QB + r32;         // this lane's query (within the sample) in the wave's first block

  // Q^T as the B operand: lane reads 16 bytes of its query row per 32-byte slice.
  u32x4 qf[QB][NKS];
#pragma unroll
  for (int j = 0; j < QB; ++j) {
    const int i = qi + 32 * j;
    const char* qrow = p.q + ((size_t)(q_begin + (i < nq ? i : 0)) * p.ldq + head * HD) * ES;
#pragma unroll
    for (int s = 0; s < NKS; ++s)
      qf[j][s] = i < nq ? *reinterpret_cast<const u32x4*>(qrow + s * 32 + g * 16) : u32x4{0, 0, 0, 0};
  }

  // Tile staging: K row-major, V transposed (pairs of keys per 32/64-bit write).
  // Keys past the end are read from the last key (always valid) and masked.
  // Two register sets: tile t+2 is fetched while tile t+1 waits to be staged.
  // Every thread issues the same loads (threads past the item count re-read
  // the last item and skip the LDS write): a branch around some of the loads
  // would make the compiler's wait before staging cover the loads in flight.
  u32x4 rk[2][KCH], rv[2][VPR][2];
  auto fetch = [&](int kv0, int r) {
#pragma unroll
    for (int q = 0; q < KCH; ++q) {
      const int ch = min(tid + NT * q, KITEMS - 1), row = ch / CPR, col = ch % CPR;
      const int key = min(kv0 + row, nk - 1);
      rk[r][q] = *reinterpret_cast<const u32x4*>(p.k + ((size_t)(k_begin + key) * p.ldk + head * HD) * ES + col * 16);
    }
#pragma unroll
    for (int q = 0; q < VPR; ++q) {
      const int it = min(tid + NT * q, VITEMS - 1), pr = it / CPR, col = it % CPR;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int key = min(kv0 + 2 * pr + h, nk - 1);
        rv[r][q][h] = *reinterpret_cast<const u32x4*>(p.v + ((size_t)(k_begin + key) * p.ldv + head * HD) * ES + col * 16);
      }
    }
  };
  auto stage = [&](int buf, int r) {
    char* Ks = lds + buf * (KBUF + VBUF);
    char* Vt = Ks + KBUF;
#pragma unroll
    for (int q = 0; q < KCH; ++q) {
      const int ch = tid + NT * q, row = ch / CPR, col = ch % CPR;
      if (KITEMS % NT != 0 && ch >= KITEMS) break;
      *reinterpret_cast<u32x4*>(Ks + row * KRS + col * 16) = rk[r][q];
    }
#pragma unroll
    for (int q = 0; q < VPR; ++q) {
      const int it = tid + NT * q, pr = it / CPR, col = it % CPR;
      if (VITEMS % NT != 0 && it >= VITEMS) break;
      const T* v0 = reinterpret_cast<const T*>(&rv[r][q][0]);
      const T* v1 = reinterpret_cast<const T*>(&rv[r][q][1]);
#pragma unroll
      for (int e = 0; e < PER16; ++e) {
        char* dst = Vt + (col * PER16 + e) * VRS + 2 * pr * ES;
        if constexpr (ES == 2) {
          const uint32_t lo = __builtin_bit_cast(uint16_t, v0[e]), hi = __builtin_bit_cast(uint16_t, v1[e]);
          *reinterpret_cast<uint32_t*>(dst) = lo | (hi << 16);
        } else {
          *reinterpret_cast<float2*>(dst) = make_float2(v0[e], v1[e]);
        }
      }
    }
  };

  // DMA path: one wave instruction fills 1 KiB = 8 rows; lane l writes 16-byte
  // slot l, i.e. row l/8 and physical chunk l%8, with the logical chunk the
  // row's swizzle maps there (XOR is its own inverse).
  //   K: physical chunk = chunk ^ ((row >> 1) & 7)  (16 lanes read 16 rows)
  //   V: physical chunk = chunk ^ (((row >> 1) & 1) << 2)  (transpose reads
  //      take 32 bytes from each of 4 consecutive rows)
  constexpr int DBLK = kBKV / 8;                       // 8-row blocks per tile
  constexpr int DQ = (DBLK + NW - 1) / NW;             // blocks per wave
  // DMA addresses: a buffer descriptor per operand over this sample's rows of
  // this head, and 32-bit lane offsets, the same for every tile but for the
  // tile's first row (the host checks that nk rows of either operand stay
  // below 2 GiB). Rows past the last lie outside the descriptor and read as
  // zero, so no lane clamps its row: two vector instructions per tile and 1 KiB
  // block pair, and two registers.
  const uint32_t ldk_b = (uint32_t)p.ldk * ES, ldv_b = (uint32_t)p.ldv * ES;
  const uint32_t lds_u = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds;
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);
  auto descriptor = [&](const char* base, uint32_t ld_b) {
    const uint64_t a = (uint64_t)base;
    const uint32_t bytes = nk > 0 ? (uint32_t)(nk - 1) * ld_b + HD * ES : 0u;
    return u32x4{(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)a),
                 (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(a >> 32) & 0xffffu),
                 (uint32_t)__builtin_amdgcn_readfirstlane(bytes), 0x00020000u};
  };
  const u32x4 kdesc = descriptor(p.k + ((size_t)k_begin * p.ldk + head * HD) * ES, ldk_b);
  const u32x4 vdesc = descriptor(p.v + ((size_t)k_begin * p.ldv + head * HD) * ES, ldv_b);
  uint32_t kofs[DQ], vofs[DQ];
#pragma unroll
  for (int q = 0; q < DQ; ++q) {
    const int row = min(wave_u + NW * q, DBLK - 1) * 8 + (lane >> 3), phys = lane & 7;
    kofs[q] = row * ldk_b + (uint32_t)((phys ^ ((row >> 1) & 7)) << 4);
    vofs[q] = row * ldv_b + (uint32_t)((phys ^ (((row >> 1) & 1) << 2)) << 4);
    asm("" : "+v"(kofs[q]), "+v"(vofs[q]));            // kept, not recomputed per tile
  }
  auto fetch_dma = [&](int kv0, int stage, int k) {
#pragma unroll
    for (int q = 0; q < DQ; ++q) {
      const int blk_u = min(wave_u + NW * q, DBLK - 1);
      const uint32_t ko = kofs[q] + (uint32_t)kv0 * ldk_b, vo = vofs[q] + (uint32_t)kv0 * ldv_b;
      const uint32_t kl = lds_u + (uint32_t)((stage * KS + k) * KBUF + blk_u * 1024);
      const uint32_t vl = lds_u + (uint32_t)(VREG + (stage * KS + k) * VBUF + blk_u * 1024);
      asm volatile("buffer_load_dwordx4 %0, %1, 0 offen lds" : : "v"(ko), "s"(kdesc), "{m0}"(kl) : "memory");
      asm volatile("buffer_load_dwordx4 %0, %1, 0 offen lds" : : "v"(vo), "s"(vdesc), "{m0}"(vl) : "memory");
    }
  };

  f32x16 oacc[QB][HT];
  float m_run[QB], l_run[QB];          // running max (raw logits), unnormalised sum
#pragma unroll
  for (int j = 0; j < QB; ++j) {
#pragma unroll
    for (int t = 0; t < HT; ++t)
#pragma unroll
      for (int e = 0; e < 16; ++e) oacc[j][t][e] = 0.0f;
    m_run[j] = -INFINITY;
    l_run[j] = 0.0f;
  }
  const float c = p.scale_log2;
  // Key tiles [t_begin, t_end) of this split (balanced; empty when the sample
  // has fewer tiles than splits).
  const int ntiles = (nk + kBKV - 1) / kBKV;
  const int t_begin = sp * ntiles / nsp, t_end = (sp + 1) * ntiles / nsp;
  const int last_kv = (t_end - 1) * kBKV;

  // Per-lane constants of the DMA path's fragment reads: the K swizzle of rows
  // 32*kt + r32, and for the transpose read the source row and column within
  // the lane's 16-lane group (rows kb + vi/4, columns db + 4*(vi%4)).
  const int kswz = (r32 >> 1) & 7;
  const int vi = lane & 15;
  const int vrow = vi >> 2, vswz = ((vi >> 3) & 1) << 2, vcol = 4 * (vi & 3) + 16 * ((lane >> 4) & 1);

  if constexpr (DMA) {
    // Software pipeline over half steps of 32 keys. Half step (i, h) takes the
    // probabilities of half h of tile i on the vector unit while the matrix
    // cores take the scores of the next 32 keys and the PV product of the
    // 32 keys before: three independent pieces of work, written as 8 * QB groups of
    // one MFMA and its share of the vector work, and a scheduling barrier
    // after each group keeps them so. (Left to the compiler, the score
    // product's MFMAs stood alone and the vector work gathered behind them:
    // both waves of a SIMD then want the same unit at the same time.)
    // Fragments are read from LDS LA groups before their MFMAs.
    auto fence = [] { __builtin_amdgcn_sched_barrier(0); };
    // Row sums of the probabilities as rounded for the PV product: one 16x16x32
    // MFMA per fragment with a selector as its A operand. The fragment's lane
    // l holds query l % 32, which that instruction takes for column l % 16 of
    // K-group l / 16; row m selects the K-groups with the parity of m / 4, so
    // that every element of lane l's result is the sum of query l % 32 over
    // both key halves. (A v_dot2 per pair holds the matrix pipe 16 cycles, as
    // long as this MFMA does for eight values.)
    u32x4 sel;
    {
      const uint32_t w = ((lane >> 4) & 1) == ((lane >> 2) & 1) ? 0x3f803f80u : 0u;   // two ones
      sel = u32x4{w, w, w, w};
    }
    auto row_sum = [&](const bf16x8& f, const f32x4& acc) {
      return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, sel), f, acc, 0, 0, 0);
    };
    typedef __attribute__((address_space(3))) const u32x4 lds_u32x4;
    auto mma_k = [&](const u32x4& kf, const u32x4& q, const f32x16& acc) {
      return Mfma<T>::mma(__builtin_bit_cast(bf16x8, kf), __builtin_bit_cast(bf16x8, q), acc);
    };
    // Keys of element e of half kt: kv0 + 8*(e/4) + 4*g + e%4; mask those past nk.
    auto mask = [&](int t, int kt, f32x16& s) {
      const int kv0 = t * kBKV + kt * 32;
      if (kv0 + 32 > nk) {
#pragma unroll
        for (int e = 0; e < 16; ++e)
          if (kv0 + 8 * (e >> 2) + 4 * g + (e & 3) >= nk) s[e] = -INFINITY;
      }
    };
    // The shift by the reference max. Safe passes (one query block per wave): a
    // score accumulation starts from -(reference max) (minit), so a probability
    // is one exponential (after a multiply unless the queries were stored
    // scaled), and the reference moves where a sum outgrows it. Raw passes (two
    // blocks, which leave no registers for that): a probability is 2^(s c)
    // outright. That is the same result up to rounding while sums and outputs
    // neither overflow nor, where the sums are small, come near underflow. A
    // workgroup where one does takes its queries again in safe passes, one block
    // after the other. As a rule that is known after the first tile, by its max
    // (9831 x 9831, 16 heads: 437 us against 359 in raw passes; waves of 32 queries
    // with four v_dot2 per row sum, in a launch of their own, 417). Scores of about
    // 110 and more (base 2) after a first tile without are known at the end only
    // (key norms growing 30-fold: 857 us; 661 in such waves of 32).
    const float limit = kTileSumLimit * (float)(t_end - t_begin);
    auto prob = [&](float s) { return __builtin_amdgcn_exp2f(QS ? s : s * c); };
    // Steps i = 0, 1, ...: this wave's tile is t_begin + KS*i + kgrp; stage i
    // % NBUF holds the KS tiles of step i. Step i's barrier makes tile i + 1
    // readable and retires the stage of step i - 2, whose V fragments were
    // last read in half step (i - 1, 0); it receives step i + DIST (past the
    // end the last tile is read again, so that the wait counts stay fixed).
    constexpr int DIST = NBUF - 2;
    constexpr int DS = KS * 2 * DQ;                     // DMA instructions per step and wave
    constexpr int SK = KS * KBUF;
    static_assert(KBUF == VBUF, "one stage stride for keys and values");
    const int n_steps = (t_end - t_begin + KS - 1) / KS;
    auto tile_of = [&](int i) { return t_begin + KS * i + kgrp; };
    auto fetch_step = [&](int i, int stage) {
#pragma unroll
      for (int k = 0; k < KS; ++k) fetch_dma(min((t_begin + KS * i + k) * kBKV, last_kv), stage, k);
    };
    // Every query of block j in `qf`, its output (unnormalised), reference max
    // and row sum. False: a raw pass left its range (the same for the workgroup).
    auto pass = [&](auto pbc, const u32x4 (&qf)[decltype(pbc)::value][NKS], f32x16 (&oacc)[decltype(pbc)::value][HT],
                    float (&m_run)[decltype(pbc)::value], float (&l_run)[decltype(pbc)::value]) {
      constexpr int PB = decltype(pbc)::value;
      constexpr bool RAW = PB > 1;
      constexpr int LA = 4 / PB;
      // Lane addresses of the fragment reads in the current K and V stages (the
      // V^T fragment of keys kb..kb+3 and kb+8..kb+11 at column 32 h + lane % 32
      // comes from two transpose reads of the row-major tile, the K-slot order
      // of P); they move from stage to stage.
      uint32_t kad[NKS], vad[HT];
#pragma unroll
      for (int q = 0; q < NKS; ++q) {
        kad[q] = lds_u + (uint32_t)(kgrp * KBUF + r32 * KRS + (((2 * q + g) ^ kswz) << 4));
        asm("" : "+v"(kad[q]));
      }
#pragma unroll
      for (int h = 0; h < HT; ++h) {
        const int col = h * 32 + vcol;
        vad[h] = lds_u + (uint32_t)(VREG + kgrp * VBUF + (4 * g + vrow) * (HD * ES) + (((col >> 3) ^ vswz) << 4) +
                                    (col & 7) * ES);
        asm("" : "+v"(vad[h]));
      }
      auto rd_k = [&](int kt, int q) {             // keys 32 kt.., head columns 16 q..
        return *(lds_u32x4*)(uintptr_t)(kad[q] + (uint32_t)(kt * 32 * KRS));
      };
      auto rd_v = [&](int kt, int m) {             // keys 32 kt + 16 (m >> 1).., output columns 32 (m & 1)..
        const uint32_t a = vad[m & 1] + (uint32_t)((kt * 32 + 16 * (m >> 1)) * (HD * ES));
        const auto lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(uintptr_t)a);
        const auto hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(uintptr_t)(a + 8 * HD * ES));
        return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
      };
      f32x16 minit[PB];
      f32x4 ls[PB];                                // row sums (every element the same)
      float l_prev[PB];                            // the same without the newest probabilities
      auto probs = [&](const f32x16 (&s)[PB], bf16x8 (&pr)[PB][2]) {
#pragma unroll
        for (int j = 0; j < PB; ++j)
#pragma unroll
          for (int u = 0; u < 2; ++u) {
#pragma unroll
            for (int e = 0; e < 8; ++e) pr[j][u][e] = (bf16)prob(s[j][8 * u + e]);
            ls[j] = row_sum(pr[j][u], ls[j]);
          }
      };
      // Before the newest probabilities pr (of scores s) enter the PV product.
      // Rare: some query's row sum has outgrown its reference; move the reference
      // above the largest of these scores and the sum so far, rescale what was
      // accumulated and the scores taken since (next), and take pr again.
      auto fixup = [&](f32x16 (&s)[PB], f32x16 (&next)[PB], bf16x8 (&pr)[PB][2]) {
        if constexpr (RAW) return;
        // (a NaN sum too: an infinity or NaN among one query's probabilities
        // reaches the row sum of the query 16 lanes away, as 0 * inf)
        if (__builtin_amdgcn_ballot_w64(!(ls[0][0] <= limit)) != 0) {
#pragma unroll
          for (int j = 0; j < PB; ++j) {
            const float mx = max16(s[j]);
            float tm = __builtin_amdgcn_logf(l_prev[j]) + kHeadroomLog2;   // log2
            float tx = fmaxf(mx, __shfl_xor(mx, 32));
            if constexpr (!QS) tm /= c;
            tx += QS ? kHeadroomLog2 : kHeadroomLog2 / c;
            tm = fmaxf(0.0f, fmaxf(tm, tx));
            const float alpha = __builtin_amdgcn_exp2f(QS ? -tm : -tm * c);
            m_run[j] += tm;
#pragma unroll
            for (int u = 0; u < HT; ++u)
#pragma unroll
              for (int e = 0; e < 16; ++e) oacc[j][u][e] *= alpha;
#pragma unroll
            for (int e = 0; e < 16; ++e) {
              minit[j][e] -= tm;
              s[j][e] -= tm;
              next[j][e] -= tm;
            }
            // each query's sum from its own lanes alone
            float lt = 0.0f;
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
              for (int e = 0; e < 8; ++e) {
                pr[j][u][e] = (bf16)prob(s[j][8 * u + e]);
                lt += (float)pr[j][u][e];
              }
            lt = l_prev[j] * alpha + (lt + __shfl_xor(lt, 32));
            ls[j] = f32x4{lt, lt, lt, lt};
            // one opaque tuple: seen as a splat, it makes the loop carry copies
            asm("" : "+v"(ls[j]));
          }
        }
#pragma unroll
        for (int j = 0; j < PB; ++j) l_prev[j] = ls[j][0];
      };
      int k_stage = 0, v_stage = 0, d_stage = DIST;       // stages of kad, of vad and of the next fetch
      auto step_of = [](int& stage) {
        const uint32_t d = stage == NBUF - 1 ? (uint32_t)(-(NBUF - 1) * SK) : (uint32_t)SK;
        stage = stage == NBUF - 1 ? 0 : stage + 1;
        return d;
      };
      auto advance_k = [&] {
        const uint32_t d = step_of(k_stage);
#pragma unroll
        for (int q = 0; q < NKS; ++q) kad[q] += d;
      };
      auto advance_v = [&] {
        const uint32_t d = step_of(v_stage);
#pragma unroll
        for (int h = 0; h < HT; ++h) vad[h] += d;
      };
      auto sync = [&](int i) {
        wait_vm<(DIST - 2) * DS>();
        __builtin_amdgcn_s_barrier();
        fence();
        fetch_step(i + DIST, d_stage);
        d_stage = d_stage == NBUF - 1 ? 0 : d_stage + 1;
      };
      const f32x16 zero = {};
      u32x4 kf[NKS];
      bf16x8 vf[4];
      f32x16 s0[PB], s1[PB];                       // scores of a tile's first and second 32 keys
      bf16x8 p0[PB][2], p1[PB][2];                 // and their probabilities
      // Half step (i, KT): scores next = S(i, 1) or S(i + 1, 0), PV of pprev =
      // P(i - 1, 1) or P(i, 0), probabilities cur -> pcur of half KT of tile i.
      // Group n: score MFMA (even) or PV MFMA (odd), fragment n / PB >> 1 for
      // query block n % PB.
      auto half = [&](auto ktc, const f32x16 (&cur)[PB], f32x16 (&next)[PB], const bf16x8 (&pprev)[PB][2],
                         bf16x8 (&pcur)[PB][2]) {
        constexpr int KT = decltype(ktc)::value;
        float ex[16 * PB];
        static_for<8 * PB>([&](auto nc) {
          constexpr int n = decltype(nc)::value, grp = n / PB, j = n % PB, m = grp >> 1;
          if constexpr (j == 0) {
            if constexpr (KT == 0 && grp == 8 - LA) {
              advance_k();
              advance_v();
            }
            constexpr int ahead = (grp + LA) % 8, m2 = ahead >> 1, kt = grp + LA < 8 ? KT ^ 1 : KT;
            if constexpr (ahead % 2 == 0) kf[m2] = rd_k(kt, m2);
            else vf[m2] = rd_v(kt, m2);
          }
          if constexpr (grp % 2 == 0) next[j] = mma_k(kf[m], qf[j][m], m == 0 ? (RAW ? zero : minit[j]) : next[j]);
          else oacc[j][m & 1] = Mfma<T>::mma(vf[m], pprev[j][m >> 1], oacc[j][m & 1]);
          // Exponentials, their conversion one group later, the sum of a
          // fragment one group after its last conversion; the last sum lies
          // groups before the next half step's check of it.
          constexpr int N = 16 * PB;
          constexpr int E0 = n == 0 ? 0 : std::min(N, 3 * n + 1), E1 = std::min(N, 3 * n + 4);
          constexpr int C0 = n < 2 ? 0 : std::min(N, 3 * n - 2) & ~1, C1 = n == 0 ? 0 : std::min(N, 3 * n + 1) & ~1;
          constexpr int R0 = n < 2 ? 0 : n < 3 ? 0 : (std::min(N, 3 * n - 5) & ~1) / 8, R1 = C0 / 8;
          static_for<E1 - E0>([&](auto k) {
            constexpr int e = E0 + decltype(k)::value;
            ex[e] = prob(cur[e >> 4][e & 15]);
          });
          static_for<C1 - C0>([&](auto k) {
            constexpr int e = C0 + decltype(k)::value;
            pcur[e >> 4][(e >> 3) & 1][e & 7] = (bf16)ex[e];
          });
          static_for<R1 - R0>([&](auto k) {
            constexpr int u = R0 + decltype(k)::value;
            ls[u >> 1] = row_sum(pcur[u >> 1][u & 1], ls[u >> 1]);
          });
          fence();
        });
      };
      const std::integral_constant<int, 0> h0{};
      const std::integral_constant<int, 1> h1{};
      if (t_begin < t_end) {               // uniform over the workgroup
        // Q first: otherwise the compiler, which does not see the DMA, keeps its
        // wait for the Q fragments inside the loop as a full vmcnt(0).
        fence();
        wait_vm<0>();
#pragma unroll
        for (int i = 0; i < DIST; ++i) fetch_step(i, i);
        wait_vm<(DIST - 1) * DS>();
        // the last stage is not fetched before step 1's barrier
        volatile int* flag = reinterpret_cast<volatile int*>(lds + (NBUF - 1) * SK);
        if (RAW && tid == 0) *flag = 0;
        __syncthreads();
        // Tile 0's scores; the reference max is that tile's.
#pragma unroll
        for (int q = 0; q < NKS; ++q) {
          const u32x4 k0 = rd_k(0, q), k1 = rd_k(1, q);
#pragma unroll
          for (int j = 0; j < PB; ++j) {
            s0[j] = mma_k(k0, qf[j][q], q == 0 ? zero : s0[j]);
            s1[j] = mma_k(k1, qf[j][q], q == 0 ? zero : s1[j]);
          }
        }
#pragma unroll
        for (int j = 0; j < PB; ++j) {
          if (n_steps == 1) {
            mask(tile_of(0), 0, s0[j]);
            mask(tile_of(0), 1, s1[j]);
          }
          const float m0 = max16(s0[j]), m1 = max16(s1[j]);
          const float mx = max3(m0, m1, m1);
          m_run[j] = fmaxf(mx, __shfl_xor(mx, 32));
          if constexpr (!RAW) {
            const float sub = m_run[j] == -INFINITY ? 0.0f : m_run[j];   // a key group's tile may lie past the end
#pragma unroll
            for (int e = 0; e < 16; ++e) {
              minit[j][e] = -sub;
              s0[j][e] -= sub;
              s1[j][e] -= sub;
            }
          }
          ls[j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
          l_prev[j] = 0.0f;
        }
        if constexpr (RAW) {
          bool out = false;                // (a NaN is out)
#pragma unroll
          for (int j = 0; j < PB; ++j) out = out || !(m_run[j] * c >= kRawMin && m_run[j] * c <= kRawMax);
          if (__builtin_amdgcn_ballot_w64(out) != 0) *flag = 1;
        }
        if (n_steps > 1) {
          // (0, 0): S(0, 1) is there and no PV is due
          if constexpr (RAW) __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0): the flag
          sync(0);
          if constexpr (RAW) {
            if (__builtin_amdgcn_readfirstlane(*flag) != 0) {
              wait_vm<0>();
              __syncthreads();
              return false;
            }
          }
          probs(s0, p0);
          advance_k();
#pragma unroll
          for (int m = 0; m < LA / 2; ++m) {
            kf[m] = rd_k(0, m);
            vf[m] = rd_v(0, m);
          }
          fence();
          fixup(s0, s1, p0);
          half(h1, s1, s0, p0, p1);
          for (int i = 1; i < n_steps - 1; ++i) {
            sync(i);
            fixup(s1, s0, p1);
            half(h0, s0, s1, p1, p0);
            fixup(s0, s1, p0);
            half(h1, s1, s0, p0, p1);
          }
          // PV of the last P(i, 1), and the last tile's second scores
          fixup(s1, s0, p1);
#pragma unroll
          for (int m = 0; m < 4; ++m) {
            if (m >= LA / 2) {
              vf[m] = rd_v(1, m);
              kf[m] = rd_k(1, m);
            }
#pragma unroll
            for (int j = 0; j < PB; ++j) {
              oacc[j][m & 1] = Mfma<T>::mma(vf[m], p1[j][m >> 1], oacc[j][m & 1]);
              s1[j] = mma_k(kf[m], qf[j][m], m == 0 ? (RAW ? zero : minit[j]) : s1[j]);
            }
          }
          advance_v();
        }
        // Last tile (maybe ragged or past the end).
        const int t = tile_of(n_steps - 1);
#pragma unroll
        for (int j = 0; j < PB; ++j) {
          mask(t, 0, s0[j]);
          mask(t, 1, s1[j]);
        }
        probs(s0, p0);
        fixup(s0, s1, p0);
#pragma unroll
        for (int m = 0; m < 4; ++m) {
          const bf16x8 v = rd_v(0, m);
#pragma unroll
          for (int j = 0; j < PB; ++j) oacc[j][m & 1] = Mfma<T>::mma(v, p0[j][m >> 1], oacc[j][m & 1]);
        }
        probs(s1, p1);
        fixup(s1, s0, p1);
#pragma unroll
        for (int m = 0; m < 4; ++m) {
          const bf16x8 v = rd_v(1, m);
#pragma unroll
          for (int j = 0; j < PB; ++j) oacc[j][m & 1] = Mfma<T>::mma(v, p1[j][m >> 1], oacc[j][m & 1]);
        }
#pragma unroll
        for (int j = 0; j < PB; ++j) l_run[j] = ls[j][0];
        // no DMA may still target this workgroup's LDS when it retires
        wait_vm<0>();
        if constexpr (RAW) {
          float z = 0.0f;                  // NaN where a sum or output is not finite
          bool low = false;
#pragma unroll
          for (int j = 0; j < PB; ++j) {
            z = __builtin_fmaf(l_run[j], 0.0f, z);
#pragma unroll
            for (int h = 0; h < HT; ++h)
#pragma unroll
              for (int e = 0; e < 16; ++e) z = __builtin_fmaf(oacc[j][h][e], 0.0f, z);
            if (__builtin_amdgcn_ballot_w64(l_run[j] < kRawSumMin) != 0) {
#pragma unroll
              for (int h = 0; h < HT; ++h)
#pragma unroll
                for (int e = 0; e < 16; ++e) low = low || fabsf(oacc[j][h][e]) < kRawOutMin;
            }
          }
          __syncthreads();                 // every wave past its last tile read
          if (tid == 0) *flag = 0;
          __syncthreads();
          if (__builtin_amdgcn_ballot_w64(z != 0.0f || low) != 0) *flag = 1;
          __syncthreads();
          const bool bad = __builtin_amdgcn_readfirstlane(*flag) != 0;
          __syncthreads();                 // read by every wave before a safe pass fetches
          return !bad;
        }
      }
      return true;
    };
    if constexpr (QB == 1) {
      pass(std::integral_constant<int, 1>{}, qf, oacc, m_run, l_run);
    } else if (!pass(std::integral_constant<int, QB>{}, qf, oacc, m_run, l_run)) {
      static_for<QB>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        f32x16 o[1][HT] = {};
        float m[1] = {-INFINITY}, l[1] = {0.0f};
        u32x4 q[1][NKS];
#pragma unroll
        for (int s = 0; s < NKS; ++s) q[0][s] = qf[j][s];
        pass(std::integral_constant<int, 1>{}, q, o, m, l);
        __syncthreads();                 // every wave past its last tile read
#pragma unroll
        for (int h = 0; h < HT; ++h) oacc[j][h] = o[0][h];
        l_run[j] = l[0];
      });
    }
    if constexpr (KS > 1) {
      // Merge the key groups' (max, sum, output) through LDS, in group order:
      // M = max(m_0, m_1), each group weighted by 2^((m_k - M) c).
      __syncthreads();                   // every wave past its last tile read
      float* xs = reinterpret_cast<float*>(lds) + (size_t)qw * (16 * HT + 2) * 64;
      if (kgrp == 1) {
#pragma unroll
        for (int u = 0; u < HT; ++u)
#pragma unroll
          for (int e = 0; e < 16; ++e) xs[(16 * u + e) * 64 + lane] = oacc[0][u][e];
        xs[16 * HT * 64 + lane] = m_run[0];
        xs[(16 * HT + 1) * 64 + lane] = l_run[0];
      }
      __syncthreads();
      if (kgrp == 1) return;
      const float m1 = xs[16 * HT * 64 + lane], l1 = xs[(16 * HT + 1) * 64 + lane];
      const float mm = fmaxf(m_run[0], m1);
      const float a0 = __builtin_amdgcn_exp2f((m_run[0] - mm) * c);
      const float a1 = m1 == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f((m1 - mm) * c);
#pragma unroll
      for (int u = 0; u < HT; ++u)
#pragma unroll
        for (int e = 0; e < 16; ++e) oacc[0][u][e] = oacc[0][u][e] * a0 + xs[(16 * u + e) * 64 + lane] * a1;
      l_run[0] = l_run[0] * a0 + l1 * a1;
      m_run[0] = mm;
    }
  } else {
    // S^T tiles of the tile in buffer buf: rows = keys 32*kt + ..., cols = this
    // wave's 32 queries.
    auto qk = [&](int buf, f32x16 (&sacc)[2]) {
      const char* Ks = lds + buf * (KBUF + VBUF);
  #pragma unroll
      for (int kt = 0; kt < 2; ++kt) {
  #pragma unroll
        for (int s = 0; s < NKS; ++s) {
          const u32x4 kf = *reinterpret_cast<const u32x4*>(Ks + (kt * 32 + r32) * KRS + s * 32 + g * 16);
  #pragma unroll
          for (int u = 0; u < MMA_PER_READ; ++u) {
            typename Mfma<T>::frag a, bq;
            if constexpr (ES == 2) {
              a = __builtin_bit_cast(bf16x8, kf);
              bq = __builtin_bit_cast(bf16x8, qf[0][s]);
            } else {
              a = __builtin_bit_cast(f32x4, kf)[u];
              bq = __builtin_bit_cast(f32x4, qf[0][s])[u];
            }
            // the first instruction of each tile starts from a zero accumulator
            sacc[kt] = Mfma<T>::mma(a, bq, (s == 0 && u == 0) ? f32x16{} : sacc[kt]);
          }
        }
      }
    };

    // Online softmax of tile t's scores and O^T += V^T P^T with V from buffer buf.
    auto softmax_pv = [&](int t, int buf, f32x16 (&sacc)[2]) {
      const int kv0 = t * kBKV;
      const char* Vt = lds + buf * (KBUF + VBUF) + KBUF;

      // Key of element e: kv0 + 32*kt + 8*(e/4) + 4*g + e%4. Mask the ragged tail.
      if (kv0 + kBKV > nk) {
  #pragma unroll
        for (int kt = 0; kt < 2; ++kt)
  #pragma unroll
          for (int e = 0; e < 16; ++e)
            if (kv0 + kt * 32 + 8 * (e >> 2) + 4 * g + (e & 3) >= nk) sacc[kt][e] = -INFINITY;
      }
      // Max over this lane's 32 scores (two independent v_max3 chains).
      const float m0 = max16(sacc[0]), m1 = max16(sacc[1]);
      float mx = max3(m0, m1, m1);
      // Lazy rescale: move the reference max only when some score exceeds it by
      // more than 2^8 (base 2). m_run[0] is the same in lanes l and l ^ 32 (it only
      // changes here, from the query's full max), so each lane tests its own
      // 32 keys and the wave-wide vote covers the query's other 32; the
      // exchange for the full max is needed only in the (rare) branch.
      if (__builtin_amdgcn_ballot_w64((mx - m_run[0]) * c > kRescaleLog2) != 0) {
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        const float m_new = fmaxf(m_run[0], mx);
        const float alpha = __builtin_amdgcn_exp2f((m_run[0] - m_new) * c);
        m_run[0] = m_new;
        l_run[0] *= alpha;
  #pragma unroll
        for (int u = 0; u < HT; ++u)
  #pragma unroll
          for (int e = 0; e < 16; ++e) oacc[0][u][e] *= alpha;
      }
      const float mc = m_run[0] * c;
  #pragma unroll
      for (int kt = 0; kt < 2; ++kt)
  #pragma unroll
        for (int e = 0; e < 16; ++e) {
          const float pe = __builtin_amdgcn_exp2f(fmaf(sacc[kt][e], c, -mc));
          sacc[kt][e] = pe;
          if constexpr (ES == 4) l_run[0] += pe;
        }

      // O^T += V^T P^T over the 64 keys.
  #pragma unroll
      for (int kt = 0; kt < 2; ++kt)
  #pragma unroll
        for (int u = 0; u < 16 / E; ++u) {
          typename Mfma<T>::frag pf;
          if constexpr (ES == 2) {
  #pragma unroll
            for (int e = 0; e < 8; ++e) pf[e] = (bf16)sacc[kt][8 * u + e];
            // Row sum of the probabilities as rounded for the PV product (v_dot2 with 1s).
            const bf16x2 ones = {(bf16)1.0f, (bf16)1.0f};
            l_run[0] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pf, pf, 0, 1), ones, l_run[0], false);
            l_run[0] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pf, pf, 2, 3), ones, l_run[0], false);
            l_run[0] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pf, pf, 4, 5), ones, l_run[0], false);
            l_run[0] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pf, pf, 6, 7), ones, l_run[0], false);
          } else {
            pf = sacc[kt][u];
          }
  #pragma unroll
          for (int h = 0; h < HT; ++h) {
            typename Mfma<T>::frag vf;
            if constexpr (ES == 2) {
              const char* vrow = Vt + (h * 32 + r32) * VRS;
              const int key0 = kt * 32 + 16 * u + 4 * g;
              const u32x2 lo = *reinterpret_cast<const u32x2*>(vrow + key0 * ES);
              const u32x2 hi = *reinterpret_cast<const u32x2*>(vrow + (key0 + 8) * ES);
              vf = __builtin_bit_cast(bf16x8, u32x4{lo[0], lo[1], hi[0], hi[1]});
            } else {
              const char* vrow = Vt + (h * 32 + r32) * VRS;
              const int key = kt * 32 + 8 * (u >> 2) + 4 * g + (u & 3);
              vf = *reinterpret_cast<const float*>(vrow + key * ES);
            }
            oacc[0][h] = Mfma<T>::mma(vf, pf, oacc[0][h]);
          }
        }
    };
    auto compute = [&](int t, int buf) {
      f32x16 sacc[2];
      qk(buf, sacc);
      softmax_pv(t, buf, sacc);
    };
    // Fetches are unconditional (past the end they re-read the last tile), so
    // the wait before staging tile t+1 does not cover the loads of tile t+2.
    auto tile = [&](int t, int r) {      // r = (t - t_begin) & 1 (a constant at each call site)
      fetch(min(t * kBKV + 2 * kBKV, last_kv), r);
      compute(t, r);
      stage(r ^ 1, r ^ 1);
      __syncthreads();
    };
    if (t_begin < t_end) {               // uniform over the workgroup
      fetch(t_begin * kBKV, 0);
      fetch(min((t_begin + 1) * kBKV, last_kv), 1);
      stage(0, 0);
      __syncthreads();
      int t = t_begin;
      for (; t + 1 < t_end; t += 2) {
        tile(t, 0);
        tile(t + 1, 1);
      }
      if (t < t_end) tile(t, 0);
    }
  }

#pragma unroll
  for (int j = 0; j < QB; ++j) {
    const int i = qi + 32 * j;
    // the matrix-core path's sums already cover both key halves of the wave
    const float l_tot = DMA ? l_run[j] : l_run[j] + __shfl_xor(l_run[j], 32);
    if (i >= nq) return;
    if constexpr (SPLIT) {
      const size_t prow = ((size_t)sp * p.rows + (q_begin - p.qs.off[0] + i)) * p.heads + head;
      float* po = p.part_o + prow * HD;
#pragma unroll
      for (int h = 0; h < HT; ++h)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4)
          *reinterpret_cast<float4*>(po + h * 32 + 8 * q4 + 4 * g) = make_float4(
              oacc[j][h][4 * q4], oacc[j][h][4 * q4 + 1], oacc[j][h][4 * q4 + 2], oacc[j][h][4 * q4 + 3]);
      if (g == 0) *reinterpret_cast<float2*>(p.part_ml + prow * 2) = make_float2(m_run[j] * c, l_tot);
    } else {
      const float inv = 1.0f / l_tot;
      T* orow = reinterpret_cast<T*>(p.o + ((size_t)(q_begin + i) * p.ldo + head * HD) * ES);
#pragma unroll
      for (int h = 0; h < HT; ++h)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          float v[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = oacc[j][h][4 * q4 + e] * inv;
          T* dst = orow + h * 32 + 8 * q4 + 4 * g;
          if constexpr (ES == 2) {
            bf16x4 o4;
#pragma unroll
            for (int e = 0; e < 4; ++e) o4[e] = (bf16)v[e];
            *reinterpret_cast<bf16x4*>(dst) = o4;
          } else {
            *reinterpret_cast<float4*>(dst) = make_float4(v[0], v[1], v[2], v[3]);
          }
        }
    }
  }
}

// Merge of the key-range splits: one thread per (query row, head, 4 output
// columns). With M = max_s m_s, w_s = 2^(m_s - M): o = sum_s w_s O_s / sum_s w_s l_s.
template <typename T, int HD>
__global__ __launch_bounds__(256) void k_attn_combine(AttnArgs p) {
  constexpr int D4 = HD / 4;
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= (int64_t)p.rows * p.heads * D4) return;
  const int d = (int)(i % D4) * 4;
  const int64_t rh = i / D4;                           // row * heads + head
  const int head = (int)(rh % p.heads);
  const int64_t row = rh / p.heads;
  const size_t split_stride = (size_t)p.rows * p.heads;
  float mx = -INFINITY;
  for (int s = 0; s < p.splits; ++s) mx = fmaxf(mx, p.part_ml[(s * split_stride + rh) * 2]);
  float l = 0.0f;
  float4 acc = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  for (int s = 0; s < p.splits; ++s) {
    const float2 ml = *reinterpret_cast<const float2*>(p.part_ml + (s * split_stride + rh) * 2);
    const float w = exp2f(ml.x - mx);                  // 0 for an empty split (max -inf)
    const float4 o = *reinterpret_cast<const float4*>(p.part_o + (s * split_stride + rh) * HD + d);
    l += w * ml.y;
    acc.x += w * o.x;
    acc.y += w * o.y;
    acc.z += w * o.z;
    acc.w += w * o.w;
  }
  const float inv = 1.0f / l;
  T* dst = reinterpret_cast<T*>(p.o) + (size_t)(p.qs.off[0] + row) * p.ldo + head * HD + d;
  if constexpr (sizeof(T) == 2) {
    bf16x4 o4;
    o4[0] = (bf16)(acc.x * inv);
    o4[1] = (bf16)(acc.y * inv);
    o4[2] = (bf16)(acc.z * inv);
    o4[3] = (bf16)(acc.w * inv);
    *reinterpret_cast<bf16x4*>(dst) = o4;
  } else {
    *reinterpret_cast<float4*>(dst) = make_float4(acc.x * inv, acc.y * inv, acc.z * inv, acc.w * inv);
  }
}

template <typename T, int HD, int NW, int SITE, int KS = 1, bool QS = false, int QB = 1>
hipError_t launch_k(const AttnArgs& a, int tiles, hipStream_t s) {
  const dim3 block(64 * NW);
  if constexpr (KS > 1 || QB > 1) {
    if (a.splits != 1) return hipErrorInvalidValue;
    launch((k_attn<T, HD, NW, SITE, false, KS, QS, QB>), dim3(tiles * a.heads), block, 0, s, a);
    return hipGetLastError();
  } else {
    if (a.splits == 1) {
      launch((k_attn<T, HD, NW, SITE, false, 1, QS>), dim3(tiles * a.heads), block, 0, s, a);
      return hipGetLastError();
    }
    launch((k_attn<T, HD, NW, SITE, true, 1, QS>), dim3(tiles * a.heads * a.splits), block, 0, s, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int64_t n = (int64_t)a.rows * a.heads * (HD / 4);
    launch((k_attn_combine<T, HD>), dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, a);
    return hipGetLastError();
  }
}

// splits > 1 requires a.part_o / a.part_ml sized for them.
template <int NW, int SITE, int KS = 1, int QB = 1>
hipError_t launch_a(int dt, int hd, const AttnArgs& a0, int heads, int splits, hipStream_t s, bool qs) {
  AttnArgs a = a0;
  constexpr int BQ = 32 * QB * NW / KS;
  a.tile_off[0] = 0;
  for (int b = 0; b < a.qs.B; ++b) a.tile_off[b + 1] = a.tile_off[b] + (a.qs.off[b + 1] - a.qs.off[b] + BQ - 1) / BQ;
  const int tiles = a.tile_off[a.qs.B];
  if (tiles == 0) return hipSuccess;
  a.heads = heads;
  a.splits = splits;
  a.rows = a.qs.off[a.qs.B] - a.qs.off[0];
  if (dt == DT_BF16 && hd == 64) {
    if (qs) return launch_k<bf16, 64, NW, SITE, KS, true, QB>(a, tiles, s);
    // the model's own calls always store their queries scaled
    if constexpr (SITE == SITE_OP) return launch_k<bf16, 64, NW, SITE, KS, false, QB>(a, tiles, s);
    return hipErrorInvalidValue;
  }
  if constexpr (KS == 1 && QB == 1) {
    if (dt == DT_BF16 && hd == 32) return launch_k<bf16, 32, NW, SITE>(a, tiles, s);
    if (dt == DT_F32 && hd == 64) return launch_k<float, 64, NW, SITE>(a, tiles, s);
    if (dt == DT_F32 && hd == 32) return launch_k<float, 32, NW, SITE>(a, tiles, s);
  }
  return hipErrorInvalidValue;
}

// Bytes of split partials for `splits` splits of `rows` query rows.
inline size_t split_bytes(int splits, int rows, int heads, int hd) {
  return (size_t)splits * rows * heads * (hd + 2) * sizeof(float);
}

// Launch shapes of the matrix-core path (bf16, 64-wide heads). The time is
// about the number of key tiles times the rounds of workgroups over 256 CUs
// times the shape's time per tile, in us, measured on MI355X with 16 heads:
//   512 queries, 8 waves of 64        1.35   one workgroup per CU
//   256 queries, 4 waves of 64        1.35   two per CU (0.9 for one alone)
//   256 queries, 8 waves of 32        0.85   one per CU
//   128 queries, 8 waves, key groups  0.5    one per CU: half the key tiles per wave
//    64 queries, 4 waves, key groups  0.35   one per CU
// The shape with the smallest product is taken. It picks the fastest of the five
// at 820 (9.4 us; the others 11.6 to 25.2), 1639 (17.5; 23.9 to 41.3), 2000
// (21.2; 28.1 to 48.2), 6000 (136; 143 to 192), 9831 (361; 379 to 499) and
// 32768 queries (3388; 3390 to 5636), and ties at 4096 (62.3 and 62.4).
// Waves of 64 queries take raw passes, whose probabilities are relative to no
// maximum: with few keys that costs the exactness of the largest one (64 keys:
// error against float64 2.2e-3 -> 2.4e-3; from 700 keys on no difference), so
// they are left out below kRawMinTiles. There the rounds' own cost counts too
// (launch, queries, first tile, output): the other three take 3.9 + 0.27 t, 5.25 +
// 0.43 t and 4.4 + 0.92 t us per round at t key tiles, a fit that picks the fastest
// at every measured shape of 200 to 32768 queries (9831 x 64 keys: 256 queries
// 17.6 us, 128 with key groups 30.8; x 257 27.3 and 37.3; x 600 41 and 47).
//
// Key-range splits over workgroups of four waves, merged by a second kernel,
// shorten the chain of key tiles further while all of them fit one round and
// every split keeps at least 8 key tiles; they cost about 4.5 us more in fixed
// cost, so they are taken where few queries leave most of the chip idle and
// splits shorten the chain by more than kSplitGainTiles over key groups (64 x
// 4096 keys: 29.7 against 16.4 us with eight splits). Other types and head
// sizes: eight waves of 32 queries from 160 workgroups up (about 2300
// queries), else four, with splits.
constexpr long kSplitGainTiles = 5;
constexpr long kRawMinTiles = 12;

template <int SITE>
hipError_t launch_site(int dt, int hd, const AttnArgs& a, int heads, float* ws, size_t ws_bytes, hipStream_t s,
                       bool qs) {
  long t64 = 0, t128 = 0, t256 = 0, t512 = 0, kt_min = 1L << 30, kt_max = 0;
  for (int b = 0; b < a.qs.B; ++b) {
    const int nq = a.qs.off[b + 1] - a.qs.off[b];
    if (nq == 0) continue;
    t64 += (nq + 63) / 64;
    t128 += (nq + 127) / 128;
    t256 += (nq + 255) / 256;
    t512 += (nq + 511) / 512;
    const long kt = (a.ks.off[b + 1] - a.ks.off[b] + kBKV - 1) / kBKV;
    kt_min = std::min(kt_min, kt);
    kt_max = std::max(kt_max, kt);
  }
  const bool dma = dt == DT_BF16 && hd == 64;
  // The DMA path addresses a sample's key and value rows with 32-bit offsets
  // from the sample's first row.
  if (dma && kt_max * kBKV * (int64_t)std::max(a.ldk, a.ldv) * 2 >= (int64_t(1) << 31)) return hipErrorInvalidValue;
  int splits = 1;
  if (t256 * heads < 160) {
    while (splits < 8 && t128 * heads * splits * 2 <= 256 && kt_min >= 16 * splits) splits *= 2;
    const int rows = a.qs.off[a.qs.B] - a.qs.off[0];
    while (splits > 1 && (!ws || split_bytes(splits, rows, heads, hd) > ws_bytes)) splits /= 2;
    if (dma && (kt_max + 1) / 2 - (kt_max + splits - 1) / splits <= kSplitGainTiles) splits = 1;
  }
  if (dma && splits == 1) {
    const auto rounds = [&](long tiles, long wgs) { return (double)((tiles * heads + wgs - 1) / wgs); };
    enum { Q64K, Q128K, Q256, Q256P, Q512 };
    const long left = t256 * heads % 512;
    const double cost[] = {0.35 * rounds(t64, 256), 0.5 * rounds(t128, 256), 0.85 * rounds(t256, 256),
                           1.35 * (t256 * heads / 512) + (left == 0 ? 0.0 : left <= 256 ? 0.9 : 1.35),
                           1.35 * rounds(t512, 256)};
    const double t = (double)kt_max;        // (the fit holds for few tiles in every sample)
    const double few[] = {(3.9 + 0.27 * t) * rounds(t64, 256), (5.25 + 0.43 * t) * rounds(t128, 256),
                          (4.4 + 0.92 * t) * rounds(t256, 256)};
    int pick = Q64K;
    for (int i = Q128K; i <= (kt_min >= kRawMinTiles ? Q512 : Q256); ++i) {
      const double* c = kt_max >= kRawMinTiles ? cost : few;
      if (c[i] <= c[pick]) pick = i;
    }
    switch (pick) {
      case Q64K: return launch_a<4, SITE, 2>(dt, hd, a, heads, 1, s, qs);
      case Q128K: return launch_a<8, SITE, 2>(dt, hd, a, heads, 1, s, qs);
      case Q256: return launch_a<8, SITE>(dt, hd, a, heads, 1, s, qs);
      case Q256P: return launch_a<4, SITE, 1, 2>(dt, hd, a, heads, 1, s, qs);
      default: return launch_a<8, SITE, 1, 2>(dt, hd, a, heads, 1, s, qs);
    }
  }
  if (t256 * heads >= 160) return launch_a<8, SITE>(dt, hd, a, heads, 1, s, qs);
  AttnArgs b = a;
  if (splits > 1) {
    b.part_o = ws;
    b.part_ml = ws + (size_t)splits * (a.qs.off[a.qs.B] - a.qs.off[0]) * heads * hd;
  }
  return launch_a<4, SITE>(dt, hd, b, heads, splits, s, qs);
}

}  // namespace

hipError_t launch_attention(int site, int dt, int heads, int hd, const Segs& qs, const Segs& ks, const void* q,
                            int ldq, const void* k, int ldk, const void* v, int ldv, void* o, int ldo, float* ws,
                            size_t ws_bytes, hipStream_t s, bool q_scaled) {
  AttnArgs a;
  a.qs = qs;
  a.ks = ks;
  a.q = (const char*)q;
  a.k = (const char*)k;
  a.v = (const char*)v;
  a.o = (char*)o;
  a.ldq = ldq;
  a.ldk = ldk;
  a.ldv = ldv;
  a.ldo = ldo;
  a.scale_log2 = q_scaled ? 1.0f : attention_q_scale(hd);
  a.splits = 1;
  a.part_o = a.part_ml = nullptr;
  if (site == SITE_SELF) return launch_site<SITE_SELF>(dt, hd, a, heads, ws, ws_bytes, s, q_scaled);
  if (site == SITE_CROSS) return launch_site<SITE_CROSS>(dt, hd, a, heads, ws, ws_bytes, s, q_scaled);
  return launch_site<SITE_OP>(dt, hd, a, heads, ws, ws_bytes, s, q_scaled);
}

}  // namespace f3c
