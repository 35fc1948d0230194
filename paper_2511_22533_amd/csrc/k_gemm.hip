// Dense projections of the transformer blocks on the matrix cores:
// C = A W^T + bias, A = activations [M][K] (row-major, K contiguous),
// W = weights [N][K] (torch Linear layout, K contiguous), f32 accumulation.
// Epilogues fuse the bias with a dtype store (QKV / cross-attention Q / KV),
// GELU (tanh form, MLP fc1), or a gated residual update in f32
// (h += gate * (.), attention output projections and MLP fc2).
//
// bf16 (k_gemm_dma): K tiles go HBM -> LDS by DMA into two to four stages, and
// each MFMA stands in a scheduling group of its own with a fragment read of the
// next 16-element K-step (and, with more than two stages, its share of the
// DMA). f32 (k_gemm_f32): K staged 128 bytes at a time through registers into
// padded LDS rows (144-byte stride: the 16-byte fragment reads of 16
// consecutive lanes cover all 64 banks once), two tiles ahead.
//
// Every output is one workgroup's sum in one K order, the same for every tile
// shape, so the shape may follow the row count without changing a result.
//
// The weight fragment is the MFMA's A operand and the activation fragment its
// B operand, i.e. each instruction produces a tile of C^T: a lane then
// holds one activation row and four consecutive output columns per
// accumulator group, moved as 16-byte vectors. A lane reads 16 contiguous bytes
// of one row at K-group offset l/32 for both operands; any common assignment
// of K elements to the instruction's K slots yields the same dot products.
#include <algorithm>
#include <cmath>
#include <initializer_list>

#include "common.h"
#include "kernels.h"

namespace f3c {

namespace {

constexpr int kBKB = 128;             // K bytes per LDS tile row
constexpr int kRS = kBKB + 16;        // padded LDS row stride (bytes)

struct GemmArgs {
  int M, N, K;
  const char* A;
  int lda;                            // elements
  const char* W;
  int ldw;
  const float* bias;
  const float* gate;
  void* out;
  int ldo;
  float* resid;
  int ldr;
  int xq;                             // column groups of the XCD tile partition (divides N / BN)
  float oscale;                       // stored outputs of columns < oscale_cols are multiplied by oscale
  int oscale_cols;
  bool out16;                         // stored rows are 16-byte aligned (else 8)
};

// f32 projections on the 16x16x4 matrix instruction (the rate of 32x32x2 at a
// quarter of the tile): four waves in a 2 x 2 arrangement, each with TM x TN
// tiles. What bounds them at a few hundred rows is the chain of matrix
// instructions of one wave, so few rows take few tiles per wave; at many rows
// the matrix rate, which more waves per SIMD keep up. Measured, us, with one
// 64 x 128 workgroup of 32x32x2 / the workgroup tile taken: 512 x 128 x 512 21.6 /
// 5.9 (32 x 32), 1728 x 256 x 1024 39.6 / 13.5 (32 x 32), 4096 x 256 x 1024 39.9 /
// 22.8 (32 x 64), 9831 x 1024 x 1024 171 / 170 (64 x 64; 176 with 64 x 128), 9831 x
// 4096 x 1024 664 / 645, 32768 x 1024 x 1024 538 / 532 (64 x 64).
template <int TM, int TN, int EPI, int SITE>
__global__ __launch_bounds__(256) void k_gemm_f32(GemmArgs p) {
  constexpr int WTM = 16 * TM, WTN = 16 * TN, BM = 2 * WTM, BN = 2 * WTN, NT = 256, PF = 2;
  constexpr int CA = BM * 8 / NT, CB = BN * 8 / NT;         // 16-byte chunks per thread
  constexpr int ABUF = BM * kRS, BBUF = BN * kRS;
  static_assert(CA >= 1 && CB >= 1, "tile too small for the workgroup");
  __shared__ __attribute__((aligned(16))) char lds[2 * (ABUF + BBUF)];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int g = lane >> 4, r16 = lane & 15;
  // Tile of this workgroup. Workgroups go round-robin to the 8 XCDs, each with
  // its own L2; the 1-D grid is remapped so that XCD j gets one contiguous run
  // of a tile order that is column-group major (xq groups of N/BN/xq column
  // tiles), then row-panel major. Each XCD then reads about 1/(8/xq) of A and
  // 1/xq of W instead of all of A (a row panel's column tiles on different
  // XCDs): HBM-side traffic xq*|A| + (8/xq)*|W|.
  int n0, m0;
  {
    const int gx = p.N / BN, gy = (p.M + BM - 1) / BM;
    const int l = xcd_logical_id(blockIdx.x, gx * gy);
    const int gq = gx / p.xq, per_group = gy * gq;
    const int grp = l / per_group, r = l - grp * per_group;
    const int y = r / gq;
    n0 = (grp * gq + (r - y * gq)) * BN;
    m0 = y * BM;
  }
  const size_t lda_b = (size_t)p.lda * 4, ldw_b = (size_t)p.ldw * 4;
  const int KT = (p.K * 4) / kBKB;

  // Rows past M are loaded from row M-1 (always valid) and never stored.
  const char* a_row[CA];
  const char* w_row[CB];
  int chunk_a[CA], chunk_b[CB];
#pragma unroll
  for (int q = 0; q < CA; ++q) {
    const int c = tid + NT * q, row = c >> 3;
    a_row[q] = p.A + (size_t)min(m0 + row, p.M - 1) * lda_b + (c & 7) * 16;
    chunk_a[q] = row * kRS + (c & 7) * 16;
  }
#pragma unroll
  for (int q = 0; q < CB; ++q) {
    const int c = tid + NT * q, row = c >> 3;
    w_row[q] = p.W + (size_t)(n0 + row) * ldw_b + (c & 7) * 16;
    chunk_b[q] = row * kRS + (c & 7) * 16;
  }

  // PF register sets: set r holds the tile whose index is congruent to r mod PF.
  u32x4 ra[PF][CA], rb[PF][CB];
  auto load_tile = [&](int kt, int r) {
    const size_t kb = (size_t)kt * kBKB;
#pragma unroll
    for (int q = 0; q < CA; ++q) ra[r][q] = *reinterpret_cast<const u32x4*>(a_row[q] + kb);
#pragma unroll
    for (int q = 0; q < CB; ++q) rb[r][q] = *reinterpret_cast<const u32x4*>(w_row[q] + kb);
  };
  auto store_tile = [&](int buf, int r) {
    char* As = lds + buf * (ABUF + BBUF);
    char* Bs = As + ABUF;
#pragma unroll
    for (int q = 0; q < CA; ++q) *reinterpret_cast<u32x4*>(As + chunk_a[q]) = ra[r][q];
#pragma unroll
    for (int q = 0; q < CB; ++q) *reinterpret_cast<u32x4*>(Bs + chunk_b[q]) = rb[r][q];
  };

  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

  // A lane reads 16 bytes of row l%16 at K-group l/16 of every 16 floats of K;
  // element u of both operands meets in instruction u.
  auto compute = [&](int buf) {
    const char* As = lds + buf * (ABUF + BBUF);
    const char* Bs = As + ABUF;
#pragma unroll
    for (int ks = 0; ks < kBKB / 64; ++ks) {
      f32x4 fa[TM], fb[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i)
        fa[i] = *reinterpret_cast<const f32x4*>(As + (wm * WTM + i * 16 + r16) * kRS + ks * 64 + g * 16);
#pragma unroll
      for (int j = 0; j < TN; ++j)
        fb[j] = *reinterpret_cast<const f32x4*>(Bs + (wn * WTN + j * 16 + r16) * kRS + ks * 64 + g * 16);
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)   // C^T tile: rows = output columns
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[j][u], fa[i][u], acc[i][j], 0, 0, 0);
    }
  };

  // Two LDS buffers: at step kt the loads of tile kt + 2 are issued while tile
  // kt is consumed and tile kt + 1 (loaded a step earlier) is staged. Loads are
  // issued unconditionally (past the end they re-read the last tile), so the
  // wait before staging only covers the oldest load group.
#pragma unroll
  for (int r = 0; r < PF; ++r) load_tile(min(r, KT - 1), r);
  store_tile(0, 0);
  __syncthreads();
  auto step = [&](int kt, int r) {     // r = kt % 2 (a constant at each call site)
    load_tile(min(kt + PF, KT - 1), r);
    compute(r);
    store_tile(r ^ 1, r ^ 1);
    __syncthreads();
  };
  int kt = 0;
  for (; kt + 2 <= KT; kt += 2) {
    step(kt, 0);
    step(kt + 1, 1);
  }
  if (kt < KT) step(kt, 0);

  // Epilogue. Tile (i, j): activation row m0 + wm*WTM + 16 i + r16, output
  // columns n0 + wn*WTN + 16 j + 4 g + (0..3).
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int row = m0 + wm * WTM + i * 16 + r16;
    if (row >= p.M) continue;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int col = n0 + wn * WTN + j * 16 + 4 * g;
      const float4 bv = *reinterpret_cast<const float4*>(p.bias + col);
      const f32x4& c = acc[i][j];
      float v[4] = {c[0] + bv.x, c[1] + bv.y, c[2] + bv.z, c[3] + bv.w};
      if constexpr (EPI == EPI_RESID) {
        float4 gv = make_float4(1.0f, 1.0f, 1.0f, 1.0f);
        if (p.gate) gv = *reinterpret_cast<const float4*>(p.gate + col);
        float4* r = reinterpret_cast<float4*>(p.resid + (size_t)row * p.ldr + col);
        float4 h = *r;
        h.x += gv.x * v[0];
        h.y += gv.y * v[1];
        h.z += gv.z * v[2];
        h.w += gv.w * v[3];
        *r = h;
      } else {
        if constexpr (EPI == EPI_GELU) {
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = gelu_tanh(v[e]);
        }
        if (col < p.oscale_cols) {        // four columns: all in or all out (oscale_cols % 4 == 0)
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] *= p.oscale;
        }
        *reinterpret_cast<float4*>(reinterpret_cast<float*>(p.out) + (size_t)row * p.ldo + col) =
            make_float4(v[0], v[1], v[2], v[3]);
      }
    }
  }
}

// bf16 projections. What bounds them: at 32768 rows and K = 4096 the 256 x 256
// tiles run at about half of the matrix rate (270 us, 1.02 PFLOP/s; the main
// loop alone, from the slope over K, at 1.44), with the residual's read and
// write and each round's fill and drain beside it; at a few hundred rows it is
// the chain of K tiles of one workgroup. Against the kernels these replaced
// (register-staged 128 x 128, 64 x 128 and 64 x 64 tiles, a 256 x 256 kernel
// with hand-written K-steps, four K-groups per tile for K = 4096), each call
// repeated by itself on the same operands (in a step, behind other
// kernels, the large ones gain less: fc1 and fc2 at 32768 rows 15 us together), us:
//   QKV   32768 x 3072 x 1024  235 -> 192   9831 rows  78 -> 63   1639 rows 21.7 -> 16.0
//   fc1   32768 x 4096 x 1024  317 -> 295   9831 rows 115 -> 103  820 rows  14.6 -> 12.0
//   fc2   32768 x 1024 x 4096  288 -> 270   9831 rows 114 -> 97   4096 rows 46 -> 38
//   O     32768 x 1024 x 1024  115 -> 90    4096 rows 19.4 -> 18  820 rows  8.3 -> 7.0
// over 225 shapes of width 512 to 2048 and 200 to 32768 rows, 1.24 times as fast
// in the geometric mean, from 0.99 (2048 x 8192, 200 rows) to 2.4.
template <int BM, int BN, int WGM, int WGN, int STAGES, int OCC, int EPI, int SITE, bool WIDE = false>
__global__ __launch_bounds__(64 * WGM * WGN, OCC) void k_gemm_dma(GemmArgs p) {
  constexpr int NW = WGM * WGN, WTM = BM / WGM, WTN = BN / WGN, TM = WTM / 32, TN = WTN / 32;
  constexpr int KTB = 128, SBUF = (BM + BN) * KTB, ABUF = BM * KTB;    // bytes of a K tile row, a stage, its A rows
  constexpr int KSTEPS = KTB / 32, CPR = KTB / 16, RPB = 1024 / KTB;   // 16-element K-steps, 16-byte chunks, DMA rows
  constexpr int DA = BM / RPB, DB = BN / RPB, DQ = (DA + DB) / NW;
  static_assert(DB % NW == 0 && DA % NW == 0, "whole DMA blocks per wave");
  static_assert(BM % (32 * WGM) == 0 && BN % (32 * WGN) == 0 && STAGES >= 2, "tile shape");
  __shared__ __attribute__((aligned(16))) char lds[STAGES * SBUF];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WGN, wn = wave % WGN;
  const int g = lane >> 5, r32 = lane & 31;
  int n0, m0;
  {
    const int gx = p.N / BN, gy = (p.M + BM - 1) / BM;
    const int l = xcd_logical_id(blockIdx.x, gx * gy);
    const int gq = gx / p.xq, per_group = gy * gq;
    const int grp = l / per_group, r = l - grp * per_group;
    const int y = r / gq;
    n0 = (grp * gq + (r - y * gq)) * BN;
    m0 = y * BM;
  }
  // (the tile order is k_gemm_f32's)
  const uint32_t lda_b = (uint32_t)p.lda * 2, ldw_b = (uint32_t)p.ldw * 2;
  const int KT = (p.K * 2) / KTB;
  // LDS rows are the 128 bytes of a row's K tile, their 16-byte chunks
  // XOR-swizzled by row (the fragment reads of 16 consecutive rows are then
  // free of bank conflicts).
  auto swizzle = [](int row) { return (row >> 1) & 7; };
  auto descriptor = [](const char* base) {
    const uint64_t a = (uint64_t)base;
    return u32x4{(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)a),
                 (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(a >> 32) & 0xffffu), 0xffffffffu, 0x00020000u};
  };
  const u32x4 adesc = descriptor(p.A + (size_t)m0 * p.lda * 2), wdesc = descriptor(p.W + (size_t)n0 * p.ldw * 2);
  // DMA instruction q of this wave fills the 8 rows of block wave + NW q (A's
  // blocks first): lane l row l/8 at physical chunk l%8, with the logical chunk
  // that the row's swizzle maps there. Lane offsets from the tile's first row;
  // rows past M re-read row M - 1 (never stored). WIDE: row strides that 32-bit
  // offsets cannot span, as whole addresses.
  uint32_t dofs[DQ];
  const char* dsrc[DQ];
#pragma unroll
  for (int q = 0; q < DQ; ++q) {
    const int blk = wave + NW * q, phys = lane % CPR;
    if (q < DA / NW) {
      const int row = RPB * blk + lane / CPR, src = min(row, p.M - 1 - m0), ch = (phys ^ swizzle(row)) << 4;
      dofs[q] = (uint32_t)src * lda_b + ch;
      dsrc[q] = p.A + (size_t)(m0 + src) * p.lda * 2 + ch;
    } else {
      const int row = RPB * (blk - DA) + lane / CPR, ch = (phys ^ swizzle(row)) << 4;
      dofs[q] = (uint32_t)row * ldw_b + ch;
      dsrc[q] = p.W + (size_t)(n0 + row) * p.ldw * 2 + ch;
    }
    asm("" : "+v"(dofs[q]));
  }
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds;
  // DMA instruction q of K tile kt
  auto fetch1 = [&](int q, uint32_t k, int stage) {
    const uint32_t dst = lds0 + (uint32_t)(stage * SBUF + (wave + NW * q) * 1024);
    if constexpr (WIDE) {
      dma16(dsrc[q] + k, lds + stage * SBUF + (wave + NW * q) * 1024);
    } else if (q < DA / NW) {
      asm volatile("buffer_load_dwordx4 %0, %1, %2 offen lds"
                   : : "v"(dofs[q]), "s"(adesc), "s"(k), "{m0}"(dst) : "memory");
    } else {
      asm volatile("buffer_load_dwordx4 %0, %1, %2 offen lds"
                   : : "v"(dofs[q]), "s"(wdesc), "s"(k), "{m0}"(dst) : "memory");
    }
  };
  constexpr int GS = TM * TN, G = KSTEPS * GS;     // MFMA groups per K-step and per K tile
  // A tile's DMA instructions are spread over a whole tile's groups, or, with
  // two stages (no time to lose before the next barrier waits for them), over
  // one K-step's.
  constexpr bool SPR = STAGES > 2;
  constexpr int SPREAD = SPR ? G : GS;
  auto dpos = [](int q) { return q * SPREAD / DQ; };
  const int swz = swizzle(r32);
  uint32_t aad[KSTEPS], wad[KSTEPS];
#pragma unroll
  for (int ks = 0; ks < KSTEPS; ++ks) {
    const uint32_t ch = (uint32_t)(((2 * ks + g) ^ swz) << 4);
    aad[ks] = lds0 + (wm * WTM + r32) * KTB + ch;
    wad[ks] = lds0 + ABUF + (wn * WTN + r32) * KTB + ch;
    asm("" : "+v"(aad[ks]), "+v"(wad[ks]));
  }
  typedef __attribute__((address_space(3))) const u32x4 lds_u32x4;
  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;
  u32x4 fa[2][TM], fw[2][TN];
  // Fragment reads stand one per MFMA group, a K-step ahead; the barrier fixes
  // the groups (the compiler's own order gathers reads before the MFMAs).
  auto fence = [] { __builtin_amdgcn_sched_barrier(0); };
  auto read = [&](int set, int ks, int f) {       // fragment f of a K-step: A 0..TM-1, then W
    if (f < TM) fa[set][f] = *(lds_u32x4*)(uintptr_t)(aad[ks] + (uint32_t)(f * 32 * KTB));
    else fw[set][f - TM] = *(lds_u32x4*)(uintptr_t)(wad[ks] + (uint32_t)((f - TM) * 32 * KTB));
  };
  // Tile kt + STAGES goes into tile kt's stage, from the barrier before tile
  // kt's last K-step on; the part spread past that K-step is issued during
  // tile kt + 1.
  int stage = 0, dstage = STAGES - 1;
  uint32_t dk = (uint32_t)min(STAGES - 1, KT - 1) * KTB;
#pragma unroll
  for (int s = 0; s < STAGES; ++s)
#pragma unroll
    for (int q = 0; q < DQ; ++q)
      if (s < STAGES - 1 || dpos(q) < GS) fetch1(q, (uint32_t)min(s, KT - 1) * KTB, s);
  {
    constexpr int LATE = SPR ? DQ - (GS * DQ + G - 1) / G : 0;   // instructions of tile STAGES - 1 still to come
    wait_vm<(STAGES - 1) * DQ - LATE>();
  }
  __syncthreads();
#pragma unroll
  for (int f = 0; f < TM + TN; ++f) read(0, 0, f);
  fence();
  for (int kt = 0; kt < KT; ++kt) {
#pragma unroll
    for (int ks = 0; ks < KSTEPS; ++ks) {
      const int cur = ks & 1, nxt = cur ^ 1, kn = (ks + 1) % KSTEPS;
      if (ks == KSTEPS - 1) {
        // every wave holds this tile's last fragments and tile kt + 1 has
        // landed: one barrier retires tile kt's stage and opens kt + 1's
        __builtin_amdgcn_s_waitcnt(0xc07f);        // lgkmcnt(0)
        wait_vm<(STAGES - 2) * DQ>();
        __builtin_amdgcn_s_barrier();
        fence();
        dstage = stage;
        dk = (uint32_t)min(kt + STAGES, KT - 1) * KTB;
        const uint32_t d = stage == STAGES - 1 ? (uint32_t)(-(STAGES - 1) * SBUF) : (uint32_t)SBUF;
        stage = stage == STAGES - 1 ? 0 : stage + 1;
#pragma unroll
        for (int k = 0; k < KSTEPS; ++k) {
          aad[k] += d;
          wad[k] += d;
        }
        fence();
      }
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          const int n = i * TN + j;
          // the next K-step's fragments and the DMA, spread over the MFMAs
          constexpr int PER = (TM + TN + TM * TN - 1) / (TM * TN);
#pragma unroll
          for (int r = 0; r < PER; ++r)
            if (n * PER + r < TM + TN) read(nxt, kn, n * PER + r);
#pragma unroll
          for (int q = 0; q < DQ; ++q)
            if (dpos(q) == ((ks + 1) % KSTEPS) * GS + n) fetch1(q, dk, dstage);
          acc[i][j] = Mfma<bf16>::mma(__builtin_bit_cast(bf16x8, fw[cur][j]), __builtin_bit_cast(bf16x8, fa[cur][i]),
                                      acc[i][j]);
          fence();
        }
    }
  }
  wait_vm<0>();
  __syncthreads();                                 // no DMA in flight, every wave past its last fragment read
  // Epilogue through LDS, 32 rows of the wave at a time: a lane of the MFMA
  // layout holds four columns of one row, and storing those outright leaves
  // 16 bytes here and there of 32 rows per instruction (4096 x 4096 x 256:
  // 27.4 us, 17.6 through LDS with whole 64- to 256-byte row pieces). The
  // region is the wave's own and LDS operations of a wave keep their order.
  constexpr int RS = WTN * 4 + 16;
  static_assert(NW * 32 * RS <= STAGES * SBUF, "epilogue buffer");
  typedef __attribute__((address_space(3))) f32x4 lds_f4;
  const uint32_t eb = lds0 + (uint32_t)(wave * 32 * RS);
  // columns per lane, lanes per row, rows per pass
  constexpr int VC = EPI == EPI_RESID ? 4 : 8, LPR = WTN / VC, RPI = 64 / LPR;
  const int ecol = n0 + wn * WTN + (lane % LPR) * VC;
  float bv[VC], gv[VC];
#pragma unroll
  for (int e = 0; e < VC; e += 4) {
    const float4 b4 = *reinterpret_cast<const float4*>(p.bias + ecol + e);
    float4 g4 = make_float4(1.0f, 1.0f, 1.0f, 1.0f);
    if (EPI == EPI_RESID && p.gate) g4 = *reinterpret_cast<const float4*>(p.gate + ecol + e);
    bv[e] = b4.x, bv[e + 1] = b4.y, bv[e + 2] = b4.z, bv[e + 3] = b4.w;
    gv[e] = g4.x, gv[e + 1] = g4.y, gv[e + 2] = g4.z, gv[e + 3] = g4.w;
  }
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *(lds_f4*)(uintptr_t)(eb + (uint32_t)(r32 * RS + (j * 32 + 8 * q + 4 * g) * 4)) =
            f32x4{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
    // (the lanes read what others wrote: the compiler must not reorder, either)
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    const int row0 = m0 + wm * WTM + i * 32 + lane / LPR;
#pragma unroll
    for (int t = 0; t < 32 / RPI; ++t) {
      const int row = row0 + t * RPI;
      float v[VC];
#pragma unroll
      for (int e = 0; e < VC; e += 4) {
        const uint32_t at = eb + (uint32_t)((t * RPI + lane / LPR) * RS + ((lane % LPR) * VC + e) * 4);
        const f32x4 c4 = *(lds_f4*)(uintptr_t)at;
#pragma unroll
        for (int x = 0; x < 4; ++x) v[e + x] = c4[x] + bv[e + x];
      }
      if (row >= p.M) continue;
      if constexpr (EPI == EPI_RESID) {
        float4* r = reinterpret_cast<float4*>(p.resid + (size_t)row * p.ldr + ecol);
        float4 h = *r;
        h.x += gv[0] * v[0];
        h.y += gv[1] * v[1];
        h.z += gv[2] * v[2];
        h.w += gv[3] * v[3];
        *r = h;
      } else {
        bf16x8 o;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          if constexpr (EPI == EPI_GELU) v[e] = gelu_tanh(v[e]);
          if (ecol + (e & 4) < p.oscale_cols) v[e] *= p.oscale;
          o[e] = (bf16)v[e];
        }
        bf16* dst = reinterpret_cast<bf16*>(p.out) + (size_t)row * p.ldo + ecol;
        if (p.out16) {
          *reinterpret_cast<bf16x8*>(dst) = o;
        } else {                                   // rows aligned to 8 bytes only
          *reinterpret_cast<bf16x4*>(dst) = __builtin_shufflevector(o, o, 0, 1, 2, 3);
          *reinterpret_cast<bf16x4*>(dst + 4) = __builtin_shufflevector(o, o, 4, 5, 6, 7);
        }
      }
    }
  }
}

// Column groups of the XCD tile partition (see k_gemm_f32): the xq (dividing the
// column-tile count) with the least traffic beyond the XCDs' L2s. A is read xq
// times. An XCD's share of W (|W|/xq) is read once where it stays in half of the
// 4 MiB L2, and otherwise again for each of the XCD's rounds of 32 workgroups.
// Over 280 measured calls (512 to 24576 columns, K = 512 to 8192, 512 to 32768
// rows) the pick is 0.2% slower than the best xq in the mean, 4% at worst. A share
// that stays was preferred whatever A cost before, but for K >= 4096 on 256-wide
// tiles, where xq was 1; in us: 8192 x 1024 x 8192 157 -> 118, 32768 x 1024 x 2048
// 169 -> 146, 16384 x 2048 x 2048 149 -> 134, 32768 x 4096 x 4096 1045 -> 997.
inline int choose_xq(int M, int N, int K, int es, int BM, int BN) {
  const int gx = N / BN;
  const double a = (double)M * K * es, w = (double)N * K * es, l2_share = 2.0 * 1024 * 1024;
  const double rounds = std::max(1.0, (double)((M + BM - 1) / BM) * gx / 256.0);
  int best = 1;
  double best_cost = 0.0;
  for (int q = 1; q <= 8; q *= 2) {
    if (gx % q) continue;
    const double cost = a * q + (w / q <= l2_share ? w * (8.0 / q) : 8.0 * rounds * (w / q));
    if (q == 1 || cost < best_cost) {
      best = q;
      best_cost = cost;
    }
  }
  return best;
}

// Tile shapes of the bf16 kernel, by a cost model in us: a fixed cost, per 1024
// of K a fixed cost, a cost per round of 256 workgroups (a partial round costs a
// whole one) and one per 256 workgroups' load, and per round and load the
// epilogue; a least-squares fit to 663 measured calls on MI355X (widths 128 to 8192
// and 24576 columns, K = 64 to 8192, 64 to 65536 rows, every epilogue). Over those
// it picks a tile 0.3% slower than the best in the mean (the four projections of
// widths 512 to 2048: 0.1%), 11% at worst up to 8192 columns and K >= 128; the
// residual epilogue into 24576 columns is the worst, 32% at 1374 rows (its writes,
// which the model takes for a load, take longer in narrow row pieces). A fit
// without the store's load, to widths 512 to 2048 alone, was up to 46% off: 32768
// x 4096 x 64 113 us (77 now), 5496 x 24576 x 1024 residual 589 us (443).
struct TileCost { int bm, bn; double fixed, k, k_round, k_load, round, load_store, load_resid, load_gelu; };
constexpr TileCost kTileCost[] = {
    {256, 256, 1.31, 0.00, 13.73, 10.63, 8.11, 0.00, 14.74, 5.98},
    {256, 128, 0.88, 0.00, 6.98, 6.45, 4.49, 1.30, 8.56, 4.15},
    {128, 128, 0.88, 0.00, 4.59, 3.61, 2.95, 0.00, 3.91, 1.54},
    {64, 128, 1.89, 0.43, 3.61, 1.08, 0.96, 0.11, 1.15, 0.56},
    {64, 64, 1.76, 0.58, 2.48, 0.20, 0.86, 0.00, 0.64, 0.20},
};

inline int choose_tiles(int M, int N, int K, int epi, std::initializer_list<int> among = {0, 1, 2, 3, 4}) {
  int best = -1;
  double best_t = 0.0;
  for (const int c : among) {
    const TileCost& m = kTileCost[c];
    if (N % m.bn) continue;
    const double load = (double)((M + m.bm - 1) / m.bm) * (N / m.bn) / 256.0, rounds = std::ceil(load), k = K / 1024.0;
    const double t = m.fixed + k * (m.k + m.k_round * rounds + m.k_load * load) + m.round * rounds +
                     (epi == EPI_RESID ? m.load_resid : epi == EPI_GELU ? m.load_gelu : m.load_store) * load;
    if (best < 0 || t < best_t) {
      best = c;
      best_t = t;
    }
  }
  return best;
}

// Tile shapes of the f32 kernel (N is a multiple of 128), by the same model without
// the epilogue: a fit to 52 measured calls (128 to 24576 columns, K = 32 to 4096,
// 257 to 32768 rows) that picks a tile 0.4% slower than the best of six in the
// mean, 3% at worst (128 x 128 leads from 9831 x 4096 columns on, by up to 3%; 64 x
// 128 and 128 x 64 nowhere).
struct F32TileCost { int bm, bn; double fixed, k, k_round, k_load, load; };
constexpr F32TileCost kF32TileCost[] = {
    {64, 64, 2.65, 4.97, 15.26, 0.28, 1.01},
    {32, 64, 2.45, 3.40, 8.41, 0.14, 0.55},
    {32, 32, 2.35, 1.56, 4.81, 0.00, 0.27},
};

inline int choose_f32_tiles(int M, int N, int K) {
  int best = 0;
  double best_t = 0.0;
  for (int c = 0; c < 3; ++c) {
    const F32TileCost& m = kF32TileCost[c];
    const double load = (double)((M + m.bm - 1) / m.bm) * (N / m.bn) / 256.0;
    const double t = m.fixed + K / 1024.0 * (m.k + m.k_round * std::ceil(load) + m.k_load * load) + m.load * load;
    if (c == 0 || t < best_t) {
      best = c;
      best_t = t;
    }
  }
  return best;
}

template <int BM, int BN, int WGM, int WGN, int STAGES, int OCC, int EPI, int SITE, bool WIDE = false>
hipError_t launch_dma(const GemmArgs& a0, hipStream_t s) {
  GemmArgs a = a0;
  a.xq = choose_xq(a.M, a.N, a.K, 2, BM, BN);
  if (a.xq < 1 || a.N % BN || (a.N / BN) % a.xq || a.K % 64) return hipErrorInvalidValue;
  launch((k_gemm_dma<BM, BN, WGM, WGN, STAGES, OCC, EPI, SITE, WIDE>), dim3((a.N / BN) * ((a.M + BM - 1) / BM)),
         dim3(64 * WGM * WGN), 0, s, a);
  return hipGetLastError();
}

template <int TM, int TN, int EPI, int SITE>
hipError_t launch_f32(const GemmArgs& a0, hipStream_t s) {
  constexpr int BM = 32 * TM, BN = 32 * TN;
  GemmArgs a = a0;
  a.xq = choose_xq(a.M, a.N, a.K, 4, BM, BN);
  if (a.xq < 1 || a.N % BN || (a.N / BN) % a.xq) return hipErrorInvalidValue;
  launch((k_gemm_f32<TM, TN, EPI, SITE>), dim3((a.N / BN) * ((a.M + BM - 1) / BM)), dim3(256), 0, s, a);
  return hipGetLastError();
}

template <typename T, int EPI, int SITE>
hipError_t launch_t(const GemmArgs& a0, hipStream_t s) {
  GemmArgs a = a0;
  if constexpr (sizeof(T) == 2) {
    a.out16 = a.ldo % 8 == 0 && ((uintptr_t)a.out & 15) == 0;
    // a tile's rows span less than 4 GiB up to this row stride
    if (std::max(a.lda, a.ldw) >= (1 << 22)) {
      // (two of the tiles: 1000 x 4096 x 1024 13.7 us, 20.7 with 64 x 64 alone)
      if constexpr (SITE == SITE_OP) {
        if (choose_tiles(a.M, a.N, a.K, EPI, {2, 4}) == 2)
          return launch_dma<128, 128, 2, 4, 4, 2, EPI, SITE, true>(a, s);
        return launch_dma<64, 64, 2, 2, 4, 2, EPI, SITE, true>(a, s);
      }
      return hipErrorInvalidValue;
    }
    switch (choose_tiles(a.M, a.N, a.K, EPI)) {
      case 0: return launch_dma<256, 256, 2, 4, 2, 2, EPI, SITE>(a, s);
      case 1: return launch_dma<256, 128, 4, 2, 3, 2, EPI, SITE>(a, s);
      case 2: return launch_dma<128, 128, 2, 4, 4, 2, EPI, SITE>(a, s);
      case 3: return launch_dma<64, 128, 2, 4, 3, 4, EPI, SITE>(a, s);
      case 4: return launch_dma<64, 64, 2, 2, 4, 2, EPI, SITE>(a, s);
    }
    return hipErrorInvalidValue;
  } else {
    switch (choose_f32_tiles(a.M, a.N, a.K)) {
      case 0: return launch_f32<2, 2, EPI, SITE>(a, s);
      case 1: return launch_f32<1, 2, EPI, SITE>(a, s);
    }
    return launch_f32<1, 1, EPI, SITE>(a, s);
  }
}

template <typename T>
hipError_t launch_site(int site, int epi, const GemmArgs& a, hipStream_t s) {
  switch (site) {
    case SITE_QKV: return launch_t<T, EPI_STORE, SITE_QKV>(a, s);
    case SITE_Q: return launch_t<T, EPI_STORE, SITE_Q>(a, s);
    case SITE_COND: return launch_t<T, EPI_STORE, SITE_COND>(a, s);
    case SITE_O: return launch_t<T, EPI_RESID, SITE_O>(a, s);
    case SITE_CO: return launch_t<T, EPI_RESID, SITE_CO>(a, s);
    case SITE_FC2: return launch_t<T, EPI_RESID, SITE_FC2>(a, s);
    case SITE_FC1: return launch_t<T, EPI_GELU, SITE_FC1>(a, s);
    default: break;
  }
  switch (epi) {
    case EPI_STORE: return launch_t<T, EPI_STORE, SITE_OP>(a, s);
    case EPI_GELU: return launch_t<T, EPI_GELU, SITE_OP>(a, s);
    case EPI_RESID: return launch_t<T, EPI_RESID, SITE_OP>(a, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_gemm(int site, int dt, int epi, int M, int N, int K, const void* A, int lda, const void* W,
                       int ldw, const float* bias, const float* gate, void* out, int ldo, float* resid, int ldr,
                       hipStream_t s, float oscale, int oscale_cols) {
  if (M == 0) return hipSuccess;
  if (oscale_cols % 4) return hipErrorInvalidValue;
  GemmArgs a{M, N, K, (const char*)A, lda, (const char*)W, ldw, bias, gate, out, ldo, resid, ldr, 1, oscale,
             oscale_cols, false};
  return dt == DT_BF16 ? launch_site<bf16>(site, epi, a, s) : launch_site<float>(site, epi, a, s);
}

}  // namespace f3c
