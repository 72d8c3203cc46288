// bf16 MFMA GEMM for gfx950, small and middle tiles:  C[M,N] = A[M,K] * W[N,K]^T with fused epilogues.
//
// For problems that do not fill the chip with larger tiles, and for tails of K: a block is bound there by what its compute unit can draw
// through the direct-to-LDS path and by its own chain of waits, so the loop keeps several stages of loads in flight and passes few
// barriers.  Wave64, v_mfma_f32_32x32x16_bf16, the same operand roles and the same order of K as the large tiles, hence the same
// bits.  Operands go global -> LDS directly into a ring of NS stages of 64 or 128 columns; rows are unpadded with an XOR swizzle of
// the chunk position, so that the 16 lanes which read one chunk index of 16 rows touch all banks once.  Two loops:
//   several tiles per wave  fragments are read one 32-wide slice ahead of the matrix instructions that use them.  The stage's
//                           only barrier sits before its last slice: by then all its slices are in registers (the stage is
//                           free, the loads of a later one go there) and the next stage has landed.
//   one tile per wave       (STAGE_AHEAD) a slice is too little matrix work to hide an LDS read behind, so the fragments of
//                           the whole next stage are read under the matrix work of the current one; one barrier per stage.
// LW > 0: loads are issued by LW waves of their own.  A wave issues in order, and the direct-to-LDS path takes 1 KB per 10 ns, so a wave that
// loads and computes has its matrix instructions wait for its loads to be taken: 64x64 tiles at 512 x 1152 x 4608 took 0.58 us per
// stage where the loads alone take 0.34 (0.17 the fragments and matrix instructions).  They pass the same barriers and leave after the
// last one.  Tiles of which two blocks share a unit load from the waves that compute (LW = 0): each block covers the other's waits.
// So does 192x192 (hence without read-ahead, which is for launches whose blocks have a unit to themselves in eight waves): its waves take 280
// registers, and beside loader waves they would have 256.  Spilled, it was slower, and moves next to accumulators that assembly uses gave wrong bits;
// 192x128 spills under the branch epilogue alone, behind the last matrix instruction.
// What keeps a stage intact between its readers and its next loads: a wave waits for its own fragment reads (lgkmcnt(0))
// BEFORE the barrier that hands the stage on, and nothing may move across that barrier.  The barrier builtin alone does not give that:
// matrix instructions, and with them the waits for the fragments they use, are free to sink below it, and a load that hits in L2
// then overtakes reads still queued at the LDS.  What lands is awaited by count: loads into LDS complete in the order in which a wave
// issued them, like all its vector loads, and a wave lets those of later stages be.
// us, register-staged tiles of 128x64 to 256x128 -> all waves load and compute -> loader waves (cold weights, read ahead by the idle units,
// gemm_tile.h; warm weights in brackets): 512 x 1152 x 4608 32.6 -> 23.2 -> 18.1 (16.0), 77 x 3072 x 12288 80 -> 46 -> 33 (31), 1536 x 1152 x 4608
// 29 -> 25 (24), 124 x 768 x 3072 14.2 -> 10.5, 16 x 1152 x 3736 23.4 -> 14.8.

#include "gemm_tile.h"

namespace speca {

namespace {

// 16 bytes of zeros: what a lane loads for columns past K
__device__ __align__(16) const uint32_t kZeroChunk[4] = {0u, 0u, 0u, 0u};

// The matrix instructions of the first loop are written as assembly: left to the compiler, the accumulators travel between
// the vector and the accumulation registers in every step (20 to 250 moves).  Up to 6 accumulators stay in vector registers,
// the 9 of a 96x96 wave tile in the accumulation file.  The compiler adds no wait states around assembly: mma_begin fixes the
// zeros in their registers ahead of the loop and mma_end the results behind it, with the states in between written out; an
// accumulator is used again after at least one other instruction of 8 passes, and fragments come from LDS reads that were
// waited for (they must not pass through other registers: few enough of them are live).
template <bool ASM, int TILES>
__device__ __forceinline__ void mma(floatx16& c, bf16x8 a, bf16x8 b) {
  if constexpr (ASM && TILES > 6) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
  else if constexpr (ASM) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "v"(b));
  else c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

template <bool ASM, int TILES>
__device__ __forceinline__ void mma_begin(floatx16& c) {
  if constexpr (ASM && TILES > 6) asm volatile("" : "+a"(c));
  else if constexpr (ASM) asm volatile("" : "+v"(c));
}

// The accumulator as it is from here on, like mma_begin: both only pin its uses to one side (assembly keeps its order).
template <bool ASM, int TILES>
__device__ __forceinline__ void mma_end(floatx16& c) { mma_begin<ASM, TILES>(c); }

constexpr int kWaitLds = 0xC07F;                             // s_waitcnt lgkmcnt(0)
constexpr int wait_loads(int n) { return (n & 15) | ((n >> 4) << 14) | 0x0F70; }       // s_waitcnt vmcnt(n)

// Wait until all but the last `later` stages (of LPW loads each; uniform) have landed.
template <int LPW, int MOST>
__device__ __forceinline__ void wait_stage(int later) {
  if (later <= 0) { __builtin_amdgcn_s_waitcnt(wait_loads(0)); return; }
  if constexpr (MOST >= 1) {
    if (later == 1 || MOST == 1) { __builtin_amdgcn_s_waitcnt(wait_loads(LPW)); return; }
    if constexpr (MOST >= 2) {
      if (later == 2 || MOST == 2) { __builtin_amdgcn_s_waitcnt(wait_loads(2 * LPW)); return; }
      if constexpr (MOST >= 3) {
        if (later == 3 || MOST == 3) { __builtin_amdgcn_s_waitcnt(wait_loads(3 * LPW)); return; }
        if constexpr (MOST >= 4) __builtin_amdgcn_s_waitcnt(wait_loads(4 * LPW));
      }
    }
  }
}

// Rows of the tile staged through LDS per epilogue part: the whole tile when it fits into the ring, else half of it.
constexpr int epilogue_rows(int BM, int BN, int ring) { return BM * (BN + 4) * 4 <= ring ? BM : BM / 2; }
constexpr int ring_bytes(int BM, int BN, int NS, int KS) { return NS * (BM + BN) * KS * 64; }
constexpr size_t lds_bytes(int BM, int BN, int NS, int KS) {
  const int ring = ring_bytes(BM, BN, NS, KS), epi = epilogue_rows(BM, BN, ring) * (BN + 4) * 4;
  return ring > epi ? ring : epi;
}

// LW: waves that only load (0: all waves load and compute).  KTAIL: K is no multiple of a stage.
template <int BM, int BN, int WGM, int WGN, int NS, int KS, bool STAGE_AHEAD, int LW, int MODE, bool KTAIL>
__global__ __launch_bounds__((WGM* WGN + LW) * 64) void gemm_ring_kernel(const uint16_t* __restrict__ A, int64_t lda,
                                                        const uint16_t* __restrict__ W, int64_t ldw, int M, int N, int K, int tiles_m, int tiles_n,
                                                        int group_m, EpiArg<MODE> epi) {
  constexpr int NW = WGM * WGN;
  static_assert((NW == 1 || NW == 2 || NW == 4) && (KS == 2 || KS == 4) && NS >= 2 && NS <= 6, "up to four waves, stages of 64 or 128 columns");
  constexpr int WM = BM / WGM, WN = BN / WGN;
  constexpr int TM = WM / 32, TN = WN / 32;
  static_assert(STAGE_AHEAD || TM * TN >= 2, "an accumulator must not be used twice in a row");
  constexpr int COLS = 32 * KS;                              // columns of a stage
  constexpr int ROW = COLS * 2;                              // bytes of a stage row
  constexpr int CPR = 4 * KS;                                // 16-byte chunks per row
  constexpr int GR = 64 / CPR;                               // rows per load instruction (1 KiB)
  constexpr int LD = LW ? LW : NW;                           // waves that load
  constexpr int AL = BM / GR / LD, WL = BN / GR / LD, LPW = AL + WL;                 // their loads per stage
  static_assert(BM % (LD * GR) == 0 && BN % (LD * GR) == 0, "row groups must divide among the waves");
  static_assert((NS - 1) * LPW < 64, "outstanding loads of a wave");
  constexpr int STAGE = (BM + BN) * ROW;                     // bytes
  constexpr int EH = epilogue_rows(BM, BN, NS * STAGE);
  extern __shared__ __align__(16) char smem[];

  int tm, tn;
  const int held = tile_blocks(tiles_m, tiles_n);
  if (static_cast<int>(blockIdx.x) >= held) {
    read_ahead(W, ldw, N, K, blockIdx.x - held, gridDim.x - held);
    return;
  }
  if (!tile_coords(tiles_m, tiles_n, group_m, &tm, &tn)) return;
  const int m0 = tm * BM, n0 = tn * BN;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lwave = LW ? wave - NW : wave;                   // loader (negative: none)
  const int wm = wave / WGN, wn = wave % WGN;
  const int l32 = lane & 31, lhi = lane >> 5;

  floatx16 acc[TN][TM];
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int j = 0; j < TM; ++j) {
#pragma unroll
      for (int q = 0; q < 16; ++q) acc[i][j][q] = 0.0f;
      mma_begin<!STAGE_AHEAD, TM * TN>(acc[i][j]);
    }
  asm volatile("s_nop 7" ::: "memory");                      // vector writes to matrix reads

  const int nk = (K + COLS - 1) / COLS;
  // Loader: group g of a stage is rows GR g .. GR g + GR - 1, loaded by loader g % LD; lane l supplies the chunk stored at
  // position l % CPR of row l / CPR, i.e. source chunk (l % CPR) ^ swz(row).  With 128-byte rows swz(row) is
  // (row & 7) ^ ((row >> 3) & 1), with 256-byte rows row & 15.  Byte offsets from the tile's first row; rows beyond M / N
  // repeat the last one (never stored).
  const int lrow = lane / CPR;
  auto chunk = [&](int g) { return (lane % CPR) ^ (KS == 2 ? lrow ^ (g & 1) : (g & 3) * 4 + lrow); };
  const char* ba = reinterpret_cast<const char*>(A + static_cast<int64_t>(m0) * lda);
  const char* bw = reinterpret_cast<const char*>(W + static_cast<int64_t>(n0) * ldw);
  uint32_t voff[LPW];
#pragma unroll
  for (int u = 0; u < LPW; ++u) {
    if (u < AL) {
      const int g = lwave + LD * u, r = g * GR + lrow;
      voff[u] = static_cast<uint32_t>(static_cast<int64_t>(m0 + r < M ? r : M - 1 - m0) * lda * 2 + chunk(g) * 16);
    } else {
      const int g = lwave + LD * (u - AL), r = g * GR + lrow;
      voff[u] = static_cast<uint32_t>(static_cast<int64_t>(n0 + r < N ? r : N - 1 - n0) * ldw * 2 + chunk(g) * 16);
    }
  }
  auto load_one = [&](int s, int slot, int u) {              // load u of this wave's share of stage s
    const bool is_a = u < AL;
    const int g = lwave + LD * (is_a ? u : u - AL);
    const char* src = (is_a ? ba : bw) + static_cast<int64_t>(s) * ROW + voff[u];
    if (KTAIL && s == nk - 1) src = s * COLS + chunk(g) * 8 < K ? src : reinterpret_cast<const char*>(kZeroChunk);
    SPECA_GLL(src, smem + slot * STAGE + (is_a ? 0 : BM * ROW) + g * 1024);
  };
  // Reader: row = base + l32 (bases are multiples of 32), chunk 2 (16-wide piece) + lhi; a slice is two pieces
  const int sw = KS == 2 ? (l32 & 7) ^ ((l32 >> 3) & 1) : l32 & 15;
  int coff[2 * KS];
#pragma unroll
  for (int q = 0; q < 2 * KS; ++q) coff[q] = ((2 * q + lhi) ^ sw) * 16;
  const int ra = (wm * WM + l32) * ROW, rw = BM * ROW + (wn * WN + l32) * ROW;
  constexpr int SETS = STAGE_AHEAD ? 2 * KS : 2;
  bf16x8 fa[SETS][2][TM], fw[SETS][2][TN];
  auto read_a = [&](int set, int slot, int slice, int p, int j) {
    fa[set][p][j] = *reinterpret_cast<const bf16x8*>(smem + slot * STAGE + ra + coff[2 * slice + p] + j * 32 * ROW);
  };
  auto read_w = [&](int set, int slot, int slice, int p, int i) {
    fw[set][p][i] = *reinterpret_cast<const bf16x8*>(smem + slot * STAGE + rw + coff[2 * slice + p] + i * 32 * ROW);
  };
  auto read_slice = [&](int set, int slot, int slice) {
#pragma unroll
    for (int p = 0; p < 2; ++p) {
#pragma unroll
      for (int i = 0; i < TN; ++i) read_w(set, slot, slice, p, i);
#pragma unroll
      for (int j = 0; j < TM; ++j) read_a(set, slot, slice, p, j);
    }
  };
#define SPECA_PIN() __builtin_amdgcn_sched_barrier(0)
  // every memory access stays on its side of a barrier
#define SPECA_BARRIER()             \
  {                                 \
    asm volatile("" ::: "memory");  \
    __builtin_amdgcn_s_barrier();   \
    asm volatile("" ::: "memory");  \
    SPECA_PIN();                    \
  }
  if constexpr (LW > 0) {
    if (wave >= NW) {
#pragma unroll
      for (int s = 0; s < NS; ++s)
        if (s < nk) {
#pragma unroll
          for (int u = 0; u < LPW; ++u) load_one(s, s, u);
        }
      wait_stage<LPW, NS - 1>((nk < NS ? nk : NS) - 1);
      SPECA_BARRIER();
      int slot = 0;
      if constexpr (STAGE_AHEAD) {
        wait_stage<LPW, NS - 2>((nk < NS ? nk : NS) - 2);
        SPECA_BARRIER();
        for (int s = 0; s < nk; ++s) {
          if (s + NS < nk) {
#pragma unroll
            for (int u = 0; u < LPW; ++u) load_one(s + NS, slot, u);
          }
          SPECA_PIN();
          wait_stage<LPW, NS - 2>((nk - 1 < s + NS ? nk - 1 : s + NS) - (s + 2));
          SPECA_BARRIER();
          slot = slot + 1 == NS ? 0 : slot + 1;
        }
      } else {
        for (int s = 0; s < nk; ++s) {
          wait_stage<LPW, NS - 2>((nk < s + NS ? nk : s + NS) - (s + 2));
          SPECA_BARRIER();
          if (s + NS < nk) {
#pragma unroll
            for (int u = 0; u < LPW; ++u) load_one(s + NS, slot, u);
          }
          SPECA_PIN();
          slot = slot + 1 == NS ? 0 : slot + 1;
        }
      }
      return;
    }
  }
  // prologue: stages 0 .. NS-1, the first one awaited
#pragma unroll
  for (int s = 0; s < NS; ++s)
    if (!LW && s < nk) {
#pragma unroll
      for (int u = 0; u < LPW; ++u) load_one(s, s, u);
    }
  if (!LW) wait_stage<LPW, NS - 1>((nk < NS ? nk : NS) - 1);
  SPECA_BARRIER();
  int slot = 0;
  if constexpr (STAGE_AHEAD) {
#pragma unroll
    for (int q = 0; q < KS; ++q) read_slice(q, 0, q);
    __builtin_amdgcn_s_waitcnt(kWaitLds);                    // stage 0 is in registers
    if (!LW) wait_stage<LPW, NS - 2>((nk < NS ? nk : NS) - 2);  // stage 1 has landed
    SPECA_BARRIER();
    // Iteration s: stage s is in registers (set `cur`), its slot is free, stage s + 1 has landed
#define SPECA_STAGE(s, cur)                                                                                       \
  {                                                                                                               \
    const int next = slot + 1 == NS ? 0 : slot + 1;                                                               \
    if ((s) + 1 < nk) {                                                                                           \
      _Pragma("unroll") for (int q = 0; q < KS; ++q) read_slice((1 - (cur)) * KS + q, next, q);                   \
    }                                                                                                             \
    if (!LW && (s) + NS < nk) {                                                                                   \
      _Pragma("unroll") for (int u = 0; u < LPW; ++u) load_one((s) + NS, slot, u);                                \
    }                                                                                                             \
    SPECA_PIN();                                                                                                  \
    _Pragma("unroll") for (int q = 0; q < 2 * KS; ++q)                                                            \
      _Pragma("unroll") for (int i = 0; i < TN; ++i)                                                              \
        _Pragma("unroll") for (int j = 0; j < TM; ++j)                                                            \
          mma<!STAGE_AHEAD, TM * TN>(acc[i][j], fw[(cur) * KS + q / 2][q & 1][i], fa[(cur) * KS + q / 2][q & 1][j]);            \
    SPECA_PIN();                                                                                                  \
    __builtin_amdgcn_s_waitcnt(kWaitLds);                     /* stage s + 1 is in registers: its slot is free */   \
    if (!LW) wait_stage<LPW, NS - 2>((nk - 1 < (s) + NS ? nk - 1 : (s) + NS) - ((s) + 2));         /* stage s + 2 has landed */ \
    SPECA_BARRIER();                                                                                              \
    slot = next;                                                                                                  \
  }
    for (int s = 0; s < nk; s += 2) {
      SPECA_STAGE(s, 0);
      if (s + 1 >= nk) break;
      SPECA_STAGE(s + 1, 1);
    }
#undef SPECA_STAGE
  } else {
    read_slice(0, 0, 0);
    SPECA_PIN();
  // Matrix work of the slice in set `cur`, with the reads of another slice and a share of a stage's loads in front of each row of it
#define SPECA_SLICE(cur, reads, slot_r, slice_r, loads, s_l, slot_l)                                               \
  _Pragma("unroll") for (int t = 0; t < 2 * TN; ++t) {                                                            \
    if (reads) {                                                                                                  \
      read_w(1 - (cur), slot_r, slice_r, t / TN, t % TN);                                                         \
      _Pragma("unroll") for (int v = t * TM / TN; v < (t + 1) * TM / TN; ++v) read_a(1 - (cur), slot_r, slice_r, v / TM, v % TM); \
    }                                                                                                             \
    if (loads) {                                                                                                  \
      _Pragma("unroll") for (int u = t * LPW / (2 * TN); u < (t + 1) * LPW / (2 * TN); ++u) load_one(s_l, slot_l, u); \
    }                                                                                                             \
    SPECA_PIN();                                                                                                  \
    _Pragma("unroll") for (int j = 0; j < TM; ++j) mma<!STAGE_AHEAD, TM * TN>(acc[t % TN][j], fw[cur][t / TN][t % TN], fa[cur][t / TN][j]); \
    SPECA_PIN();                                                                                                  \
  }
    for (int s = 0; s < nk; ++s) {
      const int next = slot + 1 == NS ? 0 : slot + 1;
#pragma unroll
      for (int q = 0; q + 1 < KS; ++q) {
        __builtin_amdgcn_s_waitcnt(kWaitLds);                // slice q is in registers
        SPECA_PIN();
        SPECA_SLICE(q & 1, true, slot, q + 1, false, 0, 0)
      }
      __builtin_amdgcn_s_waitcnt(kWaitLds);                  // the last slice too: the stage's LDS is free
      if (!LW) wait_stage<LPW, NS - 2>((nk < s + NS ? nk : s + NS) - (s + 2));       // stage s + 1 has landed (later ones: up to s + NS - 1)
      SPECA_BARRIER();
      SPECA_SLICE((KS - 1) & 1, s + 1 < nk, next, 0, !LW && s + NS < nk, s + NS, slot)
      slot = next;
    }
#undef SPECA_SLICE
  }
#undef SPECA_BARRIER
#undef SPECA_PIN
  __builtin_amdgcn_s_waitcnt(wait_loads(0));                 // nothing is outstanding here; kept as a guard before LDS is reused
  if (!STAGE_AHEAD) {
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");       // matrix results to vector reads: 18 wait states at most
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
      for (int j = 0; j < TM; ++j) mma_end<!STAGE_AHEAD, TM * TN>(acc[i][j]);      // no read of an accumulator moves ahead of the wait
  }
  tile_epilogue<BM, BN, WGM, WGN, MODE, EH>(acc, reinterpret_cast<float*>(smem), m0, n0, M, N, epi);
}

template <int BM, int BN, int WGM, int WGN, int NS, int KS, bool SA, int LW, int MODE, bool KTAIL>
Error launch_mode(const Operands& o, const GemmEpi& epi, hipStream_t st) {
  const int tiles_m = (o.M + BM - 1) / BM, tiles_n = (o.N + BN - 1) / BN;
  const int64_t nblk = static_cast<int64_t>(tiles_m) * tiles_n;
  if (nblk > 0x7FFFFFF0) SPECA_FAIL(SPECA_EINVAL, "gemm: too many tiles");
  constexpr size_t smem = lds_bytes(BM, BN, NS, KS);
  auto kern = gemm_ring_kernel<BM, BN, WGM, WGN, NS, KS, SA, LW, MODE, KTAIL>;
  static bool attr_set = false;   // more than 64 KB of dynamic LDS must be requested once per kernel
  if (smem > 64 * 1024 && !attr_set) {
    SPECA_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(smem)));
    attr_set = true;
  }
  const int group_m = tiles_m < 4 ? tiles_m : 4;
  kern<<<LW ? launch_blocks(BM, BN, tiles_m, tiles_n, o, epi) : tile_blocks(tiles_m, tiles_n), (WGM * WGN + LW) * 64, smem, st>>>(o.a, o.lda, o.w, o.ldw, o.M, o.N, o.K, tiles_m, tiles_n, group_m,
                                                                    epi_arg<MODE>(epi));
  SPECA_HIP(hipGetLastError());
  return ok();
}

// BRANCH: the tile is offered to the branch epilogue (see the table in gemm_mfma.hip).
template <int BM, int BN, int WGM, int WGN, int NS, int KS, bool SA, bool BRANCH, int LW>
Error launch_tile(const Operands& o, const GemmEpi& epi, hipStream_t st) {
#define SPECA_LAUNCH(MODE_)                                                                                  \
  return o.K % (32 * KS) ? launch_mode<BM, BN, WGM, WGN, NS, KS, SA, LW, MODE_, true>(o, epi, st)                \
                         : launch_mode<BM, BN, WGM, WGN, NS, KS, SA, LW, MODE_, false>(o, epi, st);
  switch (epi.mode) {
    case EPI_STORE: SPECA_LAUNCH(EPI_STORE)
    case EPI_GELU: SPECA_LAUNCH(EPI_GELU)
    case EPI_SILU: SPECA_LAUNCH(EPI_SILU)
    case EPI_F32: SPECA_LAUNCH(EPI_F32)
    case EPI_BRANCH:
      if constexpr (BRANCH) { SPECA_LAUNCH(EPI_BRANCH) }
      break;
  }
#undef SPECA_LAUNCH
  SPECA_FAIL(SPECA_EINVAL, "gemm: epilogue mode %d on a %d x %d tile", epi.mode, BM, BN);
}

}  // namespace

Error launch_gemm_ring(int kind, const Operands& o, const GemmEpi& epi, hipStream_t st) {
  switch (kind) {
    case 0: return launch_tile<128, 128, 2, 2, 4, 2, false, true, 4>(o, epi, st);
    case 1: return launch_tile<128, 128, 2, 2, 2, 2, false, true, 0>(o, epi, st);
    case 2: return launch_tile<128, 64, 2, 2, 3, 4, false, true, 4>(o, epi, st);
    case 3: return launch_tile<64, 64, 2, 2, 3, 4, true, true, 4>(o, epi, st);
    case 4: return launch_tile<32, 64, 1, 2, 4, 4, true, true, 2>(o, epi, st);
    case 5: return launch_tile<192, 128, 2, 2, 3, 2, false, true, 4>(o, epi, st);
    case 6: return launch_tile<128, 192, 2, 2, 2, 2, false, true, 0>(o, epi, st);
    case 7: return launch_tile<192, 192, 2, 2, 3, 2, false, false, 0>(o, epi, st);
    case 8: return launch_tile<96, 128, 1, 4, 4, 2, false, true, 4>(o, epi, st);
  }
  SPECA_FAIL(SPECA_EINVAL, "gemm: no such tile");
}

}  // namespace speca
