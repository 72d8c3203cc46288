// bf16 MFMA GEMM for gfx950, 256x128 tiles:  C[M,N] = A[M,K] * W[N,K]^T with fused epilogues; and the choice of the tile for
// every bf16 GEMM (256x256: gemm_phase.hip, smaller tiles: gemm_ring.hip).
//
// Tiling (wave64, v_mfma_f32_32x32x16_bf16): block tile BM x BN with WGM x WGN waves, K staged through LDS in steps of 64.
// Operand roles: the weight rows are the MFMA "A" operand and the token rows the "B" operand,
// i.e. the instruction produces a tile of C^T.  A lane then owns, for one token, quads of
// four consecutive output features, which is what the epilogues want (8-byte bf16 /
// 16-byte fp32 accesses to C, the cache and the residual stream); the tile is re-laid through
// LDS before the epilogue so those accesses are also contiguous across lanes.
// K is walked in order by every tile shape, so an output element is the same fp32 sequence
// regardless of M, of the tile shape and of which rows share the launch.
// Tiles are numbered so that the 8 XCDs (round-robin block dispatch) each work on a
// contiguous range of tiles that share activations in their own L2.
// Operands go global -> LDS directly (global_load_lds_dwordx4: a wave writes 64 consecutive 16-byte chunks at a wave-uniform
// LDS address), no register staging, no LDS stores; unpadded 128-byte LDS rows with an XOR swizzle of the chunk position;
// ring of three stages with one raw barrier per K-step, loads awaited with vmcnt(0) by the waves that issued them.
// Needs K % 64 == 0.

#include <algorithm>
#include <cmath>

#include "gemm_tile.h"

namespace speca {

namespace {

constexpr int BK = 64;

// ---------------------------------------------------------------------------------------------
// Direct-to-LDS main loop.
//
// LDS stage = [BM + BN rows][64 bf16], rows unpadded (128 bytes = 8 chunks of 16 bytes).  Chunk c of
// row r sits at chunk position c ^ swz(r), swz(r) = (r & 7) ^ ((r >> 3) & 1): the 16 lanes that read
// the same chunk index of 16 consecutive rows then touch all 64 banks exactly once.
// Loader: one load instruction fills 8 rows (64 chunks, 1 KiB, contiguous in LDS); lane l supplies
// the chunk stored at position l % 8 of row l / 8, i.e. source chunk (l % 8) ^ swz(row), and the
// hardware places lane l's 16 bytes at the wave-uniform LDS address + 16 l.  A loader wave owns the
// row groups wl, wl + NL, ... (NL loader waves, NL even, so swz depends only on the lane and the
// parity of wl).  Rows beyond M / N are clamped to the last row (never stored).
//
// What keeps a stage intact between its readers and its next loads: a wave waits for its own fragment reads (lgkmcnt(0))
// BEFORE the barrier that hands the stage on.  The barrier builtin alone does not give that: matrix instructions, and with
// them the waits for the fragments they use, are free to sink below it, and a load that hits in L2 then overtakes reads still
// queued at the LDS (a ring compiled that way delivered rows of a later stage, in groups of 32, a few launches per
// step, once four row groups ran side by side and shared the LDS).  The waves form two loader groups: group
// g loads the K-steps of parity g, so at its wait a group has exactly one step outstanding (the one everybody needs next)
// while the other group's step stays in flight.
// Ring discipline per K-step kt:
//   the step's loader waves wait vmcnt(0); barrier (the step is in LDS, everyone is done reading the
//   previous step's stage); the same waves issue step kt + 2 into the stage just freed; compute.
// Rows of the tile staged through LDS per epilogue part: the whole tile when it fits into the ring's
// LDS, else half of it (no LDS beyond the ring: 128x128 stays at 64 KiB, two blocks per CU with room).
constexpr int dlds_epilogue_rows(int BM, int BN, int NS) {
  return BM * (BN + 4) * 4 <= NS * (BM + BN) * BK * 2 ? BM : BM / 2;
}

template <int BM, int BN, int WGM, int WGN, int NS, int MODE>
__global__ __launch_bounds__(WGM* WGN * 64) void gemm_dlds_kernel(const uint16_t* __restrict__ A, int64_t lda,
                                                                   const uint16_t* __restrict__ W, int64_t ldw, int M, int N, int K,
                                                                   int tiles_m, int tiles_n, int group_m, EpiArg<MODE> epi) {
  constexpr int NW = WGM * WGN;
  constexpr int WM = BM / WGM, WN = BN / WGN;
  constexpr int TM = WM / 32, TN = WN / 32;
  static_assert(NS == 3, "ring depth");
  constexpr int NL = NW / 2;                                 // loader waves per K-step
  constexpr int AG = BM / 8 / NL, WG = BN / 8 / NL;          // 8-row groups (one load instruction each) per loader wave
  static_assert(BM / 8 % NL == 0 && BN / 8 % NL == 0 && NL % 2 == 0, "row groups must divide among an even number of loader waves");
  constexpr int STAGE = (BM + BN) * BK;                      // elements per stage
  constexpr int EH = dlds_epilogue_rows(BM, BN, NS);
  extern __shared__ __align__(16) uint16_t smem[];

  int tm, tn;
  if (!tile_coords(tiles_m, tiles_n, group_m, &tm, &tn)) return;
  const int m0 = tm * BM, n0 = tn * BN;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WGN, wn = wave % WGN;
  const int l32 = lane & 31, lhi = lane >> 5;

  floatx16 acc[TN][TM];
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int j = 0; j < TM; ++j)
#pragma unroll
      for (int q = 0; q < 16; ++q) acc[i][j][q] = 0.0f;

  const int nk = K / BK;
  const int grp = wave / NL, wl = wave % NL;                 // loader group and index inside it
  const int lrow = lane >> 3;
  const int lchunk = (lane & 7) ^ lrow ^ (wl & 1);
  const uint16_t* pa[AG];
  const uint16_t* pw[WG];
#pragma unroll
  for (int g = 0; g < AG; ++g) {
    const int row = (wl + g * NL) * 8 + lrow;
    const int m = m0 + row < M ? m0 + row : M - 1;
    pa[g] = A + static_cast<int64_t>(m) * lda + lchunk * 8;
  }
#pragma unroll
  for (int g = 0; g < WG; ++g) {
    const int row = (wl + g * NL) * 8 + lrow;
    const int n = n0 + row < N ? n0 + row : N - 1;
    pw[g] = W + static_cast<int64_t>(n) * ldw + lchunk * 8;
  }
  // reader: row = base + l32 (bases are multiples of 32), chunk 2 ks + lhi
  const int sw = (l32 & 7) ^ ((l32 >> 3) & 1);
  int coff[BK / 16];
#pragma unroll
  for (int ks = 0; ks < BK / 16; ++ks) coff[ks] = ((2 * ks + lhi) ^ sw) * 8;

#define SPECA_LOADS(st, kt_)                                                                                      \
  {                                                                                                               \
    const int k0_ = (kt_) * BK;                                                                                   \
    _Pragma("unroll") for (int g = 0; g < AG; ++g) SPECA_GLL(pa[g] + k0_, smem + (st) * STAGE + (wl + g * NL) * 512);           \
    _Pragma("unroll") for (int g = 0; g < WG; ++g) SPECA_GLL(pw[g] + k0_, smem + (st) * STAGE + BM * BK + (wl + g * NL) * 512); \
  }
#define SPECA_LDFRAG(fa_, fw_, ks_)                                                                               \
  {                                                                                                               \
    _Pragma("unroll") for (int j = 0; j < TM; ++j) fa_[j] = *reinterpret_cast<const bf16x8*>(as + j * 32 * BK + coff[ks_]); \
    _Pragma("unroll") for (int i = 0; i < TN; ++i) fw_[i] = *reinterpret_cast<const bf16x8*>(ws + i * 32 * BK + coff[ks_]); \
  }
#define SPECA_MFMAS(fa_, fw_)                                                                                     \
  {                                                                                                               \
    _Pragma("unroll") for (int i = 0; i < TN; ++i) _Pragma("unroll") for (int j = 0; j < TM; ++j)                 \
      acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fw_[i], fa_[j], acc[i][j], 0, 0, 0);                    \
  }
  // fragments of the next 16-wide K slice are requested before the MFMAs of the current one
#define SPECA_COMPUTE(st)                                                                                         \
  {                                                                                                               \
    const uint16_t* as = smem + (st) * STAGE + (wm * WM + l32) * BK;                                              \
    const uint16_t* ws = smem + (st) * STAGE + BM * BK + (wn * WN + l32) * BK;                                    \
    bf16x8 fa0[TM], fw0[TN], fa1[TM], fw1[TN];                                                                    \
    SPECA_LDFRAG(fa0, fw0, 0);                                                                                    \
    SPECA_LDFRAG(fa1, fw1, 1);                                                                                    \
    SPECA_MFMAS(fa0, fw0);                                                                                        \
    SPECA_LDFRAG(fa0, fw0, 2);                                                                                    \
    SPECA_MFMAS(fa1, fw1);                                                                                        \
    SPECA_LDFRAG(fa1, fw1, 3);                                                                                    \
    SPECA_MFMAS(fa0, fw0);                                                                                        \
    SPECA_MFMAS(fa1, fw1);                                                                                        \
    /* keep that order in the instruction stream: two slices of fragments in flight ahead of the MFMAs */         \
    __builtin_amdgcn_sched_group_barrier(0x100, 2 * (TM + TN), 0);                                                \
    __builtin_amdgcn_sched_group_barrier(0x008, TM * TN, 0);                                                      \
    __builtin_amdgcn_sched_group_barrier(0x100, TM + TN, 0);                                                      \
    __builtin_amdgcn_sched_group_barrier(0x008, TM * TN, 0);                                                      \
    __builtin_amdgcn_sched_group_barrier(0x100, TM + TN, 0);                                                      \
    __builtin_amdgcn_sched_group_barrier(0x008, 2 * TM * TN, 0);                                                  \
  }
  // The same compute with the loads of a later K-step spread between its MFMAs.  Issued in a burst right
  // after the barrier, the loads (a few address instructions each) hold every wave's in-order issue while the
  // matrix cores idle; here loads and MFMAs sit in one scheduling region (no branch: past the last K-step the
  // last tile is re-read into the free stage, never consumed, awaited before the epilogue) and the group
  // barriers ask for the loads one at a time between MFMAs.
  static_assert(AG + WG == 12 && TM == 2 && TN == 2, "three loads per slice of four MFMAs");
#define SPECA_LOADS_BETWEEN_MFMAS                                                                                 \
  {                                                                                                               \
    _Pragma("unroll") for (int l = 0; l < 3; ++l) {                                                               \
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                                                          \
      __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);                                                          \
      __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);                                                          \
    }                                                                                                             \
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                                                            \
  }
#define SPECA_COMPUTE_L(st, new_, ktl_)                                                                           \
  {                                                                                                               \
    const uint16_t* as = smem + (st) * STAGE + (wm * WM + l32) * BK;                                              \
    const uint16_t* ws = smem + (st) * STAGE + BM * BK + (wn * WN + l32) * BK;                                    \
    bf16x8 fa0[TM], fw0[TN], fa1[TM], fw1[TN];                                                                    \
    SPECA_LDFRAG(fa0, fw0, 0);                                                                                    \
    SPECA_LDFRAG(fa1, fw1, 1);                                                                                    \
    SPECA_LOADS(new_, (ktl_) < nk ? (ktl_) : nk - 1);                                                             \
    SPECA_MFMAS(fa0, fw0);                                                                                        \
    SPECA_LDFRAG(fa0, fw0, 2);                                                                                    \
    SPECA_MFMAS(fa1, fw1);                                                                                        \
    SPECA_LDFRAG(fa1, fw1, 3);                                                                                    \
    SPECA_MFMAS(fa0, fw0);                                                                                        \
    SPECA_MFMAS(fa1, fw1);                                                                                        \
    __builtin_amdgcn_sched_group_barrier(0x100, 2 * (TM + TN), 0);                                                \
    SPECA_LOADS_BETWEEN_MFMAS;                                                                                    \
    /* slices 1 and 2: the fragment reads of the slice after next go one per MFMA as well */                      \
    _Pragma("unroll") for (int q = 0; q < 2; ++q) {                                                               \
      _Pragma("unroll") for (int l = 0; l < 3; ++l) {                                                             \
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);                                                        \
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                                                        \
        __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);                                                        \
        __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);                                                        \
      }                                                                                                           \
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);                                                          \
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                                                          \
    }                                                                                                             \
    SPECA_LOADS_BETWEEN_MFMAS;                                                                                    \
  }
  constexpr int WAIT_VM0 = 0x0F70;                           // s_waitcnt vmcnt(0), other counters untouched
  constexpr int WAIT_LDS = 0xC07F;                           // s_waitcnt lgkmcnt(0), other counters untouched
  // prologue: steps 0 .. NS-2, each by its loader waves
#pragma unroll
  for (int s = 0; s < NS - 1; ++s)
    if (s < nk && grp == (s & 1)) SPECA_LOADS(s, s);
  // One K-step with compile-time stage numbers and loader parity (the ring has period NS, the loader
  // groups period 2: the loop body is unrolled over their common period so every LDS address is an
  // immediate offset).
#define SPECA_STEP(kt_, cur_, new_, par_)                                                                         \
  {                                                                                                               \
    const bool mine_ = grp == (par_);                        /* wave-uniform */                                    \
    __builtin_amdgcn_s_waitcnt(WAIT_LDS);                    /* my fragment reads: the next loads may overwrite them */ \
    if (mine_) __builtin_amdgcn_s_waitcnt(WAIT_VM0);         /* my only outstanding loads are those of this step */ \
    asm volatile("" ::: "memory");                                                                                \
    __builtin_amdgcn_s_barrier();                                                                                 \
    asm volatile("" ::: "memory");                                                                                \
    if (mine_) SPECA_COMPUTE_L(cur_, new_, (kt_) + NS - 1)                                                        \
    else SPECA_COMPUTE(cur_)                                                                                      \
  }
  for (int kt = 0; kt < nk; kt += 6) {
    SPECA_STEP(kt, 0, 2, 0);
    if (kt + 1 < nk) SPECA_STEP(kt + 1, 1, 0, 1);
    if (kt + 2 < nk) SPECA_STEP(kt + 2, 2, 1, 0);
    if (kt + 3 < nk) SPECA_STEP(kt + 3, 0, 2, 1);
    if (kt + 4 < nk) SPECA_STEP(kt + 4, 1, 0, 0);
    if (kt + 5 < nk) SPECA_STEP(kt + 5, 2, 1, 1);
  }
#undef SPECA_STEP
  __builtin_amdgcn_s_waitcnt(WAIT_VM0);                      // nothing is outstanding here; kept as a guard before LDS is reused
#undef SPECA_COMPUTE
#undef SPECA_COMPUTE_L
#undef SPECA_LOADS_BETWEEN_MFMAS
#undef SPECA_MFMAS
#undef SPECA_LDFRAG
#undef SPECA_LOADS

  tile_epilogue<BM, BN, WGM, WGN, MODE, EH>(acc, reinterpret_cast<float*>(smem), m0, n0, M, N, epi);
}

template <int BM, int BN, int WGM, int WGN, int NS>
Error launch_dlds(const Operands& o, const GemmEpi& epi, hipStream_t st) {
  const int tiles_m = (o.M + BM - 1) / BM, tiles_n = (o.N + BN - 1) / BN;
  const int64_t nblk = static_cast<int64_t>(tiles_m) * tiles_n;
  if (nblk > 0x7FFFFFF0) SPECA_FAIL(SPECA_EINVAL, "gemm: too many tiles");
  if (o.K % BK != 0 || o.K < BK) SPECA_FAIL(SPECA_EINVAL, "gemm: the large tiles need K %% 64 == 0");
  constexpr int EH = dlds_epilogue_rows(BM, BN, NS);
  const size_t smem_ops = static_cast<size_t>(NS) * (BM + BN) * BK * sizeof(uint16_t);
  const size_t smem_epi = static_cast<size_t>(EH) * (BN + 4) * sizeof(float);
  const size_t smem = smem_ops > smem_epi ? smem_ops : smem_epi;
  dim3 grid(static_cast<unsigned>((nblk + 7) / 8 * 8));
  const int group_m = tiles_m < 4 ? tiles_m : 4;
#define SPECA_LAUNCH(MODE_)                                                                                       \
  case MODE_: {                                                                                                   \
    auto kern = gemm_dlds_kernel<BM, BN, WGM, WGN, NS, MODE_>;                                                    \
    static bool attr_set = false;   /* more than 64 KB of dynamic LDS must be requested once per kernel */          \
    if (smem > 64 * 1024 && !attr_set) {                                                                          \
      SPECA_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(smem))); \
      attr_set = true;                                                                                            \
    }                                                                                                             \
    kern<<<grid, WGM * WGN * 64, smem, st>>>(o.a, o.lda, o.w, o.ldw, o.M, o.N, o.K, tiles_m, tiles_n, group_m, epi_arg<MODE_>(epi)); \
    break;                                                                                                        \
  }
  switch (epi.mode) {
    SPECA_LAUNCH(EPI_STORE)
    SPECA_LAUNCH(EPI_GELU)
    SPECA_LAUNCH(EPI_SILU)
    SPECA_LAUNCH(EPI_F32)
    SPECA_LAUNCH(EPI_BRANCH)
    default: SPECA_FAIL(SPECA_EINVAL, "gemm: epilogue mode %d", epi.mode);
  }
#undef SPECA_LAUNCH
  SPECA_HIP(hipGetLastError());
  return ok();
}

}  // namespace

// ---- tile choice -------------------------------------------------------------------------------------------
// Thirteen kernels can run a given problem; which is fastest depends on how the tile count falls on the chip's compute
// units more than on anything else (a 270-tile launch of one-block-per-CU tiles takes two rounds, a 252-tile one
// takes one), and the row count M varies from call to call: per-sample rejection sends any number of guidance pairs
// to the full pass.  So the choice is made by a small cost model instead of thresholds fitted to particular shapes:
//     time(kernel) = a + (c + b * ceil(K / 64)) * rounds,     depth = ceil(tiles / compute units),
//     rounds = 1 + r * (depth - 1), or with two blocks on a compute unit  floor(depth / 2) * (1 + r) + depth % 2
// a: launch; c: prologue and epilogue; b: one 64-wide K-step; r: what a further round, or the second block, costs.  Fitted to
// 224 problems with cold weights (the layers of 384 to 3072 features at 16 to 8192 rows, and random sizes) so that the time
// of the kernels picked is least (0.9 % above the best kernel of each on the mean) and the times themselves fit (12 % rms).
// The branch epilogue (residual read and written in fp32, cache planes) is two to four times as long as a plain store, the more so
// the fewer waves a tile has for its elements, so c and r have second values for it.  Fitted to the layers of
// 384 to 3072 features inside running models, 256 to 26624 rows, both cache layouts: the time of a block lies 0.1 % above
// that with the best kernels on the mean where the plain constants lay 0.6 % (7 % at worst; 4096 x 1152 x 1152 without plane reads 6.8 us
// above, with them 22.7, 9216 x 3072 x 12288 with them 152).  192x192 and 128x96 are not offered to it: leaving them out costs
// 0.02 %.
// Fitted again since, each time on the kernels that ran then: 256x128 and 128x192 when 256x256 moved to gemm_phase.hip, 256x256
// and the r of 128x192 when its epilogue stored whole lines.  Cold weights, 256 to 27 286 rows: picks among single kernels lie 0.7 % above the
// best one on the mean over 260 layers with K % 64 == 0 (0.9 % before) and 0.8 % over 160 with tails of K (1.1 % before; r = 0.45 had sent
// 8568 x 2304 x 1448 to 128x128 tiles, 83 -> 87.5 us).  The times of long layers on 256x256 come out low (4096 x 3456 x 3072 69 us, modelled 62),
// where no other kind is near.  The branch values of the kinds other than 256x256 are older than the residual requested ahead of the staging
// (gemm_tile.h), which shortens all of them: over 223 branch layers of models with 384 to 1152 features, 1000 to 43 000 rows and both
// layouts the picks cost 0.7 % of a reference step on the mean and 8 % at worst (fc2 of 3840 x 768 x 3072 on 96x128 where 128x64 is best).
struct TileKind {
  int bm, bn;
  float a, c, b, r;    // three in microseconds, a ratio
  float cb, rb;        // c and r under the branch epilogue (cb = 0: not offered to it)
  bool two;            // two blocks fit on a compute unit
  bool whole_steps;    // K % 64 == 0
};
constexpr TileKind kTileKinds[] = {
    {256, 256, 2.4f, 7.8f, 1.07f, 1.15f, 16.5f, 0.95f, false, true},       // 0: phases (gemm_phase.hip)
    {256, 128, 2.4f, 5.66f, 0.791f, 1.17f, 9.5f, 1.00f, false, true},      // 1: large, 3 stages
    {128, 128, 0.8f, 6.40f, 0.535f, 1.00f, 11.39f, 0.98f, false, false},   // 2: ring of 4 stages x 64 columns
    {128, 128, 0.9f, 3.71f, 0.771f, 0.31f, 8.66f, 0.11f, true, false},     // 3: ring of 2 x 64
    {128, 64, 0.8f, 4.18f, 0.314f, 1.08f, 7.46f, 0.98f, false, false},     // 4: ring of 3 x 128
    {128, 64, 2.1f, 1.41f, 0.379f, 0.66f, 5.21f, 0.50f, true, false},      // 5: ring of 3 x 64
    {64, 64, 0.0f, 3.98f, 0.294f, 0.95f, 4.60f, 0.86f, false, false},      // 6: ring of 4 x 128
    {32, 64, 0.0f, 3.67f, 0.266f, 0.98f, 4.61f, 0.77f, false, false},      // 7: ring of 4 x 128, two waves
    {192, 128, 1.3f, 5.69f, 0.656f, 1.15f, 21.68f, 0.85f, false, false},   // 8: ring of 3 x 64
    {128, 192, 0.5f, 5.27f, 0.945f, 0.40f, 14.96f, 0.155f, true, false},    // 9: ring of 2 x 64
    {192, 192, 2.5f, 11.1f, 0.879f, 1.08f, 0.0f, 0.0f, false, false},      // 10: ring of 3 x 64
    {96, 128, 0.0f, 4.72f, 0.435f, 1.07f, 13.07f, 0.84f, false, false},    // 11: ring of 4 x 64
    {128, 96, 1.2f, 3.06f, 0.710f, 0.30f, 0.0f, 0.0f, true, false},        // 12: ring of 2 x 64
};
constexpr int kKinds = sizeof(kTileKinds) / sizeof(kTileKinds[0]);

static int compute_units() {
  static const int n = [] {
    int dev = 0, cu = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cu < 1) {
      (void)hipGetLastError();
      cu = 256;
    }
    return cu;
  }();
  return n;
}

static double tile_cost(const TileKind& t, bool branch, int M, int N, int K) {
  const double tiles = static_cast<double>((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn);
  const double depth = std::ceil(tiles / compute_units());
  const double odd = std::fmod(depth, 2.0);
  const double c = branch ? t.cb : t.c, r = branch ? t.rb : t.r;
  const double rounds = t.two ? (depth - odd) / 2 * (1.0 + r) + odd : 1.0 + r * (depth - 1.0);
  return t.a + (c + t.b * ((K + BK - 1) / BK)) * rounds;
}

// Whether a kind can run the problem.  The rings hold a row's place inside the tile as a 32-bit byte offset, which bounds the
// stride of the rows (11 million elements for the tallest tile); the large tiles hold pointers.
static bool tile_fits(const TileKind& t, const Operands& o) {
  if (t.bn == 256) return gemm_phase_fits(o);
  if (t.whole_steps) return o.K % BK == 0 && o.K >= BK;
  constexpr int64_t kReach = (int64_t{1} << 31) - 128;               // elements, less a row's own 256 bytes
  return (std::min(t.bm, o.M) - 1) * o.lda < kReach && (std::min(t.bn, o.N) - 1) * o.ldw < kReach;
}

// cheapest eligible kernel for the problem (-1: none); *cost receives its modelled time
static int pick_tile(const Operands& o, bool branch, double* cost) {
  int best = -1;
  double bc = 0.0;
  for (int k = 0; k < kKinds; ++k) {
    const TileKind& t = kTileKinds[k];
    if (!tile_fits(t, o) || (branch && t.cb == 0.0f)) continue;
    const double c = tile_cost(t, branch, o.M, o.N, o.K);
    if (best < 0 || c < bc) { best = k; bc = c; }
  }
  *cost = bc;
  return best;
}

static Error launch_kind(int kind, const Operands& o, const GemmEpi& epi, hipStream_t st) {
  switch (kind) {
    case 0: return launch_gemm_phase(o, epi, st);
    case 1: return launch_dlds<256, 128, 4, 2, 3>(o, epi, st);
    default: return launch_gemm_ring(kind - 2, o, epi, st);
  }
}

bool gemm_mfma_supported(const Operands& o) {
  double cost = 0.0;
  return (o.K % 8 == 0) && (o.lda % 8 == 0) && (o.ldw % 8 == 0) && (o.N % 4 == 0) && (reinterpret_cast<uintptr_t>(o.a) % 16 == 0) &&
         (reinterpret_cast<uintptr_t>(o.w) % 16 == 0) && pick_tile(o, true, &cost) >= 0;     // the smallest tile, which fits whenever one does, serves every epilogue
}

// How a layer is run: all of it on one kind, or `head` columns ahead on the 256x256 tile and the rest on `kind`.
struct Choice {
  int kind;
  int head;
  double time;
};
// What a second launch costs beyond the two modelled times, in microseconds.  Over 220 layers that the model would split without it, splits of
// layers under 40 us lost 5 % on the mean (7000 x 3072 x 192 21.2 -> 23.1 us); with it 156 are split, 6 % faster on the mean and one of them
// slower by more than 2 %, and the choice lies 0.1 % above the better form of each on the mean (0.9 % without).
constexpr double kSecondLaunch = 4.0;
static Choice choose(const Operands& o, bool branch) {
  Choice c{-1, 0, 0.0};
  c.kind = pick_tile(o, branch, &c.time);
  // A little more than whole rounds of 256x256 tiles (the 4096 x 4608 x 1152 fc1 GEMM: 288): the columns that make whole
  // rounds go on the large tile, the remaining columns in a second launch (together 47.6 us against 61.8 for the best single
  // kernel, 128x192; 4096 x 9216 x 3072, 576 tiles: 207 -> 181 us).  Column ranges only shift pointers, so this is limited to the epilogues that store into `out`.
  if (!branch && o.M >= 256 && gemm_phase_fits(o)) {
    const int tiles_m = (o.M + 255) / 256;
    for (int rounds = 1;; ++rounds) {
      const int n1 = static_cast<int>(static_cast<int64_t>(rounds) * compute_units() / tiles_m) * 256;
      if (n1 >= o.N) break;
      if (n1 < 256) continue;
      Operands tail = o;
      tail.N = o.N - n1;
      double rest = 0.0;
      const int kind = pick_tile(tail, false, &rest);
      rest += tile_cost(kTileKinds[0], false, o.M, n1, o.K);
      if (c.head ? rest < c.time : rest + kSecondLaunch < 0.96 * c.time) c = {kind, n1, rest};
    }
  }
  return c;
}

double layer_time(bool branch, int M, int N, int K, bool paired) {
  const Operands o{nullptr, K, nullptr, K, M, N, K};
  if (!paired) return choose(o, branch).time;
  double cost = 0.0;
  const int kind = pick_tile(o, branch, &cost);
  if (kind < 0) return cost;
  const TileKind& t = kTileKinds[kind];
  const double tiles = 2.0 * ((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn);
  const double depth = std::max(1.0, tiles / compute_units()), c = branch ? t.cb : t.c, r = branch ? t.rb : t.r;
  const double rounds = t.two && depth >= 2.0 ? depth / 2 * (1.0 + r) : 1.0 + r * (depth - 1.0);
  return t.a + (c + t.b * ((K + BK - 1) / BK)) * rounds;
}

Error launch_gemm_mfma(const Operands& o, const GemmEpi& epi, hipStream_t st) {
  const Choice c = choose(o, epi.mode == EPI_BRANCH);
  if (!c.head) return launch_kind(c.kind, o, epi, st);
  Operands first = o, tail = o;
  first.N = c.head;
  SPECA_TRY(launch_kind(0, first, epi, st));
  GemmEpi te = epi;
  if (epi.bias) te.bias = static_cast<const uint16_t*>(epi.bias) + c.head;
  te.out = epi.mode == EPI_F32 ? static_cast<void*>(static_cast<float*>(epi.out) + c.head) : static_cast<void*>(static_cast<uint16_t*>(epi.out) + c.head);
  tail.w += static_cast<int64_t>(c.head) * o.ldw;
  tail.N = o.N - c.head;
  return launch_kind(c.kind, tail, te, st);
}

}  // namespace speca
