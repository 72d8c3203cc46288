// bf16 MFMA GEMM for gfx950, tiles of 128 columns:  C[M,N] = A[M,K] * W[N,K]^T with fused epilogues, BM x 128 per block, BM = 64, 128,
// 192 or 256.
//
// For layers that 256x256 tiles leave the chip partly empty at.  Eight waves, BM / 4 x 64 each (4 x 2), v_mfma_f32_16x16x32_bf16, with
// the same order of K and the same bits as every other tile.  Operands go global -> LDS directly into a ring of three (BM = 256) or four stages
// of 64 columns.  Waves 0 .. 3 and 4 .. 7, one of each on every SIMD, take turns (ping-pong): while one group reads the fragments of
// a whole K-step and issues its loads, the other runs the matrix instructions of its own.  In the order of the barriers, with
// s the K-step and G0 / G1 the groups:  G0 reads s, G1 multiplies s - 1 | G0 multiplies s, G1 reads s | G0 reads s + 1, ...
//   - free: at its reads of s a wave loads its share of s + NS - 1 into the stage of s - 1.  Both groups read that stage in the two
//     turns before, and a wave waits for its own fragment reads (lgkmcnt(0)) ahead of the barrier that ends them.
//   - landed: ahead of that same barrier a wave waits until its own loads of s + 1 are in LDS (loads complete in issue order: all but
//     the NS - 2 K-steps issued later).  G1's barrier is the one that G0's reads of s + 1 follow.
// The loop without its last K-steps has no branch: with the waits chosen at run time a K-step of 192x128 took 0.60 us, so 0.51.
// What bounds it: the operands, 40 KB per K-step of 192x128 at 89 bytes per ns and unit (0.46 us alone, warm weights; the path gives 150 from
// L2 and 94 from beyond it), beside the matrix instructions (0.37 us alone on random data, 0.33 on zeros: power).
// us with cold weights, best other tile -> this one: 4096 x 1152 x 4608 53.0 -> 43.0 (192x128), 4096 x 1152 x 1152 18.2 -> 15.5,
// 2560 x 3072 x 15360 227 -> 182 (256x128), 768 x 3072 x 12288 97 -> 75 (128x128), 2560 x 1152 x 4608 39.1 -> 32.1.
// The epilogue is that of gemm_phase.hip.  Needs K % 64 == 0 and the tile's operand rows within 4 GB.
#include "lane_epilogue.h"

namespace speca {

namespace {

constexpr int BN = 128, BK = 64;
constexpr int ROW = BK * 2;                    // bytes of a staged row
constexpr int kWaitLds = 0xC07F;               // s_waitcnt lgkmcnt(0)
constexpr int stage_bytes(int BM) { return (BM + BN) * ROW; }
constexpr int stages(int BM) { return 160 * 1024 / stage_bytes(BM) < 4 ? 160 * 1024 / stage_bytes(BM) : 4; }

constexpr int wait_loads(int n) { return (n & 15) | ((n >> 4) << 14) | 0x0F70; }       // s_waitcnt vmcnt(n)

// Wait until all but the last `later` K-steps (of L loads each; uniform) have landed.
template <int L, int MOST>
__device__ __forceinline__ void wait_steps(int later) {
  if (later <= 0) { __builtin_amdgcn_s_waitcnt(wait_loads(0)); return; }
  if constexpr (MOST >= 1) {
    if (later == 1 || MOST == 1) { __builtin_amdgcn_s_waitcnt(wait_loads(L)); return; }
    if constexpr (MOST >= 2) {
      if (later == 2 || MOST == 2) { __builtin_amdgcn_s_waitcnt(wait_loads(2 * L)); return; }
      if constexpr (MOST >= 3) __builtin_amdgcn_s_waitcnt(wait_loads(3 * L));
    }
  }
}

template <int BM, int MODE, bool STREAMS>
__global__ __launch_bounds__(512, 2) void gemm_duo_kernel(const uint16_t* __restrict__ A, int64_t lda, const uint16_t* __restrict__ W,
                                                          int64_t ldw, int M, int N, int K, int tiles_m, int tiles_n, int group_m, EpiArg<MODE> epi,
                                                          StreamArg<STREAMS> streams) {
  constexpr int WM = BM / 4, TM = WM / 16, TN = 4;
  constexpr int NS = stages(BM), STAGE = stage_bytes(BM);
  constexpr int AL = BM / 64, L = AL + BN / 64;              // loads of a wave per K-step: activations, all
  static_assert(BM % 64 == 0 && NS >= 3 && (NS - 1) * L < 64, "row groups divide among the waves");
  extern __shared__ __align__(16) char smem[];               // [NS][A: BM rows, W: 128 rows][64 columns]
  int tm, tn;
  const int held = tile_blocks(tiles_m, tiles_n);
  if (static_cast<int>(blockIdx.x) >= held) {
    const int part = blockIdx.x - held, parts = gridDim.x - held;
    if constexpr (STREAMS) read_ahead(part & 1 ? streams.w2 : W, ldw, N, K, part / 2, (parts + 1 - (part & 1)) / 2);
    else read_ahead(W, ldw, N, K, part, parts);
    return;
  }
  if (!tile_coords(tiles_m, tiles_n, group_m, &tm, &tn)) return;
  const BlockRows<STREAMS> block(streams, W, M, tm, BM);
  const int m0 = block.m0, n0 = tn * BN;
  const int64_t first = block.map.at(m0);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 1, wn = wave & 1, l16 = lane & 15, g4 = lane >> 4;
  const bool second = wave >= 4;               // G1

  floatx4 acc[TN][TM];
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int j = 0; j < TM; ++j) acc[i][j] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};

  // LDS rows and their swizzles are those of gemm_phase.hip; load u of a wave fills the 8 rows of group wave + 8 u
  const int lrow = lane >> 3;
  uint32_t off[L];                             // bytes from the tile's first row
#pragma unroll
  for (int u = 0; u < L; ++u) {
    const int g = wave + 8 * (u < AL ? u : u - AL), r = g * 8 + lrow;
    if (u < AL) off[u] = static_cast<uint32_t>(block.map.at(min(m0 + r, block.map.M - 1)) - first) * static_cast<uint32_t>(lda) * 2 + ((lane & 7) ^ ((r >> 1) & 7)) * 16;
    else off[u] = static_cast<uint32_t>(n0 + r < N ? r : N - 1 - n0) * static_cast<uint32_t>(ldw) * 2 + ((lane & 7) ^ (((r >> 1) & 1) | (((r >> 3) & 3) << 1))) * 16;
  }
  const auto abuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(A) + first * lda, 0, -1, 0x00020000);
  const auto wbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(block.w) + static_cast<int64_t>(n0) * ldw, 0, -1, 0x00020000);
  // this wave's share of K-step s, to the stage at byte `at` (plain variables: the host pass drops the kernel where arguments of the
  // builtin depend on its template parameters)
#define SPECA_LOAD_STEP(s, at)                                                                                     \
  _Pragma("unroll") for (int u = 0; u < L; ++u) {                                                                  \
    char* const dst = smem + (at) + (u < AL ? (wave + 8 * u) * 1024 : BM * ROW + (wave + 8 * (u - AL)) * 1024);    \
    const uint32_t from = off[u];                                                                                  \
    const int col = (s) * ROW;                                                                                     \
    if (u < AL) __builtin_amdgcn_raw_ptr_buffer_load_lds(abuf, (__attribute__((address_space(3))) void*)dst, 16, from, col, 0, 0); \
    else __builtin_amdgcn_raw_ptr_buffer_load_lds(wbuf, (__attribute__((address_space(3))) void*)dst, 16, from, col, 0, 0); \
  }
  const int aswz = l16 >> 1, wswz = ((l16 >> 1) & 1) | ((l16 >> 2) << 1);
  int ard[2], wrd[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    ard[s] = (wm * WM + l16) * ROW + ((4 * s + g4) ^ aswz) * 16;
    wrd[s] = BM * ROW + (wn * 64 + (l16 >> 2) * 8 + (l16 & 3)) * ROW + ((4 * s + g4) ^ wswz) * 16;
  }
  // every memory access stays on its side of a barrier
#define SPECA_BARRIER()                   \
  {                                       \
    asm volatile("" ::: "memory");        \
    __builtin_amdgcn_s_barrier();         \
    asm volatile("" ::: "memory");        \
    __builtin_amdgcn_sched_barrier(0);    \
  }
  const int nk = K / BK;
#pragma unroll
  for (int s = 0; s < NS - 1; ++s)
    if (s < nk) SPECA_LOAD_STEP(s, s * STAGE)
  wait_steps<L, NS - 2>((nk < NS - 1 ? nk : NS - 1) - 1);
  SPECA_BARRIER()
  if (second) SPECA_BARRIER()                  // half a K-step behind from here on
  int here = 0, free_at = (NS - 1) * STAGE;    // the stage of K-step s, and the one of s - 1
  // One K-step: fragments, this wave's loads of K-step s + NS - 1 (`loads`), own loads of s + 1 awaited | matrix instructions |
#define SPECA_K_STEP(loads, landed)                                                                                \
  {                                                                                                                \
    bf16x8 fa[2][TM], fw[2][TN];                                                                                   \
    _Pragma("unroll") for (int q = 0; q < 2; ++q) {                                                                \
      _Pragma("unroll") for (int i = 0; i < TN; ++i)                                                               \
        fw[q][i] = *reinterpret_cast<const bf16x8*>(smem + here + wrd[q] + ((i >> 1) * 32 + (i & 1) * 4) * ROW);   \
      _Pragma("unroll") for (int j = 0; j < TM; ++j) fa[q][j] = *reinterpret_cast<const bf16x8*>(smem + here + ard[q] + j * 16 * ROW); \
    }                                                                                                              \
    if (loads) SPECA_LOAD_STEP(s + NS - 1, free_at)                                                                \
    __builtin_amdgcn_sched_barrier(0);                                                                             \
    landed;                                                                                                        \
    __builtin_amdgcn_s_waitcnt(kWaitLds);                                                                          \
    SPECA_BARRIER()                                                                                                \
    _Pragma("unroll") for (int q = 0; q < 2; ++q) _Pragma("unroll") for (int i = 0; i < TN; ++i)                   \
      _Pragma("unroll") for (int j = 0; j < TM; ++j)                                                               \
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[q][i], fa[q][j], acc[i][j], 0, 0, 0);               \
    __builtin_amdgcn_sched_barrier(0);                                                                             \
    SPECA_BARRIER()                                                                                                \
    free_at = here;                                                                                                \
    here = here + STAGE == NS * STAGE ? 0 : here + STAGE;                                                          \
  }
  int s = 0;
  for (; s + NS - 1 < nk; ++s) SPECA_K_STEP(true, __builtin_amdgcn_s_waitcnt(wait_loads((NS - 2) * L)))
  for (; s < nk; ++s) SPECA_K_STEP(false, (wait_steps<L, NS - 2>(nk - 1 - (s + 1))))
#undef SPECA_K_STEP
  if (!second) SPECA_BARRIER()
#undef SPECA_BARRIER
#undef SPECA_LOAD_STEP
  const void* bias = epi.bias;
  const float* gate = nullptr;
  if constexpr (MODE == EPI_BRANCH) gate = epi.gate;
  if constexpr (STREAMS) {
    if (block.second) { bias = streams.bias2; gate = streams.gate2; }
  }
  lane_epilogue<BM, MODE>(acc, block.map, bias, gate, m0, wm * WM + l16, n0 + wn * 64 + g4 * 8, N, epi);
}

template <int BM, int MODE, bool STREAMS>
Error launch_mode(const Operands& o, const GemmEpi& epi, const StreamArg<STREAMS>& streams, hipStream_t st) {
  const int tiles_m = stream_tiles(streams, o.M, BM), tiles_n = (o.N + BN - 1) / BN;
  const int64_t nblk = static_cast<int64_t>(tiles_m) * tiles_n;
  if (nblk > 0x7FFFFFF0) SPECA_FAIL(SPECA_EINVAL, "gemm: too many tiles");
  auto kern = gemm_duo_kernel<BM, MODE, STREAMS>;
  constexpr int smem = stages(BM) * stage_bytes(BM);
  static bool attr_set = false;   // more than 64 KB of dynamic LDS must be requested once per kernel
  if (!attr_set) {
    SPECA_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, smem));
    attr_set = true;
  }
  kern<<<launch_blocks(BM, BN, tiles_m, tiles_n, o, epi), 512, smem, st>>>(o.a, o.lda, o.w, o.ldw, o.M, o.N, o.K, tiles_m, tiles_n, tiles_m < 4 ? tiles_m : 4,
                                                                     epi_arg<MODE>(epi), streams);
  SPECA_HIP(hipGetLastError());
  return ok();
}

template <int BM>
Error launch_tile(const Operands& o, const GemmEpi& epi, hipStream_t st) {
#define SPECA_LAUNCH(MODE) \
  case MODE: return launch_mode<BM, MODE, false>(o, epi, {}, st);
  switch (epi.mode) {
    SPECA_LAUNCH(EPI_STORE)
    SPECA_LAUNCH(EPI_GELU)
    SPECA_LAUNCH(EPI_SILU)
    SPECA_LAUNCH(EPI_F32)
    SPECA_LAUNCH(EPI_BRANCH)
  }
#undef SPECA_LAUNCH
  SPECA_FAIL(SPECA_EINVAL, "gemm: epilogue mode %d", epi.mode);
}

template <int BM>
Error launch_streams(const Operands& o, const GemmEpi& epi, TwoStreams streams, hipStream_t st) {
  streams.tiles1 = (streams.rows * streams.len1 + BM - 1) / BM;
  switch (epi.mode) {
    case EPI_STORE: return launch_mode<BM, EPI_STORE, true>(o, epi, streams, st);
    case EPI_GELU: return launch_mode<BM, EPI_GELU, true>(o, epi, streams, st);
    case EPI_F32: return launch_mode<BM, EPI_F32, true>(o, epi, streams, st);
    case EPI_BRANCH: return launch_mode<BM, EPI_BRANCH, true>(o, epi, streams, st);
  }
  SPECA_FAIL(SPECA_EINVAL, "gemm: epilogue mode %d of two streams", epi.mode);
}

}  // namespace

Error launch_gemm_duo(int bm, const Operands& o, const GemmEpi& epi, hipStream_t st) {
  if (!gemm_phase_fits(o)) SPECA_FAIL(SPECA_EINVAL, "gemm: K=%d or the row strides do not fit the tiles of 128 columns", o.K);
  switch (bm) {
    case 64: return launch_tile<64>(o, epi, st);
    case 128: return launch_tile<128>(o, epi, st);
    case 192: return launch_tile<192>(o, epi, st);
    case 256: return launch_tile<256>(o, epi, st);
  }
  SPECA_FAIL(SPECA_EINVAL, "gemm: no such tile");
}

Error launch_gemm_duo_streams(int bm, const Operands& o, const GemmEpi& epi, const TwoStreams& streams, hipStream_t st) {
  switch (bm) {
    case 64: return launch_streams<64>(o, epi, streams, st);
    case 128: return launch_streams<128>(o, epi, streams, st);
    case 192: return launch_streams<192>(o, epi, streams, st);
    case 256: return launch_streams<256>(o, epi, streams, st);
  }
  SPECA_FAIL(SPECA_EINVAL, "gemm: no such tile");
}

}  // namespace speca
