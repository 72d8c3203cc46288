// bf16 MFMA GEMM for gfx950, the largest tile:  C[M,N] = A[M,K] * W[N,K]^T with fused epilogues, 256 x 256 per block.
//
// Eight waves, 128 x 64 each (2 x 4), v_mfma_f32_16x16x32_bf16.  Its results have the bits of two chained 32x32x16
// instructions (compared on 600 000 random sums), so a row keeps its bits across the tile kinds, and on random data the chip,
// whose matrix rate is then bound by power, sustains 2131 TFLOP/s of it from registers against 1814 of 32x32x16.
//
// The operands of a K-step (64 columns) are staged in LDS as four halves: A0 / A1, the first / second 64 token rows of both
// wave rows, and W0 / W1, the first / second 32 weight rows of all four wave columns.  A K-step is four phases, each one
// 64 x 32 quadrant of every wave (16 matrix instructions): (A0,W0) (A0,W1) (A1,W1) (A1,W0).  In front of its matrix part a
// phase reads the one half that is new to it, in the order W0(0) A0(0) W1(0) A1(0) W0(1) A0(1) ... (W0(0) ahead of the loop),
// so every phase reads at most eight fragments and issues the two direct-to-LDS loads (per wave) of one later half.
// Waves 4..7 run half a phase behind waves 0..3 (one barrier more ahead of the loop; known as ping-pong): while one wave of a SIMD issues its reads
// and loads the other has the matrix cores.  Two barriers per phase keep the groups in step:  reads, loads | matrix part |.
//
// With c the position of a half in that order, phase p = 1, 2, ... reads c = p and loads c = p + 6, which takes the LDS of
// c = p - 2 (a ring of two K-steps = eight halves):
//   - landed: ahead of the barrier that ends its read part of phase p a wave waits until its own loads of c = p + 1 are in LDS
//     (loads complete in issue order: all but the 5 halves = 10 loads issued later, fewer at the end); every wave of either
//     group passes that barrier before any wave reads c = p + 1.
//   - free: c = p - 2 was read in phase p - 2.  The fragments of a phase are used by its own matrix part, so the reads are
//     complete before the barrier behind it; W0, read in a K-step's last phase and used in the next one, is waited for there.
//     The group behind passes that barrier two barriers before any wave issues the loads of phase p.
// Every load has five phases, 1.6 us, to land, and no wait empties the queue.
// What bounds it: LDS traffic (192 KB read and 64 KB written per K-step, 1.13 us alone) beside the matrix instructions
// (1.02 us alone at the power limit): 1.28 us a K-step where the in-phase loop with one barrier and an empty load queue per
// K-step and 32x32x16 took 1.46.  us with warm weights, that loop -> this one with the epilogue below: 4608 x 3072 x 12288 287 -> 245,
// 4608 x 9216 x 3072 238 -> 206, 4096 x 3456 x 1152 36.2 -> 32.1, 27286 x 9216 x 3072 1327 -> 1138, 8192^3 860 -> 744 (1478 TFLOP/s).
// Without the half-phase offset between the groups: 1012 instead of 1339 TFLOP/s at 4608 x 3072 x 12288.  Four waves of 128 x 128 with
// accumulators in the accumulation file (a quarter less LDS traffic): the same K-step, 2 us more in prologue and epilogue.
//
// Epilogue from registers, without LDS: the weight rows of a pair of 16-row tiles are interleaved in fours, so that a lane
// ends up with eight consecutive features of one token (16 bytes of bf16, 64 bytes per token and instruction).  The two pairs of a
// token are stored one behind the other, so that whole lines of 128 bytes leave together.  All tokens of one pair ahead of the other
// pair's, and 8 bytes per lane where N % 8 == 4, cost up to a third of a short layer (us with cold weights, half lines / whole lines;
// the in-phase loop with its epilogue through LDS): 4096 x 4096 x 128 17.0 / 13.3 (16.0), 4096 x 3456 x 1152 36.2 / 32.6 (36.6),
// 8192 x 8192 x 256 87 / 66 (70), 24808 x 12288 x 448 438 / 347 (370), 4089 x 4092 x 256 24.6 / 17.4 (17.9).  The branch epilogue takes both
// pairs of a token together for the same reason, and needs half as many round trips where it goes token by token (us of a reference
// step of 4 blocks in one row group, planes of differences, one pair at a time / both; in-phase loop): 30 rows x 784 tokens x 1152 features
// 5538 / 5318 (6633), 28 x 1024 x 768 4078 / 4002 (4039), 57 x 256 x 1152 3496 / 3478 (3544); without planes 45 x 400 x 1152 3554 / 3442 (3748).
// Needs K % 64 == 0 and the tile's operand rows within 4 GB.

#include "lane_epilogue.h"

namespace speca {

namespace {

constexpr int BM = 256, BN = 256, WM = 128, WN = 64, BK = 64;
constexpr int ROW = BK * 2;                    // bytes of a staged row
constexpr int STAGE = (BM + BN) * ROW;         // bytes of a K-step
constexpr int TM = WM / 16, TN = WN / 16;
static_assert(TM == 8 && TN == 4, "two halves of tokens, two pairs of feature tiles");

constexpr int kWaitLds = 0xC07F;               // s_waitcnt lgkmcnt(0)
template <int N> __device__ __forceinline__ void wait_loads() { __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0F70); }

template <int MODE, bool STREAMS>
__global__ __launch_bounds__(512, 2) void gemm_phase_kernel(const uint16_t* __restrict__ A, int64_t lda, const uint16_t* __restrict__ W,
                                                            int64_t ldw, int M, int N, int K, int tiles_m, int tiles_n, int group_m, EpiArg<MODE> epi,
                                                            StreamArg<STREAMS> streams) {
  extern __shared__ __align__(16) char smem[];               // [2][A: 256 rows, W: 256 rows][64 columns]
  int tm, tn;
  if (!tile_coords(tiles_m, tiles_n, group_m, &tm, &tn)) return;
  const BlockRows<STREAMS> block(streams, W, M, tm, BM);
  const int m0 = block.m0, n0 = tn * BN;
  const int64_t first = block.map.at(m0);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 2, wn = wave & 3, l16 = lane & 15, g4 = lane >> 4;

  floatx4 acc[TN][TM];
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int j = 0; j < TM; ++j) acc[i][j] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};

  // LDS rows are unpadded (128 bytes, 8 chunks of 16); chunk c of a row sits at position c ^ swz(row).  A 16-byte read takes the lanes
  // {0-3, 12-15, 20-27} at a time, {4-11, 16-19, 28-31}, and the same 32 further on (measured), i.e. all 16 rows of a fragment, half of them
  // at the next chunk; they touch all banks once with swz = (r >> 1) & 7 for token rows r .. r + 15 and
  // ((r >> 1) & 1) | ((r >> 3) & 3) << 1 for weight rows r + {0-3, 8-11, 16-19, 24-27}.  ((r & 7) ^ ((r >> 3) & 1), which is free of conflicts for
  // 16 consecutive lanes, read token rows at 302 bytes per ns and unit instead of 585: 8192^3 711 -> 698 us, 4608 x 9216 x 3072 197.5 -> 193.8.)
  // Loader: one instruction fills 8 rows (1 KiB); lane l supplies the chunk stored at position l % 8 of row l / 8.  A half has 16
  // such groups, wave w loads two.  Rows beyond M / N repeat the last one (never stored).
  const int lrow = lane >> 3;
  uint32_t aoff[2][2], woff[2][2];             // bytes from the tile's first row, [half][load]
  int adst[2][2], wdst[2][2];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int ga = u * 16 + h * 8 + wave, gw = u * 16 + (wave >> 2) * 8 + h * 4 + (wave & 3);
      const int ra = ga * 8 + lrow, rw = gw * 8 + lrow;
      aoff[h][u] = static_cast<uint32_t>(block.map.at(min(m0 + ra, block.map.M - 1)) - first) * static_cast<uint32_t>(lda) * 2 + ((lane & 7) ^ ((ra >> 1) & 7)) * 16;
      woff[h][u] = static_cast<uint32_t>(n0 + rw < N ? rw : N - 1 - n0) * static_cast<uint32_t>(ldw) * 2 +
                   ((lane & 7) ^ (((rw >> 1) & 1) | (((rw >> 3) & 3) << 1))) * 16;
      adst[h][u] = ga * 1024;
      wdst[h][u] = BM * ROW + gw * 1024;
    }
  // Loads through buffer descriptors: the K-step is a scalar offset, and the compiler does not take them for LDS reads that every
  // later fragment would have to wait for.
  const auto abuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(A) + first * lda, 0, -1, 0x00020000);
  const auto wbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(block.w) + static_cast<int64_t>(n0) * ldw, 0, -1, 0x00020000);
#define SPECA_BUFFER_TO_LDS(buf, dst, off, col) \
  __builtin_amdgcn_raw_ptr_buffer_load_lds(buf, (__attribute__((address_space(3))) void*)(dst), 16, off, col, 0, 0)
#define SPECA_LOAD_A(h, st, col)                                                     \
  {                                                                                  \
    SPECA_BUFFER_TO_LDS(abuf, smem + (st) * STAGE + adst[h][0], aoff[h][0], col);    \
    SPECA_BUFFER_TO_LDS(abuf, smem + (st) * STAGE + adst[h][1], aoff[h][1], col);    \
  }
#define SPECA_LOAD_W(h, st, col)                                                     \
  {                                                                                  \
    SPECA_BUFFER_TO_LDS(wbuf, smem + (st) * STAGE + wdst[h][0], woff[h][0], col);    \
    SPECA_BUFFER_TO_LDS(wbuf, smem + (st) * STAGE + wdst[h][1], woff[h][1], col);    \
  }
  // Reader: a fragment is 16 rows x 32 columns, lane l holds chunk 4 s + l / 16 of row l % 16.  Weight tile i of a wave: the rows
  // 32 (i / 2) + 4 (i % 2) + {0-3, 8-11, 16-19, 24-27}, so that the 4 x 2 results of a lane are 8 consecutive features.
  const int aswz = l16 >> 1, wswz = ((l16 >> 1) & 1) | ((l16 >> 2) << 1);
  int ard[2], wrd[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    ard[s] = (wm * WM + l16) * ROW + ((4 * s + g4) ^ aswz) * 16;
    wrd[s] = BM * ROW + (wn * WN + (l16 >> 2) * 8 + (l16 & 3)) * ROW + ((4 * s + g4) ^ wswz) * 16;
  }
  bf16x8 fa[2][TM / 2], fw[2][2][TN / 2];      // [slice][tile]; W halves alternate between two sets
#define SPECA_READ_A(h, st)                                                                                        \
  _Pragma("unroll") for (int s = 0; s < 2; ++s) _Pragma("unroll") for (int j = 0; j < TM / 2; ++j)                 \
    fa[s][j] = *reinterpret_cast<const bf16x8*>(smem + (st) * STAGE + ard[s] + ((h) * (WM / 2) + j * 16) * ROW);
#define SPECA_READ_W(set, h, st)                                                                                   \
  _Pragma("unroll") for (int s = 0; s < 2; ++s) _Pragma("unroll") for (int i = 0; i < TN / 2; ++i)                 \
    fw[set][s][i] = *reinterpret_cast<const bf16x8*>(smem + (st) * STAGE + wrd[s] + ((h) * (WN / 2) + i * 4) * ROW);
  // every memory access stays on its side of a barrier
#define SPECA_BARRIER()                   \
  {                                       \
    asm volatile("" ::: "memory");        \
    __builtin_amdgcn_s_barrier();         \
    asm volatile("" ::: "memory");        \
    __builtin_amdgcn_sched_barrier(0);    \
  }
#define SPECA_MATRIX(ha, hw, set)                                                                                  \
  {                                                                                                                \
    _Pragma("unroll") for (int s = 0; s < 2; ++s) _Pragma("unroll") for (int i = 0; i < TN / 2; ++i)               \
      _Pragma("unroll") for (int j = 0; j < TM / 2; ++j) {                                                         \
        floatx4& c = acc[(hw) * (TN / 2) + i][(ha) * (TM / 2) + j];                                                \
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[set][s][i], fa[s][j], c, 0, 0, 0);                          \
      }                                                                                                            \
    __builtin_amdgcn_sched_barrier(0);                                                                             \
  }
  // End of a read part: the next half has landed (loads that may be outstanding with two or more, one and no K-step to come)
#define SPECA_LANDED(full, two_left, one_left, none_left) \
  {                                                       \
    __builtin_amdgcn_sched_barrier(0);                    \
    if (full || left >= 2) wait_loads<two_left>();        \
    else if (left == 1) wait_loads<one_left>();           \
    else wait_loads<none_left>();                         \
    SPECA_BARRIER()                                       \
  }
  // One K-step in stage c; W0 is in set c, W1 goes to the other one, where the next K-step's W0 follows it
#define SPECA_K_STEP(c, full)                                            \
  {                                                                      \
    SPECA_READ_A(0, c)                                                   \
    if (full || left >= 1) SPECA_LOAD_A(1, 1 - (c), col + ROW)           \
    SPECA_LANDED(full, 10, 10, 2)                                        \
    SPECA_MATRIX(0, 0, c)                                                \
    SPECA_BARRIER()                                                      \
    SPECA_READ_W(1 - (c), 1, c)                                          \
    if (full || left >= 2) SPECA_LOAD_W(0, c, col + 2 * ROW)             \
    SPECA_LANDED(full, 10, 8, 0)                                         \
    SPECA_MATRIX(0, 1, 1 - (c))                                          \
    SPECA_BARRIER()                                                      \
    SPECA_READ_A(1, c)                                                   \
    if (full || left >= 2) SPECA_LOAD_A(0, c, col + 2 * ROW)             \
    SPECA_LANDED(full, 10, 6, 0)                                         \
    SPECA_MATRIX(1, 1, 1 - (c))                                          \
    SPECA_BARRIER()                                                      \
    if (full || left >= 1) { SPECA_READ_W(1 - (c), 0, 1 - (c)) }         \
    if (full || left >= 2) SPECA_LOAD_W(1, c, col + 2 * ROW)             \
    SPECA_LANDED(full, 10, 4, 0)                                         \
    SPECA_MATRIX(1, 0, c)                                                \
    __builtin_amdgcn_s_waitcnt(kWaitLds);                                \
    SPECA_BARRIER()                                                      \
    col += ROW;                                                          \
  }
  const int nk = K / BK;
  SPECA_LOAD_W(0, 0, 0)
  SPECA_LOAD_A(0, 0, 0)
  SPECA_LOAD_W(1, 0, 0)
  SPECA_LOAD_A(1, 0, 0)
  if (nk > 1) {
    SPECA_LOAD_W(0, 1, ROW)
    SPECA_LOAD_A(0, 1, ROW)
    SPECA_LOAD_W(1, 1, ROW)
    wait_loads<12>();                          // W0 has landed
  } else {
    wait_loads<6>();
  }
  SPECA_BARRIER()
  SPECA_READ_W(0, 0, 0)
  __builtin_amdgcn_s_waitcnt(kWaitLds);
  if (nk > 1) wait_loads<10>();                // A0 has landed
  else wait_loads<4>();
  SPECA_BARRIER()
  if (wm) SPECA_BARRIER()                      // half a phase behind from here on
  int col = 0, left = nk - 1;                  // byte column of the K-step, K-steps to come after it
  for (; left >= 3; left -= 2) {
    SPECA_K_STEP(0, true)
    SPECA_K_STEP(1, true)
  }
  for (;; left -= 2) {                         // the last two or three
    SPECA_K_STEP(0, false)
    if (left < 1) break;
    --left;
    SPECA_K_STEP(1, false)
    ++left;
    if (left < 2) break;
  }
  if (!wm) SPECA_BARRIER()
#undef SPECA_K_STEP
#undef SPECA_LANDED
#undef SPECA_MATRIX
#undef SPECA_BARRIER
#undef SPECA_READ_W
#undef SPECA_READ_A
#undef SPECA_LOAD_W
#undef SPECA_LOAD_A
#undef SPECA_BUFFER_TO_LDS
  const void* bias = epi.bias;
  const float* gate = nullptr;
  if constexpr (MODE == EPI_BRANCH) gate = epi.gate;
  if constexpr (STREAMS) {
    if (block.second) { bias = streams.bias2; gate = streams.gate2; }
  }
  lane_epilogue<BM, MODE>(acc, block.map, bias, gate, m0, wm * WM + l16, n0 + wn * WN + g4 * 8, N, epi);
}

template <int MODE, bool STREAMS>
Error launch_mode(const Operands& o, const GemmEpi& epi, const StreamArg<STREAMS>& streams, hipStream_t st) {
  const int tiles_m = stream_tiles(streams, o.M, BM), tiles_n = (o.N + BN - 1) / BN;
  const int64_t nblk = static_cast<int64_t>(tiles_m) * tiles_n;
  if (nblk > 0x7FFFFFF0) SPECA_FAIL(SPECA_EINVAL, "gemm: too many tiles");
  auto kern = gemm_phase_kernel<MODE, STREAMS>;
  static bool attr_set = false;   // more than 64 KB of dynamic LDS must be requested once per kernel
  if (!attr_set) {
    SPECA_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, 2 * STAGE));
    attr_set = true;
  }
  kern<<<tile_blocks(tiles_m, tiles_n), 512, 2 * STAGE, st>>>(o.a, o.lda, o.w, o.ldw, o.M, o.N, o.K, tiles_m, tiles_n, tiles_m < 4 ? tiles_m : 4,
                                                                   epi_arg<MODE>(epi), streams);
  SPECA_HIP(hipGetLastError());
  return ok();
}

}  // namespace

bool gemm_phase_fits(const Operands& o) {
  const int64_t stride = o.lda > o.ldw ? o.lda : o.ldw;
  return o.K % BK == 0 && o.K >= BK && stride < (int64_t{1} << 31) / 256 - o.K;      // 255 rows and a row's own bytes below 2^32
}

Error launch_gemm_phase(const Operands& o, const GemmEpi& epi, hipStream_t st) {
  if (!gemm_phase_fits(o)) SPECA_FAIL(SPECA_EINVAL, "gemm: K=%d or the row strides do not fit the 256x256 tile", o.K);
  switch (epi.mode) {
    case EPI_STORE: return launch_mode<EPI_STORE, false>(o, epi, {}, st);
    case EPI_GELU: return launch_mode<EPI_GELU, false>(o, epi, {}, st);
    case EPI_SILU: return launch_mode<EPI_SILU, false>(o, epi, {}, st);
    case EPI_F32: return launch_mode<EPI_F32, false>(o, epi, {}, st);
    case EPI_BRANCH: return launch_mode<EPI_BRANCH, false>(o, epi, {}, st);
  }
  SPECA_FAIL(SPECA_EINVAL, "gemm: epilogue mode %d", epi.mode);
}

Error launch_gemm_phase_streams(const Operands& o, const GemmEpi& epi, TwoStreams streams, hipStream_t st) {
  streams.tiles1 = (streams.rows * streams.len1 + BM - 1) / BM;
  switch (epi.mode) {
    case EPI_STORE: return launch_mode<EPI_STORE, true>(o, epi, streams, st);
    case EPI_GELU: return launch_mode<EPI_GELU, true>(o, epi, streams, st);
    case EPI_F32: return launch_mode<EPI_F32, true>(o, epi, streams, st);
    case EPI_BRANCH: return launch_mode<EPI_BRANCH, true>(o, epi, streams, st);
  }
  SPECA_FAIL(SPECA_EINVAL, "gemm: epilogue mode %d of two streams", epi.mode);
}

}  // namespace speca
