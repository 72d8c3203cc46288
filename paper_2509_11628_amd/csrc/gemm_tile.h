// What the bf16 GEMM kernels share: types, operand description, tile numbering, the epilogue of a block tile.
#pragma once

#include "epilogue.h"
#include "gemm.h"

namespace speca {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

struct Operands {
  const uint16_t* a;
  int64_t lda;
  const uint16_t* w;
  int64_t ldw;
  int M, N, K;
};

// Blocks of a launch of one block (a tile of bm x bn) per compute unit: those of the tiles and, if they leave units idle, one for each of these
// (read_ahead).
unsigned launch_blocks(int bm, int bn, int tiles_m, int tiles_n, const Operands& o, const GemmEpi& epi);

// gemm_phase.hip: 256 x 256
bool gemm_phase_fits(const Operands& o);      // the tiles of gemm_duo.hip, too
Error launch_gemm_phase(const Operands& o, const GemmEpi& epi, hipStream_t st);

// gemm_duo.hip: bm x 128, bm = 64, 128, 192, 256 (what gemm_phase_fits)
Error launch_gemm_duo(int bm, const Operands& o, const GemmEpi& epi, hipStream_t st);

// gemm_ring.hip: kinds 0 .. 8 (its switch; places 2 .. 10 of the table in gemm_mfma.hip)
Error launch_gemm_ring(int kind, const Operands& o, const GemmEpi& epi, hipStream_t st);

#define SPECA_GLL(src, dst)                                                                                       \
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src),                         \
                                   (__attribute__((address_space(3))) void*)(dst), 16, 0, 0)

// Blocks of a launch that hold tiles: a multiple of the 8 XCDs.
__host__ __device__ __forceinline__ int tile_blocks(int tiles_m, int tiles_n) { return (tiles_m * tiles_n + 7) / 8 * 8; }

// Reads of a layer that leaves compute units idle wait for weights: a unit keeps about 50 KB on their way, 94 bytes per ns from the
// memory-side cache and 56 from HBM.  So the idle units read the weights ahead into that cache: blocks behind those of the tiles
// walk W in the order of K, 128 columns of all rows at a time, which they finish long before the tiles reach the last of them.
// Operands alone, 64x64 tiles at 512 x 1152 x 4608: 22.0 us cold, 16.0 with the weights and activations read ahead, 14.5 warm.
__device__ __forceinline__ void read_ahead(const uint16_t* W, int64_t ldw, int N, int K, int part, int parts) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), waves = blockDim.x >> 6, lane = threadIdx.x & 63;
  const int groups = (N + 3) / 4;                            // 4 rows x 256 bytes per instruction
  const int total = groups * ((K + 127) / 128), step = parts * waves;
  constexpr int U = 8;                                       // instructions of a wave on their way
  for (int i = part * waves + wave; i < total; i += U * step) {
    u32x4_t v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int at = i + u * step < total ? i + u * step : total - 1, slab = at / groups, g = at - slab * groups;
      const int row = g * 4 + (lane >> 4) < N ? g * 4 + (lane >> 4) : N - 1, col = slab * 128 + (lane & 15) * 8 < K ? slab * 128 + (lane & 15) * 8 : 0;
      v[u] = *reinterpret_cast<const u32x4_t*>(W + row * ldw + col);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) asm volatile("" : : "v"(v[u]));        // the values are of no use, only their being read
  }
}

// XCD-aware tile id: blocks b, b+8, b+16, ... run on the same XCD; give them neighbouring tiles
// (surplus blocks leave at once).  Inside an XCD's
// range tiles are walked in groups of group_m M-panels, N fastest across the group's panels,
// so that the tiles in flight at one time form a compact rectangle and share operand panels
// in that XCD's L2.
__device__ __forceinline__ bool tile_coords(int tiles_m, int tiles_n, int group_m, int* tm, int* tn) {
  const int bid = blockIdx.x;
  const int per_xcd = tile_blocks(tiles_m, tiles_n) / 8;
  const int tile = (bid % 8) * per_xcd + bid / 8;
  if (tile >= tiles_m * tiles_n) return false;
  const int per_group = group_m * tiles_n;
  const int g = tile / per_group;
  const int first = g * group_m;
  const int h = tiles_m - first < group_m ? tiles_m - first : group_m;
  const int r = tile - g * per_group;
  *tm = first + r % h;
  *tn = r / h;
  return true;
}

// Which quads of a tile are a thread's in the epilogue: row qr + p RPP of a half, column quad part QPR + tid % QPR.
template <int BM, int BN, int NT, int EH>
struct TileQuads {
  static constexpr int PARTS = NT % (BN / 4) ? 3 : 1;       // a tile of 192 columns is written 64 columns at a time
  static constexpr int QPR = BN / 4 / PARTS;                // quads per row
  static constexpr int RPP = NT / QPR;                      // rows per pass
  static constexpr int PASSES = EH / RPP;
  static constexpr int HALVES = BM / EH;
  static_assert(BM % EH == 0 && NT % QPR == 0 && EH % RPP == 0, "epilogue shape");
};

// Branch epilogue without planes to read back (ring layout, order 0, no refresh) of a tile inside one batch row.  What bounds an
// epilogue is its chain of memory round trips: a load behind a store is waited for together with that store.  So the residual
// of the whole tile and the gate are requested at once, ahead of the staging through LDS, and only stores follow (before, 4 batches of
// 4 rows on 256x128 tiles, 16 single rows on 128x128).  16 rows x 256 tokens x 1152 features, 28 blocks, 50 steps 105.4 -> 103.2 ms;
// 2 rows 37.94 -> 37.82, two rows of 845 tokens x 3072 features, 6 blocks, 8 steps 14.60 -> 14.48.  Every tile gains (us per layer inside
// reference steps, 2 to 24 rows): 64x64 0.6 to 3.7, 32x64 1.3 to 2.8, 128x64 2.1 to 10, 96x128 1.3 to 14, 128x128 3.4 to 19, 128x192 6.6 to 21,
// 192x128 1.5 to 17, 256x128 5.8 to 29.  The same loads ahead of the K loop on the small tiles hold the first operands back: 2 rows 37.8 -> 41.6.
template <int BM, int BN, int NT, int EH>
struct BranchAhead {
  using Q = TileQuads<BM, BN, NT, EH>;
  BranchRow<bf16_t> br;
  float gate[Q::PARTS][4], hv[Q::HALVES][Q::PARTS][Q::PASSES][4];

  __device__ __forceinline__ bool load(const GemmEpi& epi, int m0, int n0, int M, int N) {
    const int i_first = m0 / epi.tokens;
    if (i_first != ((m0 + BM < M ? m0 + BM : M) - 1) / epi.tokens) return false;
    br = branch_row<bf16_t>(epi, i_first, m0);
    if (br.order) return false;
    const int tid = threadIdx.x, qr = tid / Q::QPR;
#pragma unroll
    for (int part = 0; part < Q::PARTS; ++part) {
      const int n = n0 + (part * Q::QPR + tid % Q::QPR) * 4;
      if (n < N) Store4<float>::ld(br.gate + n, gate[part]);
    }
#pragma unroll
    for (int h = 0; h < Q::HALVES; ++h)
#pragma unroll
      for (int part = 0; part < Q::PARTS; ++part)
#pragma unroll
        for (int p = 0; p < Q::PASSES; ++p) {
          const int r = h * EH + qr + p * Q::RPP, n = n0 + (part * Q::QPR + tid % Q::QPR) * 4;
          if (n < N && m0 + r < M) Store4<float>::ld(br.h + static_cast<int64_t>(br.t0 + r) * epi.ldh + n, hv[h][part][p]);
        }
    return true;
  }

  // the quad's result v (bias added)
  __device__ __forceinline__ void store(const GemmEpi& epi, int h, int part, int p, int n, const float (&v)[4]) const {
    const int64_t pos = static_cast<int64_t>(br.t0 + h * EH + static_cast<int>(threadIdx.x) / Q::QPR + p * Q::RPP) * epi.ldh + n;
    if (br.refresh) st4_stream(br.d[0] + pos, v);
    float x[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) x[q] = fmaf(gate[part][q], v[q], hv[h][part][p][q]);
    Store4<float>::st(br.h + pos, x);
  }
};

// the tile's rows h EH .. on their way through LDS, by the waves that hold them
template <int BM, int BN, int WGM, int WGN, int EH>
__device__ __forceinline__ void stage_rows(const floatx16 (&acc)[BN / WGN / 32][BM / WGM / 32], float* Cs, int h) {
  constexpr int WM = BM / WGM, WN = BN / WGN;
  static_assert(EH % WM == 0, "epilogue shape");
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave / WGN, wn = wave % WGN, l32 = lane & 31, lhi = lane >> 5;
  if (wm * WM / EH != h) return;
#pragma unroll
  for (int j = 0; j < WM / 32; ++j)
#pragma unroll
    for (int i = 0; i < WN / 32; ++i)
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) {
        const int r = wm * WM - h * EH + j * 32 + l32, c = wn * WN + i * 32 + 8 * jj + 4 * lhi;
        *reinterpret_cast<float4*>(Cs + r * (BN + 4) + c) =
            make_float4(acc[i][j][4 * jj], acc[i][j][4 * jj + 1], acc[i][j][4 * jj + 2], acc[i][j][4 * jj + 3]);
      }
}

// Epilogue of one block tile.  acc[i][j][4*jj + ii] = C[m][n] with m = wm*WM + j*32 + l32,
// n = wn*WN + i*32 + 8*jj + 4*lhi + ii inside the tile.  The tile goes through LDS (fp32, rows padded
// by 16 bytes: conflict-free for the 16-byte writes of 16 consecutive lanes), EH rows at a time, so
// that every global access of the epilogue is a contiguous run along n: a half-wave covers one
// 512-byte (fp32) / 256-byte (bf16) row segment.  Cs must hold EH x (BN + 4) floats; the operand
// buffers it overlays must be dead (all waves past their last read, no load in flight).
template <int BM, int BN, int WGM, int WGN, int MODE, int EH>
__device__ __forceinline__ void tile_epilogue(floatx16 (&acc)[BN / WGN / 32][BM / WGM / 32], float* Cs, int m0, int n0, int M, int N,
                                              const EpiArg<MODE>& epi) {
  constexpr int NT = WGM * WGN * 64;
  using Q = TileQuads<BM, BN, NT, EH>;
  constexpr int CST = BN + 4;                        // floats per staged row
  constexpr int PARTS = Q::PARTS, QPR = Q::QPR, RPP = Q::RPP, PASSES = Q::PASSES;
  const int tid = threadIdx.x;
  const int qr = tid / QPR;
  float bias_p[PARTS][4] = {};                       // on its way while the tile goes through LDS
#pragma unroll
  for (int part = 0; part < PARTS; ++part) {
    const int n = n0 + (part * QPR + tid % QPR) * 4;
    if (epi.bias && n < N) Store4<bf16_t>::ld(static_cast<const bf16_t*>(epi.bias) + n, bias_p[part]);
  }
  if constexpr (MODE == EPI_BRANCH) {
    BranchAhead<BM, BN, NT, EH> ahead;
    if (ahead.load(epi, m0, n0, M, N)) {
      // own LDS accesses done, then a barrier; the loads above stay in flight
      auto turn = [] {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0xC07F);
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
      };
#pragma unroll
      for (int h = 0; h < Q::HALVES; ++h) {
        turn();
        stage_rows<BM, BN, WGM, WGN, EH>(acc, Cs, h);
        turn();
#pragma unroll
        for (int part = 0; part < PARTS; ++part) {
          const int qc = (part * QPR + tid % QPR) * 4;
#pragma unroll
          for (int p = 0; p < PASSES; ++p) {
            const int r = qr + p * RPP;
            if (n0 + qc < N && m0 + h * EH + r < M) {
              const float4 t = *reinterpret_cast<const float4*>(Cs + r * CST + qc);
              const float* bias = bias_p[part];
              const float v[4] = {t.x + bias[0], t.y + bias[1], t.z + bias[2], t.w + bias[3]};
              ahead.store(epi, h, part, p, n0 + qc, v);
            }
          }
        }
      }
      return;
    }
  }
  // block-uniform row table when the whole tile lies inside one batch row: scalar loads
  const int m_last = (m0 + BM < M ? m0 + BM : M) - 1;
  int i_first = 0;
  bool uniform = false;
  BranchRow<bf16_t> br;
  if constexpr (MODE == EPI_BRANCH) {
    i_first = m0 / epi.tokens;
    uniform = i_first == m_last / epi.tokens;
    if (uniform) br = branch_row<bf16_t>(epi, i_first, m0);
  }
#pragma unroll 1
  for (int h = 0; h < BM / EH; ++h) {
    __syncthreads();                                 // operand buffers / previous part consumed
    stage_rows<BM, BN, WGM, WGN, EH>(acc, Cs, h);
    __syncthreads();
    const int mh = m0 + h * EH;                      // first global row of this part
#pragma unroll
    for (int part = 0; part < PARTS; ++part) {
      const int qc = (part * QPR + tid % QPR) * 4, n = n0 + qc;
      if (n >= N) break;
      const float* bias = bias_p[part];
      if constexpr (MODE == EPI_BRANCH) {
        // batches of EB rows: all loads of the batch are issued before its first store
        // (single rows when the accumulators of a later part are still live: pairs take more than the 256 registers that two
        // waves per SIMD have)
        constexpr int EBMAX = (BM / EH > 1) ? 1 : 4;
        constexpr int EB = PASSES % EBMAX == 0 ? EBMAX : (PASSES % 2 == 0 ? 2 : 1);
        if (uniform) {
          float g4[4];
          Store4<float>::ld(br.gate + n, g4);
          for (int p0 = 0; p0 < PASSES; p0 += EB) {
            BranchRegs<bf16_t> regs[EB];
#pragma unroll
            for (int u = 0; u < EB; ++u) {
              const int r = qr + (p0 + u) * RPP;
              if (mh + r < M) branch_load_u<bf16_t>(epi, br, h * EH + r, n, regs[u]);
            }
#pragma unroll
            for (int u = 0; u < EB; ++u) {
              const int r = qr + (p0 + u) * RPP;
              if (mh + r < M) {
                const float4 t = *reinterpret_cast<const float4*>(Cs + r * CST + qc);
                const float v[4] = {t.x + bias[0], t.y + bias[1], t.z + bias[2], t.w + bias[3]};
                branch_finish_u<bf16_t>(epi, br, h * EH + r, n, v, g4, regs[u]);
              }
            }
          }
        } else {
          for (int p0 = 0; p0 < PASSES; p0 += EB) {
            BranchRegs<bf16_t> regs[EB];
#pragma unroll
            for (int u = 0; u < EB; ++u) {
              const int m = mh + qr + (p0 + u) * RPP;
              if (m < M) branch_load<bf16_t>(epi, m, n, regs[u]);
            }
#pragma unroll
            for (int u = 0; u < EB; ++u) {
              const int r = qr + (p0 + u) * RPP;
              const int m = mh + r;
              if (m < M) {
                const float4 t = *reinterpret_cast<const float4*>(Cs + r * CST + qc);
                const float v[4] = {t.x + bias[0], t.y + bias[1], t.z + bias[2], t.w + bias[3]};
                branch_finish<bf16_t>(epi, m, n, v, regs[u]);
              }
            }
          }
        }
      } else {
#pragma unroll 4
        for (int r = qr; r < EH; r += RPP) {
          const int m = mh + r;
          if (m < M) {
            const float4 t = *reinterpret_cast<const float4*>(Cs + r * CST + qc);
            float v[4] = {t.x + bias[0], t.y + bias[1], t.z + bias[2], t.w + bias[3]};
            epilogue_apply<bf16_t, MODE>(epi, m, n, v);
          }
        }
      }
    }
  }
}

}  // namespace speca
