// What the two bf16 GEMM kernels share: types, operand description, tile numbering, the epilogue of a block tile.
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

// gemm_phase.hip: 256 x 256
bool gemm_phase_fits(const Operands& o);
Error launch_gemm_phase(const Operands& o, const GemmEpi& epi, hipStream_t st);

// gemm_ring.hip: kinds 0 .. 10 (see its switch)
Error launch_gemm_ring(int kind, const Operands& o, const GemmEpi& epi, hipStream_t st);

#define SPECA_GLL(src, dst)                                                                                       \
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src),                         \
                                   (__attribute__((address_space(3))) void*)(dst), 16, 0, 0)

// XCD-aware tile id: blocks b, b+8, b+16, ... run on the same XCD; give them neighbouring tiles
// (the grid is rounded up to a multiple of 8; surplus blocks leave at once).  Inside an XCD's
// range tiles are walked in groups of group_m M-panels, N fastest across the group's panels,
// so that the tiles in flight at one time form a compact rectangle and share operand panels
// in that XCD's L2.
__device__ __forceinline__ bool tile_coords(int tiles_m, int tiles_n, int group_m, int* tm, int* tn) {
  const int bid = blockIdx.x;
  const int per_xcd = gridDim.x / 8;
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
  constexpr int WM = BM / WGM, WN = BN / WGN;
  constexpr int TM = WM / 32, TN = WN / 32;
  constexpr int CST = BN + 4;                        // floats per staged row
  constexpr int PARTS = NT % (BN / 4) ? 3 : 1;       // a tile of 192 columns is written 64 columns at a time
  constexpr int QPR = BN / 4 / PARTS;                // quads per row
  constexpr int RPP = NT / QPR;                      // rows per pass
  constexpr int PASSES = EH / RPP;
  static_assert(BM % EH == 0 && EH % WM == 0 && NT % QPR == 0 && EH % RPP == 0, "epilogue shape");
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WGN, wn = wave % WGN;
  const int l32 = lane & 31, lhi = lane >> 5;
  const int qr = tid / QPR;
  float bias_p[PARTS][4] = {};                       // on its way while the tile goes through LDS
#pragma unroll
  for (int part = 0; part < PARTS; ++part) {
    const int n = n0 + (part * QPR + tid % QPR) * 4;
    if (epi.bias && n < N) Store4<bf16_t>::ld(static_cast<const bf16_t*>(epi.bias) + n, bias_p[part]);
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
    if (wm * WM / EH == h) {
#pragma unroll
      for (int j = 0; j < TM; ++j)
#pragma unroll
        for (int i = 0; i < TN; ++i)
#pragma unroll
          for (int jj = 0; jj < 4; ++jj) {
            const int r = wm * WM - h * EH + j * 32 + l32, c = wn * WN + i * 32 + 8 * jj + 4 * lhi;
            *reinterpret_cast<float4*>(Cs + r * CST + c) =
                make_float4(acc[i][j][4 * jj], acc[i][j][4 * jj + 1], acc[i][j][4 * jj + 2], acc[i][j][4 * jj + 3]);
          }
    }
    __syncthreads();
    const int mh = m0 + h * EH;                      // first global row of this part
#pragma unroll
    for (int part = 0; part < PARTS; ++part) {
      const int qc = (part * QPR + tid % QPR) * 4, n = n0 + qc;
      if (n >= N) break;
      const float* bias = bias_p[part];
      if constexpr (MODE == EPI_BRANCH) {
        // batches of EB rows: all loads of the batch are issued before its first store
        // (fewer when the accumulators of a later part are still live: 128 registers for a 64x128 wave tile)
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
