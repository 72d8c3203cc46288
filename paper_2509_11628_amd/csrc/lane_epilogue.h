// What the tiles that compute with 16x16x32 matrix instructions share (gemm_phase.hip, gemm_duo.hip): the rows of a launch, and the epilogue from
// registers.  A wave owns 64 features, whose weight rows are interleaved in fours per pair of 16-row tiles, so that a lane holds eight
// consecutive features of one token in each of two pairs, 32 features apart.
#pragma once

#include <type_traits>

#include "gemm_tile.h"

namespace speca {

typedef float floatx4 __attribute__((ext_vector_type(4)));

// The rows of a launch.  Plain: M of them, one behind the other.  Streams: the tokens of every batch row are split into two ranges with weights
// of their own (image and text of a dual-stream block); a tile holds rows of one of them, numbered over the batch, and row v of a
// stream lies at (v / len) tokens + off + v % len.
template <bool STREAMS> struct RowMap;
template <> struct RowMap<false> {
  int M;
  __device__ __forceinline__ int64_t at(int v) const { return v; }
};
template <> struct RowMap<true> {
  int M, len, off, tokens;
  __device__ __forceinline__ int64_t at(int v) const {
    const int i = v / len;
    return static_cast<int64_t>(i) * tokens + off + (v - i * len);
  }
};

// The two streams of a launch: tiles [0, tiles1) of the M direction are rows of the first one.
struct TwoStreams {
  const uint16_t* w2;
  const void* bias2;
  const float* gate2;
  int tiles1, rows, tokens;      // batch rows; tokens of each
  int len1, off1, len2, off2;
};
struct OneStream {};
template <bool STREAMS> using StreamArg = std::conditional_t<STREAMS, TwoStreams, OneStream>;

// tiles of a launch in the M direction
inline int stream_tiles(const OneStream&, int M, int bm) { return (M + bm - 1) / bm; }
inline int stream_tiles(const TwoStreams& s, int, int bm) { return (s.rows * s.len1 + bm - 1) / bm + (s.rows * s.len2 + bm - 1) / bm; }

// What a block works on: its rows, its first one among them, its weights.
template <bool STREAMS>
struct BlockRows {
  RowMap<STREAMS> map;
  int m0;
  const uint16_t* w;
  bool second;

  __device__ __forceinline__ BlockRows(const StreamArg<STREAMS>& s, const uint16_t* W, int M, int tm, int bm) {
    if constexpr (STREAMS) {
      second = tm >= s.tiles1;
      m0 = (second ? tm - s.tiles1 : tm) * bm;
      w = second ? s.w2 : W;
      const int len = second ? s.len2 : s.len1;
      map = {s.rows * len, len, second ? s.off2 : s.off1, s.tokens};
    } else {
      second = false;
      m0 = tm * bm;
      w = W;
      map = {M};
    }
  }
};

// Eight consecutive features of a token (`two`: only the first four exist otherwise).  Rows start at multiples of four features, so
// 16 bytes may lie at 8-byte alignment, which global stores allow.
typedef u32x4_t __attribute__((aligned(8))) u32x4_a8;
__device__ __forceinline__ u32x4_t pack8(const float* v) {
  return u32x4_t{pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]), pack_bf16(v[4], v[5]), pack_bf16(v[6], v[7])};
}
__device__ __forceinline__ void st8(bf16_t* p, const float* v, bool two) {
  if (two) *reinterpret_cast<u32x4_a8*>(p) = pack8(v);
  else Store4<bf16_t>::st(p, v);
}
__device__ __forceinline__ void st8(float* p, const float* v, bool two) {
  Store4<float>::st(p, v);
  if (two) Store4<float>::st(p + 4, v + 4);
}
__device__ __forceinline__ void st8_stream(bf16_t* p, const float* v, bool two, bool wide) {
  if (wide && two) {
    __builtin_nontemporal_store(pack8(v), reinterpret_cast<u32x4_t*>(p));
  } else {
    st4_stream(p, v);
    if (two) st4_stream(p + 4, v + 4);
  }
}

// The lane's token j, its eight features of pair P of the tiles (bias added)
template <int TM>
__device__ __forceinline__ void lane_values(const floatx4 (&acc)[4][TM], int j, int P, float (&v)[8]) {
#pragma unroll
  for (int q = 0; q < 8; ++q) v[q] = acc[2 * P + q / 4][j][q % 4];
}

// Eight values of features n .. n + 7; past N, a multiple of 4, the last four again (never used, whatever the lane they belong to has
// stored by then), so that no branch parts the loads
template <typename T>
__device__ __forceinline__ void ld8(const T* p, int n, int N, float (&v)[8]) {
  Store4<T>::ld(p + min(n, N - 4), v);
  Store4<T>::ld(p + min(n + 4, N - 4), v + 4);
}
__device__ __forceinline__ void load_gate(const float* gate, int n, int N, float (&g)[2][8]) {
  ld8(gate, n, N, g[0]);
  ld8(gate, n + 32, N, g[1]);
}

// Branch epilogue of the lane's tokens J .. J + EB - 1, features n .. n + 7 and n + 32 .. n + 39, all loads ahead of the first store;
// PLANES: planes are read back (order >= 1).
template <int J, int EB, bool PLANES, int TM>
__device__ __forceinline__ void branch_tokens(const floatx4 (&acc)[4][TM], const BranchRow<bf16_t>& br, const float (&gate)[2][8], int64_t ldh, int rows,
                                              int row0, int n, int N, bool wide) {
  float hv[EB][2][8], old[PLANES ? EB : 1][SPECA_MAX_ORDER][2][8];
#pragma unroll
  for (int u = 0; u < EB; ++u) {
    const int64_t at = (br.t0 + min(row0 + (J + u) * 16, rows - 1)) * ldh;       // rows past the end: the last one again
#pragma unroll
    for (int P = 0; P < 2; ++P) ld8(br.h + at, n + 32 * P, N, hv[u][P]);
    if constexpr (PLANES) {
#pragma unroll
      for (int o = 0; o < SPECA_MAX_ORDER; ++o)
        if (o < br.order) {
#pragma unroll
          for (int P = 0; P < 2; ++P) {
            ld4_stream(br.d[o] + at + min(n + 32 * P, N - 4), old[u][o][P]);
            ld4_stream(br.d[o] + at + min(n + 32 * P + 4, N - 4), old[u][o][P] + 4);
          }
        }
    }
  }
#pragma unroll
  for (int u = 0; u < EB; ++u) {
    const int r = row0 + (J + u) * 16;
    if (r < rows) {
      const int64_t at = (br.t0 + r) * ldh;
      float v[2][8];
#pragma unroll
      for (int P = 0; P < 2; ++P) lane_values(acc, J + u, P, v[P]);
      if (br.refresh) {
        float cur[2][8];
#pragma unroll
        for (int P = 0; P < 2; ++P) {
          const int np = n + 32 * P;
          if (np < N) st8_stream(br.d[0] + at + np, v[P], np + 4 < N, wide);
#pragma unroll
          for (int q = 0; q < 8; ++q) cur[P][q] = v[P][q];
        }
        if constexpr (PLANES) {
#pragma unroll
          for (int o = 1; o <= SPECA_MAX_ORDER; ++o)
            if (o <= br.order) {
#pragma unroll
              for (int P = 0; P < 2; ++P) {
                const int np = n + 32 * P;
#pragma unroll
                for (int q = 0; q < 8; ++q) cur[P][q] = (cur[P][q] - old[u][o - 1][P][q]) * br.inv[o - 1];
                if (np < N) st8_stream(br.d[o] + at + np, cur[P], np + 4 < N, wide);
              }
            }
        }
      }
#pragma unroll
      for (int P = 0; P < 2; ++P) {
        const int np = n + 32 * P;
#pragma unroll
        for (int q = 0; q < 8; ++q) v[P][q] = fmaf(gate[P][q], v[P][q], hv[u][P][q]);
        if (np < N) st8(br.h + at + np, v[P], np + 4 < N);
      }
    }
  }
}

// The batch row of row v of a stream or launch, for a tile that begins at its row m0
template <bool STREAMS>
__device__ __forceinline__ int batch_row(const GemmEpi& epi, const RowMap<STREAMS>& map, int v) {
  if constexpr (STREAMS) return v / map.len;
  else return v / epi.tokens;
}
template <bool STREAMS>
__device__ __forceinline__ BranchRow<bf16_t> tile_row(const GemmEpi& epi, const RowMap<STREAMS>& map, const float* gates, int m0, int v) {
  const int i = batch_row(epi, map, v);
  BranchRow<bf16_t> br = branch_row<bf16_t>(epi, i, m0);
  if constexpr (STREAMS) {
    br.gate = gates + static_cast<int64_t>(i) * epi.gate_stride;
    br.t0 = map.off + m0 - i * map.len;
  }
  return br;
}

// Token by token from J on, planes read back; where the tile spans rows of the batch every token looks its row up.
template <int J, int TM, bool STREAMS>
__device__ __forceinline__ void branch_each(const floatx4 (&acc)[4][TM], BranchRow<bf16_t>& br, float (&gate)[2][8], const GemmEpi& epi,
                                            const RowMap<STREAMS>& map, const float* gates, bool spans, int m0, int rows, int row0, int n, int N, bool wide) {
  if (spans) {
    br = tile_row(epi, map, gates, m0, m0 + min(row0 + J * 16, rows - 1));
    load_gate(br.gate, n, N, gate);
  }
  branch_tokens<J, 1, true>(acc, br, gate, epi.ldh, rows, row0, n, N, wide);
  if constexpr (J + 1 < TM) branch_each<J + 1>(acc, br, gate, epi, map, gates, spans, m0, rows, row0, n, N, wide);
}

// The epilogue of a lane (bias and gates: of its stream): rows m0 + row0, + 16, ... (TM of them), features n .. n + 7 and n + 32 .. n + 39.
template <int BM, int MODE, int TM, bool STREAMS>
__device__ __forceinline__ void lane_epilogue(floatx4 (&acc)[4][TM], const RowMap<STREAMS>& map, const void* biases, const float* gates, int m0, int row0,
                                              int n, int N, const EpiArg<MODE>& epi) {
  const int rows = map.M - m0 < BM ? map.M - m0 : BM;
  if (biases) {
    float bias[2][8] = {};
    ld8(static_cast<const bf16_t*>(biases), n, N, bias[0]);
    ld8(static_cast<const bf16_t*>(biases), n + 32, N, bias[1]);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < TM; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[i][j][q] += bias[i / 2][i % 2 * 4 + q];
  }
  if constexpr (MODE == EPI_BRANCH) {
    const bool wide = ((reinterpret_cast<uintptr_t>(epi.g.base) & 15) | ((epi.g.E | epi.cache_elem_offset | epi.ldh) & 7)) == 0;
    const int i_first = batch_row(epi, map, m0);
    float gate[2][8];
    // a tile inside one batch row needs its table once for the whole block (scalar loads)
    const bool spans = i_first != batch_row(epi, map, m0 + rows - 1);
    BranchRow<bf16_t> br = tile_row(epi, map, gates, m0, m0);
    load_gate(br.gate, n, N, gate);
    if (!spans && br.order == 0) {
      constexpr int EB = TM > 4 ? TM / 2 : TM;
      branch_tokens<0, EB, false>(acc, br, gate, epi.ldh, rows, row0, n, N, wide);
      if constexpr (EB < TM) branch_tokens<EB, TM - EB, false>(acc, br, gate, epi.ldh, rows, row0, n, N, wide);
    } else {
      branch_each<0>(acc, br, gate, epi, map, gates, spans, m0, rows, row0, n, N, wide);
    }
  } else {
    using T = std::conditional_t<MODE == EPI_F32, float, bf16_t>;
#pragma unroll
    for (int j = 0; j < TM; ++j) {
      const int r = row0 + j * 16;
      if (r < rows) {
        T* out = static_cast<T*>(epi.out) + map.at(m0 + r) * epi.ldo;
#pragma unroll
        for (int P = 0; P < 2; ++P) {
          const int np = n + 32 * P;
          float v[8];
          lane_values(acc, j, P, v);
          if constexpr (MODE == EPI_GELU || MODE == EPI_SILU) {
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] = MODE == EPI_GELU ? gelu_tanh_f(v[q]) : silu_f(v[q]);
          }
          if (np < N) st8(out + np, v, np + 4 < N);
        }
      }
    }
  }
}

Error launch_gemm_phase_streams(const Operands& o, const GemmEpi& epi, TwoStreams streams, hipStream_t st);
Error launch_gemm_duo_streams(int bm, const Operands& o, const GemmEpi& epi, const TwoStreams& streams, hipStream_t st);

}  // namespace speca
