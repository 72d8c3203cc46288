// Linear layers of the target model:  C[M,N] = A[M,K] * W[N,K]^T (+ bias) with a fused
// epilogue.  A and W are row-major with K contiguous, in the model dtype; accumulation
// is fp32.  Three kernel families implement it: bf16 MFMA with LDS-staged tiles (the dense
// contractions of reference steps), fp32 MFMA for fp32 models, with tiles through LDS where K is a
// multiple of 64 and straight from memory elsewhere, and a plain fp32-FMA tile kernel for operands whose
// strides or alignment neither takes.
#pragma once

#include <type_traits>

#include "common.h"

namespace speca {

int compute_units();               // of the device (256 where there is none)

enum EpiMode {
  EPI_STORE = 0,   // out[m][n] = T(acc + bias)
  EPI_GELU = 1,    // out[m][n] = T(gelu_tanh(acc + bias))
  EPI_SILU = 2,    // out[m][n] = T(silu(acc + bias))
  EPI_F32 = 3,     // out[m][n] = float(acc + bias)
  EPI_BRANCH = 4   // F = acc + bias is a cached branch output: optional cache refresh
                   // (D0 <- F, D^o <- (D^{o-1}_new - D^{o-1}_old) * inv_o), then h[m][n] += gate[row][n] * F
};

struct GemmEpi {
  int mode = EPI_STORE;
  const void* bias = nullptr;     // [N] model dtype
  void* out = nullptr;            // STORE/GELU/SILU/F32 destination
  int64_t ldo = 0;
  bool beside = false;            // another launch shares the chip (a row group of two): no unit counts as idle
  // EPI_BRANCH
  float* h = nullptr;             // [M][N] fp32 residual stream
  int64_t ldh = 0;
  const float* gate = nullptr;    // gate[(m / tokens) * gate_stride + n]
  int64_t gate_stride = 0;
  int tokens = 1;                 // tokens per row: m = i * tokens + t
  int refresh = 0;                // update cache slot `slot` for rows rt.row[i]
  int slot = 0;
  int64_t cache_elem_offset = 0;  // added to the position inside the cache row (a launch that covers a token sub-range)
  CacheGeom g{};
  RowTable rt{};
};

// What a kernel is given of it: only the branch epilogue needs the cache geometry and the row table (1.9 KB of arguments
// that every other launch would copy and carry for nothing).
struct EpiPlain {
  const void* bias;
  void* out;
  int64_t ldo;
};
template <int MODE> using EpiArg = std::conditional_t<MODE == EPI_BRANCH, GemmEpi, EpiPlain>;
template <int MODE> inline EpiArg<MODE> epi_arg(const GemmEpi& e) {
  if constexpr (MODE == EPI_BRANCH) return e;
  else return {e.bias, e.out, e.ldo};
}

// M may be ragged; N % 4 == 0 is required (checked).
Error launch_gemm(int dtype, const void* A, int64_t lda, const void* W, int64_t ldw, int M, int N, int K, const GemmEpi& epi,
                  hipStream_t st);
// One layer of two token ranges ("streams") of every batch row, with weights, bias and gate of their own; A, output, residual and cache
// are those of all tokens of all rows.
struct StreamLayer {
  int rows, tokens;                  // batch rows; tokens of each
  int len[2], off[2];                // tokens of a stream in a row, and the first of them
  const uint16_t* w[2];
  const void* bias[2];
  const float* gate[2];              // EPI_BRANCH: of batch row 0, epi.gate_stride apart
};
// The tile kind with which one launch for both streams of all rows is expected to take less than a launch per row and stream (the weights are
// read once, a short stream's tiles run beside the long one's, and both fill one set of rounds); negative: go row by row and stream by stream.
int streams_kind(int dtype, const void* A, int64_t lda, int64_t ldw, int N, int K, const StreamLayer& y, int mode);
Error launch_gemm_streams(int kind, const void* A, int64_t lda, int64_t ldw, int N, int K, const StreamLayer& y, const GemmEpi& epi, hipStream_t st);
// Modelled time (us) of a bf16 layer on the matrix kernels (K % 8 == 0): alone on the chip, or, `paired`, as one of two such
// layers side by side, whose tiles fill each other's partial rounds.
double layer_time(bool branch, int M, int N, int K, bool paired);

// softmax(q k^T / sqrt(hd)) v without mask.  qkv: [rows][T][3][H][hd] (model dtype),
// out: [rows][T][ldo] with the H*hd result in the first columns (ldo >= H*hd, ldo % 4 == 0).
Error launch_attention(int dtype, const void* qkv, void* out, int64_t ldo, int rows, int T, int H, int hd, hipStream_t st);

}  // namespace speca
