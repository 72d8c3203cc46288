// Dispatch of the linear layers and attention to the kernel families (see gemm.h).
#include "gemm_tile.h"

namespace speca {

Error launch_gemm_simple(int dtype, const void* A, int64_t lda, const void* W, int64_t ldw, int M, int N, int K,
                         const GemmEpi& epi, hipStream_t st);
Error launch_attention_simple(int dtype, const void* qkv, void* out, int64_t ldo, int rows, int T, int H, int hd, hipStream_t st);
bool gemm_mfma_supported(const Operands& o);
Error launch_gemm_mfma(const Operands& o, const GemmEpi& epi, hipStream_t st);
int pick_streams(const Operands& o, const StreamLayer& y, bool branch);
Error launch_gemm_mfma_streams(int kind, const Operands& o, const StreamLayer& y, const GemmEpi& epi, hipStream_t st);

bool gemm_f32_supported(const void* A, int64_t lda, const void* W, int64_t ldw, int K);
Error launch_gemm_f32(const void* A, int64_t lda, const void* W, int64_t ldw, int M, int N, int K, const GemmEpi& epi, hipStream_t st);
Error launch_attention_f32(int dtype, const void* qkv, void* out, int64_t ldo, int rows, int T, int H, int hd, hipStream_t st);

bool attention_mfma_supported(const void* qkv, const void* out, int64_t ldo, int H, int hd);
Error launch_attention_mfma(const void* qkv, void* out, int64_t ldo, int rows, int T, int H, int hd, hipStream_t st);

static Error check_epilogue(int M, int N, const GemmEpi& epi) {
  if (epi.mode == EPI_BRANCH) {
    if (!epi.h || !epi.gate || epi.tokens < 1 || epi.ldh != N) SPECA_FAIL(SPECA_EINVAL, "gemm: branch epilogue arguments");
    if (M % epi.tokens) SPECA_FAIL(SPECA_EINVAL, "gemm: M=%d is not a multiple of tokens=%d", M, epi.tokens);
    if (epi.refresh) {
      if (M / epi.tokens != epi.rt.n || epi.cache_elem_offset < 0 || epi.cache_elem_offset % 4 ||
          epi.g.E < epi.cache_elem_offset + static_cast<int64_t>(epi.tokens) * N || epi.slot < 0 || epi.slot >= epi.g.n_slots)
        SPECA_FAIL(SPECA_EINVAL, "gemm: cache refresh geometry does not match the launch");
      for (int i = 0; i < epi.rt.n; ++i)
        if (epi.rt.row[i] < 0 || epi.rt.order[i] < 0 || epi.rt.row[i] / epi.g.batch_rows + epi.rt.order[i] > epi.g.m)   // plane + order
          SPECA_FAIL(SPECA_EINVAL, "gemm: cache row table out of range");
    }
  } else if (!epi.out || epi.ldo < N) {
    SPECA_FAIL(SPECA_EINVAL, "gemm: output missing");
  }
  return ok();
}

Error launch_gemm(int dtype, const void* A, int64_t lda, const void* W, int64_t ldw, int M, int N, int K, const GemmEpi& epi,
                  hipStream_t st) {
  if (!A || !W) SPECA_FAIL(SPECA_EINVAL, "gemm: NULL operand");
  if (M < 1 || N < 4 || K < 1 || N % 4) SPECA_FAIL(SPECA_EINVAL, "gemm: M=%d N=%d K=%d (N must be a multiple of 4)", M, N, K);
  if (lda < K || ldw < K) SPECA_FAIL(SPECA_EINVAL, "gemm: leading dimensions smaller than K");
  SPECA_TRY(check_epilogue(M, N, epi));
  if (dtype == SPECA_BF16) {
    const Operands o{static_cast<const uint16_t*>(A), lda, static_cast<const uint16_t*>(W), ldw, M, N, K};
    if (gemm_mfma_supported(o)) return launch_gemm_mfma(o, epi, st);
  }
  if (dtype == SPECA_F32 && gemm_f32_supported(A, lda, W, ldw, K))
    return launch_gemm_f32(A, lda, W, ldw, M, N, K, epi, st);
  return launch_gemm_simple(dtype, A, lda, W, ldw, M, N, K, epi, st);
}

static Operands stream_operands(const void* A, int64_t lda, int64_t ldw, int N, int K, const StreamLayer& y) {
  return {static_cast<const uint16_t*>(A), lda, y.w[0], ldw, y.rows * y.tokens, N, K};
}

int streams_kind(int dtype, const void* A, int64_t lda, int64_t ldw, int N, int K, const StreamLayer& y, int mode) {
  if (dtype != SPECA_BF16 || mode == EPI_SILU || lda < K || ldw < K) return -1;
  return pick_streams(stream_operands(A, lda, ldw, N, K, y), y, mode == EPI_BRANCH);
}

Error launch_gemm_streams(int kind, const void* A, int64_t lda, int64_t ldw, int N, int K, const StreamLayer& y, const GemmEpi& epi, hipStream_t st) {
  GemmEpi e = epi;
  e.gate = y.gate[0];
  SPECA_TRY(check_epilogue(y.rows * y.tokens, N, e));
  return launch_gemm_mfma_streams(kind, stream_operands(A, lda, ldw, N, K, y), y, e, st);
}

Error launch_attention(int dtype, const void* qkv, void* out, int64_t ldo, int rows, int T, int H, int hd, hipStream_t st) {
  if (!qkv || !out || rows < 1 || T < 1 || H < 1 || ldo < static_cast<int64_t>(H) * hd || ldo % 4) SPECA_FAIL(SPECA_EINVAL, "attention: bad arguments");
  if (dtype == SPECA_BF16 && attention_mfma_supported(qkv, out, ldo, H, hd))
    return launch_attention_mfma(qkv, out, ldo, rows, T, H, hd, st);
  // the fp32 matrix instructions take 16-byte pieces of fp32 and 8-byte pieces of bf16 operands (head sizes are multiples of 8)
  const uintptr_t piece = dtype == SPECA_BF16 ? 8 : 16;
  if (reinterpret_cast<uintptr_t>(qkv) % piece == 0 && reinterpret_cast<uintptr_t>(out) % piece == 0)
    return launch_attention_f32(dtype, qkv, out, ldo, rows, T, H, hd, st);
  return launch_attention_simple(dtype, qkv, out, ldo, rows, T, H, hd, st);
}

}  // namespace speca
