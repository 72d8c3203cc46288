// fp32 GEMM and attention on the fp32 matrix instructions (v_mfma_f32_16x16x4_f32: 157 TFLOP/s on the chip, twice what
// unpacked vector FMAs reach, and exact fp32 products and sums).
//
// The models that run in fp32 are small, so their launches are bound by latency, not by rate: a 512 x 384 x 1536 layer is
// 4 us of matrix work, and a vector-FMA block walking K behind a barrier per 16 columns took 97 us (now 11; attention over
// 256 keys of two rows x 6 heads 340 us with one query per thread, now 8).  Hence, but for the larger tiles of whole 64-column stages,
//   - no LDS and no barrier in the loops: a lane's operands come from memory as 16-byte pieces that are fragments as they
//     stand.  The reduction index is a dummy, so lane l of a wave simply takes columns 4 (l / 16) .. + 3 of its row, and
//     instruction c of the step consumes component c of both operands: one load feeds four instructions;
//   - several steps of loads in flight in registers;
//   - the four waves of a block share one output tile and split K (GEMM: steps of 16 dealt round robin) or the keys
//     (attention: tiles of 16 keys), and their partial results meet once, in LDS, in wave order.  The split depends on K
//     (on the number of keys) alone, so a row's bits depend neither on M nor on the tile.
#include <algorithm>
#include <type_traits>

#include "epilogue.h"
#include "gemm.h"

namespace speca {

namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ floatx4 mfma4(float a, float b, floatx4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

// ---- GEMM ------------------------------------------------------------------------------------------------------
// Block tile (16 TM) x (16 TN); weights are the first operand, so a lane holds four consecutive output features of one row.
// PF = steps of loads in flight per wave.
// KTAIL: K is no multiple of 16.
template <int TM, int TN, int PF, int MODE, bool KTAIL>
__global__ __launch_bounds__(256) void gemm_f32_small_kernel(const float* __restrict__ A, int64_t lda, const float* __restrict__ W, int64_t ldw, int M, int N,
                                                       int K, EpiArg<MODE> epi) {
  constexpr int BM = 16 * TM, BN = 16 * TN;
  constexpr int CST = BN + 4;                     // floats per staged row
  __shared__ __align__(16) float part[4][BM * CST];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, kq = (lane >> 4) * 4;
  const int64_t mt = static_cast<int64_t>(blockIdx.z) * gridDim.y + blockIdx.y;      // more than 32768 row tiles go on in z
  if (mt * BM >= M) return;
  const int m0 = static_cast<int>(mt) * BM, n0 = blockIdx.x * BN;
  const float* pa[TM];
  const float* pw[TN];
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int m = m0 + i * 16 + l16;
    pa[i] = A + static_cast<int64_t>(m < M ? m : M - 1) * lda;      // rows beyond M / N repeat the last one and are never stored
  }
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int n = n0 + j * 16 + l16;
    pw[j] = W + static_cast<int64_t>(n < N ? n : N - 1) * ldw;
  }
  floatx4 acc[TN][TM];
#pragma unroll
  for (int j = 0; j < TN; ++j)
#pragma unroll
    for (int i = 0; i < TM; ++i) acc[j][i] = floatx4{0.f, 0.f, 0.f, 0.f};

  const int n_all = (K + 15) / 16;                                  // steps of 16 columns
  const int steps = (n_all - wave + 3) / 4;                         // this wave's: wave, wave + 4, ...
  floatx4 ra[PF][TM], rw[PF][TN];
  // A step past the end re-reads the last one (never consumed).  Columns past K re-read column 0 and are zeroed where they are
  // consumed: a select next to the load would wait for it there.
  auto load = [&](int s, floatx4 (&a)[TM], floatx4 (&w)[TN]) {
    int k = (wave + 4 * (s < steps ? s : (steps > 0 ? steps - 1 : 0))) * 16 + kq;
    if (KTAIL || steps == 0) k = k < K ? k : 0;
#pragma unroll
    for (int i = 0; i < TM; ++i) a[i] = *reinterpret_cast<const floatx4*>(pa[i] + k);
#pragma unroll
    for (int j = 0; j < TN; ++j) w[j] = *reinterpret_cast<const floatx4*>(pw[j] + k);
  };
#pragma unroll
  for (int p = 0; p < PF; ++p) load(p, ra[p], rw[p]);
  auto step = [&](int s, floatx4 (&a)[TM], floatx4 (&w)[TN]) {
    if (KTAIL && (wave + 4 * s) * 16 + kq >= K) {
#pragma unroll
      for (int i = 0; i < TM; ++i) a[i] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int j = 0; j < TN; ++j) w[j] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int i = 0; i < TM; ++i) acc[j][i] = mfma4(w[j][c], a[i][c], acc[j][i]);
  };
  // no branch around a load in the loop, so that the compiler counts the outstanding ones instead of draining them
  int s = 0;
  for (; s + PF <= steps; s += PF) {
#pragma unroll
    for (int p = 0; p < PF; ++p) {
      step(s + p, ra[p], rw[p]);
      load(s + p + PF, ra[p], rw[p]);
    }
  }
#pragma unroll
  for (int p = 0; p < PF; ++p)
    if (s + p < steps) step(s + p, ra[p], rw[p]);
#pragma unroll
  for (int j = 0; j < TN; ++j)
#pragma unroll
    for (int i = 0; i < TM; ++i) *reinterpret_cast<floatx4*>(&part[wave][(i * 16 + l16) * CST + j * 16 + kq]) = acc[j][i];
  __syncthreads();
  constexpr int QPR = BN / 4;
#pragma unroll
  for (int q = tid; q < BM * QPR; q += 256) {
    const int r = q / QPR, c = (q % QPR) * 4;
    const int m = m0 + r, n = n0 + c;
    if (m < M && n < N) {
      float v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = ((part[0][r * CST + c + e] + part[1][r * CST + c + e]) + part[2][r * CST + c + e]) + part[3][r * CST + c + e];
      epilogue_quad<float, MODE>(epi, m, n, v);
    }
  }
}

// The same for tiles that leave every unit enough to do: operands come through LDS.  Fragments straight from memory are 16 rows x 64 bytes per
// instruction, of which a unit takes 33 bytes per ns; loads that go to LDS directly take 256 bytes of each of 4 rows, 94.  A stage is 64 columns, the
// four steps of 16 that the four waves deal among themselves, so every wave adds up the same products in the same order as above.
// Chunk c (16 bytes) of row r sits at position c ^ (r % 16): the rows of a fragment touch all banks once.  A ring of NS stages; a wave
// waits for its own loads (in issue order) and for its fragments ahead of the barrier behind which the stage before is loaded over.
// Needs K % 64 == 0: with the zeros of a last stage selected in the loop, 512 x 1152 x 384 took 10.4 us and 1000 x 772 x 260 was slower than above.
// us, above -> here: 512 x 1152 x 384 11.6 -> 9.1, 512 x 384 x 1536 14.5 -> 11.3, 2048 x 1152 x 384 37.3 -> 27.8, 33 x 4608 x 1152 16.7 -> 14.5,
// 8192 x 1152 x 1152 247 -> 191, 4096^3 1392 -> 1133 (121 TFLOP/s).

constexpr int f32_stage_bytes(int TM, int TN) { return 16 * (TM + TN) * 256; }
constexpr int f32_lds_bytes(int TM, int TN, int NS) {
  const int ring = NS * f32_stage_bytes(TM, TN), part = 4 * 16 * TM * (16 * TN + 4) * 4;
  return ring > part ? ring : part;
}

template <int TM, int TN, int NS, int MODE>
__global__ __launch_bounds__(256) void gemm_f32_kernel(const float* __restrict__ A, int64_t lda, const float* __restrict__ W, int64_t ldw, int M, int N,
                                                       int K, EpiArg<MODE> epi) {
  constexpr int BM = 16 * TM, BN = 16 * TN, CST = BN + 4, STAGE = f32_stage_bytes(TM, TN);
  constexpr int L = (BM + BN) / 16;               // loads of a wave per stage
  static_assert((BM + BN) % 16 == 0 && BM % 16 == 0 && NS >= 2 && (NS - 1) * L < 64, "4 rows per load, four waves");
  extern __shared__ __align__(16) char lds[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, g4 = lane >> 4;
  const int64_t mt = static_cast<int64_t>(blockIdx.z) * gridDim.y + blockIdx.y;
  if (mt * BM >= M) return;
  const int m0 = static_cast<int>(mt) * BM, n0 = blockIdx.x * BN;
  // load u of a wave: rows 4 g .. + 3 of the tile's BM + BN, g = wave + 4 u; lane l supplies what lies at position l % 16 of row 4 g + l / 16
  const float* from[L];
#pragma unroll
  for (int u = 0; u < L; ++u) {
    const int r = (wave + 4 * u) * 4 + (lane >> 4), rw = r - BM;
    from[u] = (r < BM ? A + static_cast<int64_t>(m0 + r < M ? m0 + r : M - 1) * lda : W + static_cast<int64_t>(n0 + rw < N ? n0 + rw : N - 1) * ldw) + ((lane & 15) ^ (r & 15)) * 4;
  }
  auto load = [&](int s, int slot) {
#pragma unroll
    for (int u = 0; u < L; ++u) {
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(from[u] + static_cast<int64_t>(s) * 64), (__attribute__((address_space(3))) void*)(lds + slot * STAGE + (wave + 4 * u) * 1024), 16, 0, 0);
    }
  };
  floatx4 acc[TN][TM];
#pragma unroll
  for (int j = 0; j < TN; ++j)
#pragma unroll
    for (int i = 0; i < TM; ++i) acc[j][i] = floatx4{0.f, 0.f, 0.f, 0.f};
  const int nk = K / 64;
#pragma unroll
  for (int s = 0; s < NS - 1; ++s)
    if (s < nk) load(s, s);
  constexpr auto loads_left = [](int n) { return (n & 15) | ((n >> 4) << 14) | 0x0F70; };          // s_waitcnt vmcnt(n)
  const int at = l16 * 256 + ((4 * wave + g4) ^ l16) * 16;
  int slot = 0, next = NS - 1;                    // of stage s and of stage s + NS - 1
  for (int s = 0; s < nk; ++s) {
    if (s + NS - 2 < nk) __builtin_amdgcn_s_waitcnt(loads_left((NS - 2) * L));
    else __builtin_amdgcn_s_waitcnt(loads_left(0));
    __builtin_amdgcn_s_waitcnt(0xC07F);           // fragments of the stage before
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    if (s + NS - 1 < nk) load(s + NS - 1, next);
    floatx4 a[TM], w[TN];
#pragma unroll
    for (int i = 0; i < TM; ++i) a[i] = *reinterpret_cast<const floatx4*>(lds + slot * STAGE + at + i * 16 * 256);
#pragma unroll
    for (int j = 0; j < TN; ++j) w[j] = *reinterpret_cast<const floatx4*>(lds + slot * STAGE + at + (BM + j * 16) * 256);
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int i = 0; i < TM; ++i) acc[j][i] = mfma4(w[j][c], a[i][c], acc[j][i]);
    slot = slot + 1 == NS ? 0 : slot + 1;
    next = next + 1 == NS ? 0 : next + 1;
  }
  __syncthreads();
  float* part = reinterpret_cast<float*>(lds);
#pragma unroll
  for (int j = 0; j < TN; ++j)
#pragma unroll
    for (int i = 0; i < TM; ++i) *reinterpret_cast<floatx4*>(part + wave * (BM * CST) + (i * 16 + l16) * CST + j * 16 + 4 * g4) = acc[j][i];
  __syncthreads();
  constexpr int QPR = BN / 4;
#pragma unroll
  for (int q = tid; q < BM * QPR; q += 256) {
    const int r = q / QPR, c = (q % QPR) * 4;
    const int m = m0 + r, n = n0 + c;
    if (m < M && n < N) {
      float v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float* x = part + r * CST + c + e;
        v[e] = ((x[0] + x[BM * CST]) + x[2 * BM * CST]) + x[3 * BM * CST];
      }
      epilogue_quad<float, MODE>(epi, m, n, v);
    }
  }
}

template <int TM, int TN, int NS, int MODE>
Error launch_f32_mode(dim3 grid, const float* A, int64_t lda, const float* W, int64_t ldw, int M, int N, int K, const GemmEpi& epi, hipStream_t st) {
  auto kern = gemm_f32_kernel<TM, TN, NS, MODE>;
  constexpr int smem = f32_lds_bytes(TM, TN, NS);
  static bool attr_set = false;   // more than 64 KB of dynamic LDS must be requested once per kernel
  if (smem > 64 * 1024 && !attr_set) {
    SPECA_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, smem));
    attr_set = true;
  }
  kern<<<grid, 256, smem, st>>>(A, lda, W, ldw, M, N, K, epi_arg<MODE>(epi));
  SPECA_HIP(hipGetLastError());
  return ok();
}

template <int TM, int TN, int NS>
Error launch_f32_lds(const float* A, int64_t lda, const float* W, int64_t ldw, int M, int N, int K, const GemmEpi& epi, hipStream_t st) {
  const unsigned row_tiles = (M + 16 * TM - 1) / (16 * TM), grid_y = row_tiles < 32768 ? row_tiles : 32768;
  const dim3 grid((N + 16 * TN - 1) / (16 * TN), grid_y, (row_tiles + grid_y - 1) / grid_y);
#define SPECA_LAUNCH(MODE_) \
  case MODE_: return launch_f32_mode<TM, TN, NS, MODE_>(grid, A, lda, W, ldw, M, N, K, epi, st);
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

template <int TM, int TN, int PF>
Error launch_f32_tile(const float* A, int64_t lda, const float* W, int64_t ldw, int M, int N, int K, const GemmEpi& epi,
                      hipStream_t st) {
  const unsigned row_tiles = (M + 16 * TM - 1) / (16 * TM), grid_y = row_tiles < 32768 ? row_tiles : 32768;
  const dim3 grid((N + 16 * TN - 1) / (16 * TN), grid_y, (row_tiles + grid_y - 1) / grid_y);
#define SPECA_LAUNCH(MODE_)                                                                                                  \
  {                                                                                                                          \
    if (K % 16) gemm_f32_small_kernel<TM, TN, PF, MODE_, true><<<grid, 256, 0, st>>>(A, lda, W, ldw, M, N, K, epi_arg<MODE_>(epi)); \
    else gemm_f32_small_kernel<TM, TN, PF, MODE_, false><<<grid, 256, 0, st>>>(A, lda, W, ldw, M, N, K, epi_arg<MODE_>(epi));        \
  }
  switch (epi.mode) {
    case EPI_STORE: SPECA_LAUNCH(EPI_STORE) break;
    case EPI_GELU: SPECA_LAUNCH(EPI_GELU) break;
    case EPI_SILU: SPECA_LAUNCH(EPI_SILU) break;
    case EPI_F32: SPECA_LAUNCH(EPI_F32) break;
    case EPI_BRANCH: SPECA_LAUNCH(EPI_BRANCH) break;
    default: SPECA_FAIL(SPECA_EINVAL, "gemm: epilogue mode %d", epi.mode);
  }
#undef SPECA_LAUNCH
  SPECA_HIP(hipGetLastError());
  return ok();
}

// ---- attention ----------------------------------------------------------------------------------------------------
// One block = 16 QT queries of one (row, head); its four waves take the 16-key tiles w, w + 4, ... with an online softmax of
// their own and merge at the end.  Transposed products as in the bf16 kernels: S^T[key][query] leaves lane l with keys
// 4 (l / 16) .. + 3 of query l % 16, which is the second operand of the O^T product as it stands (instruction r takes keys
// 4 q + r).  The head dimension is dealt to the 16-row tiles of O^T in pieces of four (tile i % 4 of group i / 4 owns
// dimensions 64 g + 4 row + i), so a lane's values are 16-byte pieces of V and of the output.  Values of head size 72 past
// 64 take single elements.  T = storage type of q, k, v and the output; arithmetic is fp32.
template <typename T> __device__ inline floatx4 ld_quad(const T* p);
template <> __device__ inline floatx4 ld_quad<float>(const float* p) { return *reinterpret_cast<const floatx4*>(p); }
template <> __device__ inline floatx4 ld_quad<bf16_t>(const bf16_t* p) {
  float v[4];
  Store4<bf16_t>::ld(p, v);
  return floatx4{v[0], v[1], v[2], v[3]};
}
template <typename T> __device__ inline float ld_one(const T* p);
template <> __device__ inline float ld_one<float>(const float* p) { return *p; }
template <> __device__ inline float ld_one<bf16_t>(const bf16_t* p) { return bf16_to_f32(p->bits); }

template <typename T, int HD, int QT>
__global__ __launch_bounds__(256) void attention_f32_kernel(const T* __restrict__ qkv, T* __restrict__ out, int64_t ldo, int Tn, int64_t D, float scale_log2e) {
  constexpr int KS = (HD + 15) / 16;              // steps of 16 dimensions in q k^T
  constexpr int G = HD / 64;                      // groups of four tiles of O^T (64 dimensions)
  constexpr int REM = HD - 64 * G;                // what is left: 8, 16 or 32 dimensions in tiles of 16
  constexpr int RT = (REM + 15) / 16;
  constexpr int DT = 4 * G + RT;
  static_assert(HD % 8 == 0 && (REM == 0 || REM == 8 || REM == 16 || REM == 32), "head_dim");
  constexpr int OST = 16 * DT + 4;                // floats per query in the merge buffer
  __shared__ __align__(16) float merge[3][16 * OST];
  __shared__ float stats[4][2][16];
  const int row = blockIdx.z, head = blockIdx.y, q0 = blockIdx.x * 16 * QT;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, g4 = lane >> 4;
  const T* base = qkv + static_cast<int64_t>(row) * Tn * 3 * D + head * HD;      // D = heads x HD, of which this launch may cover a part
  const floatx4 zero = {0.f, 0.f, 0.f, 0.f};

  floatx4 qf[QT][KS];
#pragma unroll
  for (int t = 0; t < QT; ++t) {
    const int q = q0 + t * 16 + l16;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const int d = s * 16 + g4 * 4;
      qf[t][s] = d < HD ? ld_quad(base + static_cast<int64_t>(q < Tn ? q : Tn - 1) * 3 * D + d) : zero;
    }
  }
  floatx4 o[QT][DT];
  float mrun[QT], lrun[QT];
#pragma unroll
  for (int t = 0; t < QT; ++t) {
    mrun[t] = -INFINITY; lrun[t] = 0.0f;
#pragma unroll
    for (int i = 0; i < DT; ++i) o[t][i] = zero;
  }
  const int ntiles = (Tn + 15) / 16;
  floatx4 kf[KS];
  auto load_k = [&](int kt) {
    int key = kt * 16 + l16;
    key = key < Tn ? key : Tn - 1;
    const T* p = base + static_cast<int64_t>(key) * 3 * D + D + g4 * 4;
#pragma unroll
    for (int s = 0; s < KS; ++s) kf[s] = s * 16 + g4 * 4 < HD ? ld_quad(p + s * 16) : zero;
  };
  if (wave < ntiles) load_k(wave);
  for (int kt = wave; kt < ntiles; kt += 4) {
    // this tile's values, on their way during the scores
    floatx4 vf[4][G > 0 ? G : 1];
    float vr[4][RT > 0 ? RT : 1];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      int key = kt * 16 + g4 * 4 + r;
      key = key < Tn ? key : Tn - 1;
      const T* p = base + static_cast<int64_t>(key) * 3 * D + 2 * D;
#pragma unroll
      for (int g = 0; g < G; ++g) vf[r][g] = ld_quad(p + g * 64 + l16 * 4);
#pragma unroll
      for (int i = 0; i < RT; ++i) vr[r][i] = i * 16 + l16 < REM ? ld_one(p + 64 * G + i * 16 + l16) : 0.0f;
    }
    floatx4 s[QT];
#pragma unroll
    for (int t = 0; t < QT; ++t) s[t] = zero;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int t = 0; t < QT; ++t) s[t] = mfma4(kf[ks][c], qf[t][ks][c], s[t]);
    if (kt + 4 < ntiles) load_k(kt + 4);
    if (kt * 16 + 16 > Tn) {                       // keys past the end: probability 0, which must not meet an infinite value
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        if (kt * 16 + g4 * 4 + r < Tn) continue;
#pragma unroll
        for (int g = 0; g < G; ++g) vf[r][g] = zero;
#pragma unroll
        for (int i = 0; i < RT; ++i) vr[r][i] = 0.0f;
      }
    }
#pragma unroll
    for (int t = 0; t < QT; ++t) {
      if (kt * 16 + 16 > Tn) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (kt * 16 + g4 * 4 + r >= Tn) s[t][r] = -INFINITY;
      }
      float tmax = fmaxf(fmaxf(s[t][0], s[t][1]), fmaxf(s[t][2], s[t][3]));
      tmax = fmaxf(tmax, __shfl_xor(tmax, 16, 64));
      tmax = fmaxf(tmax, __shfl_xor(tmax, 32, 64));
      const float mnew = fmaxf(mrun[t], tmax);
      // A wave may see nothing but scores of -inf in its tiles (an infinite key): weight 0 then, and not -inf - (-inf).  Only a
      // query whose every score is -inf has no softmax; the merge makes that NaN.
      const float moff = mnew == -INFINITY ? 0.0f : mnew * scale_log2e;
      const float corr = __builtin_amdgcn_exp2f(fmaf(mrun[t], scale_log2e, -moff));     // the first tile: exp2(-inf) = 0
      float p[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) p[r] = __builtin_amdgcn_exp2f(fmaf(s[t][r], scale_log2e, -moff));
      lrun[t] = fmaf(lrun[t], corr, (p[0] + p[1]) + (p[2] + p[3]));
      mrun[t] = mnew;
#pragma unroll
      for (int i = 0; i < DT; ++i) o[t][i] *= corr;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
#pragma unroll
        for (int i = 0; i < 4 * G; ++i) o[t][i] = mfma4(vf[r][i / 4][i % 4], p[r], o[t][i]);
#pragma unroll
        for (int i = 0; i < RT; ++i) o[t][4 * G + i] = mfma4(vr[r][i], p[r], o[t][4 * G + i]);
      }
    }
  }
  // merge in wave order: every wave scales its sums to the common maximum; waves 1 .. 3 hand theirs over in LDS
#pragma unroll
  for (int t = 0; t < QT; ++t) {
    float l = lrun[t];
    l += __shfl_xor(l, 16, 64);
    l += __shfl_xor(l, 32, 64);
    if (t > 0) __syncthreads();
    if (lane < 16) { stats[wave][0][l16] = mrun[t]; stats[wave][1][l16] = l; }
    __syncthreads();
    const float m = fmaxf(fmaxf(stats[0][0][l16], stats[1][0][l16]), fmaxf(stats[2][0][l16], stats[3][0][l16]));
    float f[4], lsum = 0.0f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      f[w] = __builtin_amdgcn_exp2f((stats[w][0][l16] - m) * scale_log2e);            // a wave without a tile: exp2(-inf) = 0
      lsum = fmaf(stats[w][1][l16], f[w], lsum);
    }
    const float mine = wave == 0 ? f[0] : wave == 1 ? f[1] : wave == 2 ? f[2] : f[3];
    if (wave > 0) {
#pragma unroll
      for (int i = 0; i < DT; ++i) *reinterpret_cast<floatx4*>(&merge[wave - 1][l16 * OST + i * 16 + g4 * 4]) = o[t][i] * mine;
    }
    __syncthreads();
    if (wave == 0) {
      const float inv = 1.0f / lsum;
      const int q = q0 + t * 16 + l16;
#pragma unroll
      for (int i = 0; i < DT; ++i) {
        floatx4 v = o[t][i] * mine;
#pragma unroll
        for (int w = 0; w < 3; ++w) v += *reinterpret_cast<const floatx4*>(&merge[w][l16 * OST + i * 16 + g4 * 4]);
        o[t][i] = v * inv;
      }
      if (q < Tn) {
        T* op = out + (static_cast<int64_t>(row) * Tn + q) * ldo + head * HD;
        // accumulator r of tile i of group g is dimension 64 g + 4 (4 g4 + r) + i
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const float v[4] = {o[t][4 * g][r], o[t][4 * g + 1][r], o[t][4 * g + 2][r], o[t][4 * g + 3][r]};
            Store4<T>::st(op + g * 64 + 4 * (4 * g4 + r), v);
          }
#pragma unroll
        for (int i = 0; i < RT; ++i) {
          const int d = i * 16 + g4 * 4;
          const float v[4] = {o[t][4 * G + i][0], o[t][4 * G + i][1], o[t][4 * G + i][2], o[t][4 * G + i][3]};
          if (d < REM) Store4<T>::st(op + 64 * G + d, v);
        }
      }
    }
  }
}

template <typename T, int HD>
Error launch_attn_f32_hd(const void* qkv, void* out, int64_t ldo, int rows, int Tn, int H, hipStream_t st) {
  const float sl2 = 1.4426950408889634f / sqrtf(static_cast<float>(HD));
  const int64_t D = static_cast<int64_t>(H) * HD;
  // 32 queries per block read every key and value half as often; 16 keep the chip busy when there are few of them
  const bool two = static_cast<int64_t>((Tn + 31) / 32) * H * rows >= 512;
  const unsigned blocks = two ? (Tn + 31) / 32 : (Tn + 15) / 16;
  constexpr int kMost = 65535;                    // rows and heads of one grid
  for (int r0 = 0; r0 < rows; r0 += kMost)
    for (int h0 = 0; h0 < H; h0 += kMost) {
      const dim3 grid(blocks, H - h0 < kMost ? H - h0 : kMost, rows - r0 < kMost ? rows - r0 : kMost);
      const T* q = static_cast<const T*>(qkv) + static_cast<int64_t>(r0) * Tn * 3 * D + static_cast<int64_t>(h0) * HD;
      T* o = static_cast<T*>(out) + static_cast<int64_t>(r0) * Tn * ldo + static_cast<int64_t>(h0) * HD;
      if (two) attention_f32_kernel<T, HD, 2><<<grid, 256, 0, st>>>(q, o, ldo, Tn, D, sl2);
      else attention_f32_kernel<T, HD, 1><<<grid, 256, 0, st>>>(q, o, ldo, Tn, D, sl2);
      SPECA_HIP(hipGetLastError());
    }
  return ok();
}

template <typename T>
Error launch_attn_f32_t(const void* qkv, void* out, int64_t ldo, int rows, int Tn, int H, int hd, hipStream_t st) {
  switch (hd) {
    case 16: return launch_attn_f32_hd<T, 16>(qkv, out, ldo, rows, Tn, H, st);
    case 32: return launch_attn_f32_hd<T, 32>(qkv, out, ldo, rows, Tn, H, st);
    case 64: return launch_attn_f32_hd<T, 64>(qkv, out, ldo, rows, Tn, H, st);
    case 72: return launch_attn_f32_hd<T, 72>(qkv, out, ldo, rows, Tn, H, st);
    case 128: return launch_attn_f32_hd<T, 128>(qkv, out, ldo, rows, Tn, H, st);
  }
  SPECA_FAIL(SPECA_EUNSUPPORTED, "attention: head_dim %d (supported: 16, 32, 64, 72, 128)", hd);
}

}  // namespace

bool gemm_f32_supported(const void* A, int64_t lda, const void* W, int64_t ldw, int K) {
  return K % 4 == 0 && lda % 4 == 0 && ldw % 4 == 0 && reinterpret_cast<uintptr_t>(A) % 16 == 0 && reinterpret_cast<uintptr_t>(W) % 16 == 0;
}

// Which kernel runs a layer: 0 .. 4 straight from memory, 5 .. 8 through LDS.
int gemm_f32_kind(int M, int N, int K) {
  const auto blocks = [&](int bm, int bn) { return static_cast<int64_t>((M + bm - 1) / bm) * ((N + bn - 1) / bn); };
  const int rows = (M + 15) / 16 * 16, units = compute_units();
  // Straight from memory, the largest tile that still makes 128 blocks (one on every second compute unit): a block's waves read every operand
  // piece once per tile, and that traffic costs more than idle units do down to there (512 x 1152 x 384: 144 blocks of 64 x 64
  // 11.4 us, 576 of 32 x 32 12.8, 2304 of 16 x 16 18.1; 512 x 384 x 384 with 48 / 192 / 768 blocks: 11.1 / 5.6 / 7.6 us).
  // Tiles more than twice as high as the problem only read rows again.
  constexpr int bm[5] = {64, 32, 32, 16, 16}, bn[5] = {64, 64, 32, 32, 16};
  int kind = 0;
  while (kind < 4 && (bm[kind] > 2 * rows || blocks(bm[kind], bn[kind]) < units / 2)) ++kind;
  if (K % 64 || rows < 32 || kind > 2) return kind;
  // Through LDS, the tile that takes least: its rounds over the units times its stages, each the longer of 4 TM TN matrix instructions per wave
  // (32 clocks) and of its loads at 94 bytes per ns, and 0.4 us a round.  Fewer than 128 blocks of 32 x 32, or 16 rows: a step's latency
  // binds, not the loads.
  constexpr int tm[4] = {4, 4, 2, 2}, tn[4] = {4, 3, 4, 2};
  int best = 0;
  double least = 0.0;
  for (int k = 0; k < 4; ++k) {
    const double rounds = static_cast<double>((blocks(16 * tm[k], 16 * tn[k]) + units - 1) / units);
    const double stage = std::max(tm[k] * tn[k] * 0.0533, (tm[k] + tn[k]) * 16 * 256 / 94e3);
    const double time = rounds * (stage * (K / 64) + 0.4);
    if (k == 0 || time < least) { best = k; least = time; }
  }
  return 5 + best;
}

Error launch_gemm_f32(const void* A, int64_t lda, const void* W, int64_t ldw, int M, int N, int K, const GemmEpi& epi, hipStream_t st) {
  const float *a = static_cast<const float*>(A), *w = static_cast<const float*>(W);
  switch (gemm_f32_kind(M, N, K)) {
    case 0: return launch_f32_tile<4, 4, 2>(a, lda, w, ldw, M, N, K, epi, st);
    case 1: return launch_f32_tile<2, 4, 3>(a, lda, w, ldw, M, N, K, epi, st);
    case 2: return launch_f32_tile<2, 2, 4>(a, lda, w, ldw, M, N, K, epi, st);
    case 3: return launch_f32_tile<1, 2, 6>(a, lda, w, ldw, M, N, K, epi, st);
    case 4: return launch_f32_tile<1, 1, 8>(a, lda, w, ldw, M, N, K, epi, st);
    case 5: return launch_f32_lds<4, 4, 2>(a, lda, w, ldw, M, N, K, epi, st);
    case 6: return launch_f32_lds<4, 3, 2>(a, lda, w, ldw, M, N, K, epi, st);
    case 7: return launch_f32_lds<2, 4, 3>(a, lda, w, ldw, M, N, K, epi, st);
    default: return launch_f32_lds<2, 2, 4>(a, lda, w, ldw, M, N, K, epi, st);
  }
}

Error launch_attention_f32(int dtype, const void* qkv, void* out, int64_t ldo, int rows, int T, int H, int hd, hipStream_t st) {
  return dtype == SPECA_BF16 ? launch_attn_f32_t<bf16_t>(qkv, out, ldo, rows, T, H, hd, st) : launch_attn_f32_t<float>(qkv, out, ldo, rows, T, H, hd, st);
}

}  // namespace speca
