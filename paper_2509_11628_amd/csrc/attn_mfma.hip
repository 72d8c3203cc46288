// bf16 MFMA attention for gfx950: softmax(q k^T / sqrt(hd)) v without mask, online softmax
// in fp32 (no T x T matrix is ever written).
//
// Both contractions run on the bf16 matrix instructions and produce TRANSPOSED tiles:
//   S^T[key][query] = K q^T   (A operand = key rows from LDS, B operand = the wave's query
//                              rows, held in registers for the whole kernel)
//   O^T[d][query]  += V^T P^T (A operand = V^T from LDS, B operand = P^T)
// In both results a lane's values belong to ONE query (its column), so the softmax statistics and the rescaling of O are
// lane-local; only the maximum and the sum over the lanes that share a column cross lanes.  The P^T operand is taken straight
// from the S^T accumulators: the reduction index is a dummy, so the keys are simply fed to the second contraction in the order
// the first one left them in the lane, and V^T is read from LDS in that same order.
// Two kernels: a tiled one (keys/values in 64-key tiles that go global -> LDS directly, V^T fragments from the transposing
// LDS read, the next tile's scores issued under the current tile's online softmax; 16x16x32 instructions) and, for T <= 256, one
// that holds the whole sequence of a head in LDS (V transposed on its way there, in registers) and takes the softmax in one pass
// (32x32x16).  head_dim is padded with zeros to whole instructions (results that are not stored).
#include <type_traits>

#include "gemm.h"

namespace speca {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

union Frag {
  uint4 u;
  bf16x8 v;
};

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// two floats -> packed bf16 pair, round to nearest even (one v_cvt_pk_bf16_f32)
__device__ inline uint32_t cvt_pk_bf16(float a, float b) {
  const floatx2 f = {a, b};
  const bf16x2 r = __builtin_convertvector(f, bf16x2);
  return *reinterpret_cast<const uint32_t*>(&r);
}

// 2^x by the hardware instruction alone (inputs are <= 0 here; results below the normal range flush
// to 0, -inf gives 0): exp2f() wraps it in range checks and a rescale, ~5 vector instructions per value.
__device__ inline float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Transposed value tile in LDS: row = head dimension d, NK keys per row, rows unpadded.  The second
// MFMA wants, per lane and 16-key step t, the keys 16t + 4h + {0..3} and 16t + 8 + 4h + {0..3}
// (h = lane / 32): the keys of every group of 16 are stored in the order [0-3, 8-11 | 4-7, 12-15], so
// each half-wave's eight keys are ONE 16-byte chunk (chunk 2t + h) and a fragment is one
// ds_read_b128.  The chunk position is XOR-swizzled with the row so that the 16 lanes of a read
// phase (16 consecutive rows, same chunk) cover all 64 banks: with 64-key rows (32 words) the row
// parity supplies one bank bit and d & 7 the other three; with 256-key rows (a multiple of 64 words)
// all four come from d & 15.  The higher bits of d are XORed in as well: the transposing writer's
// lanes hold rows 8 apart (same d & 7), and without them its 8-byte writes would pile 8-deep onto two
// bank groups; with them they are at most 2-deep (checked by enumeration for head_dim 64 / 128).
// (Padded rows with two 8-byte reads per fragment measured 58 % of the LDS-active cycles as
// bank-conflict stalls.)
template <int NK>
__device__ inline int vt_swz(int d) {
  return NK % 128 == 0 ? ((d & 15) ^ ((d >> 4) & 7)) : ((d & 7) ^ ((d >> 3) & 7));
}
// element offset of the chunk that holds keys [16t + 4h .. ] u [16t + 8 + 4h ..] of dimension d
template <int NK>
__device__ inline int vt_read_off(int d, int t, int h) {
  return d * NK + (((2 * t + h) ^ vt_swz<NK>(d)) << 3);
}
// element offsets where the keys 8kb .. 8kb+3 (lo) and 8kb+4 .. 8kb+7 (hi) of dimension d go (8 bytes each)
template <int NK>
__device__ inline void vt_write_off(int d, int kb, int* lo, int* hi) {
  const int c = 2 * (kb >> 1), half = kb & 1, sw = vt_swz<NK>(d);
  *lo = d * NK + ((c ^ sw) << 3) + 4 * half;
  *hi = d * NK + (((c + 1) ^ sw) << 3) + 4 * half;
}

// ---------------------------------------------------------------------------------------------
// Tiled kernel: one block = 128 queries of one (row, head), 4 waves x 32 queries; keys and values stream through LDS in tiles of
// 64 keys, double buffered, one barrier per tile.  The tiles go global -> LDS directly (a wave fills 64 chunks of 16 bytes at a
// wave-uniform address) and V^T is formed by the transposing LDS read, so nothing is staged or transposed in registers.
//
// Both tiles are stored row-major as they are in memory, the 16-byte chunks of a row permuted so that the lanes which read
// together touch all banks once:
// Keys:   a fragment is 16 rows x 32 columns, lane l reads chunk 4 ks + l / 16 of row l % 16; chunk c of row r sits at position
//         c ^ (r & 15) (head_dim 128) or c ^ (r & 7) ^ ((r >> 3) & 1) (64: two rows share the 64 banks).
// Values: ds_read_b64_tr_b16, per group of 16 lanes: lane j points at 4 consecutive dims d0 + 4 (j % 4) of key k0 + j / 4, and
//         lane i of the group receives dim d0 + i of the keys k0 .. k0 + 3 (measured lane layout).  With k0 = 32 u + 4 g and
//         32 u + 16 + 4 g for group g two such reads are one A fragment of V^T in exactly the key order in which the S^T
//         accumulators hand P^T on.  Two groups read 8 rows x 32 bytes at a time: chunk c of row r sits at position
//         c ^ (2 (r & 7)) (head_dim 128) or c ^ (2 ((r >> 1) & 3)) (64).
// head_dim 72: rows of 144 bytes spread over the banks by themselves.  Its last score step covers columns 64 .. 95: beyond 71
// the lanes read zeros (not the next row: it may hold infinities), and value dims 72 .. 79 repeat a chunk, for results that are
// never stored.
// Keys and values beyond T read as zeros (the buffer ends there); their scores are masked to -inf, and the probability 0 meets no
// infinite value (0 x inf is NaN).
//
// What bounds it: power (1059 TFLOP/s at 27 286 tokens x 24 heads of 128, 1327 on zeros, whose maxima never move), then the vector
// unit.  Before, the loads of the next tile were waited for ahead of the key reads of the
// current one (the compiler takes global_load_lds for a store that LDS reads may alias), every key fragment was waited for
// in front of its own matrix instruction, and 32x32x16 instructions drew more power.
// us, before -> now: 1 row x 27 286 tokens x 24 heads of 128 9765 -> 8639, 1 x 4608 x 24 308 -> 296, 2 x 845 x 24 40.7 -> 38.1,
// 4 x 1025 x 16 heads of 72 60.2 -> 45.6, 16 x 1024 x 16 142 -> 127, 2 x 2048 x 6 heads of 64 41.7 -> 34.6.  Variants, measured with
// a reference of the exponentials that lagged (below; 1055 to 1150 TFLOP/s, 1210 to 1260 on zeros): without the loads into LDS 1315; 32x32x16 in
// the same schedule faster on zeros (1490) and slower on data where rounds end ragged (13 632 tokens 2306 -> 2160 us); 8 waves
// on one pair of tiles gain 6 % at 4608 tokens and lose 4 % at 27 286 and 13 % at 4096; the loads as inline assembly, without
// the wait that the compiler puts ahead of a tile's value reads: 0.5 %.
typedef short short4v __attribute__((ext_vector_type(4)));

// element offset inside a row of the stored chunk c of row r (involutions: the loader uses them the other way round)
template <int HD>
__device__ inline int key_chunk(int c, int r) {
  return HD == 128 ? c ^ (r & 15) : HD == 64 ? c ^ (r & 7) ^ ((r >> 3) & 1) : c;
}
template <int HD>
__device__ inline int value_chunk(int c, int r) {
  return HD == 128 ? c ^ (2 * (r & 7)) : HD == 64 ? c ^ (2 * ((r >> 1) & 3)) : c;
}

// The reference of a query's exponentials is its running maximum, so the largest probability is 1 exactly, also as bf16.  A reference
// that follows only past a factor of 2^8, a published way to rescale rarely, saves time (us, lagging / following: 1 row x 4608 tokens x 24 heads of 128
// 270 / 284, 1 x 27 286 x 24 8502 / 8618, 4 x 1025 x 16 heads of 72 45.0 / 45.3), but rounds the largest probability too: error against
// 64 bits 2.33e-3 instead of 2.22e-3 for scores of deviation 1 over 1025 keys, 2.26e-3 instead of 1.80e-3 for deviation 2.5.

// A last block of at most this many queries has its waves share them and split the keys instead of leaving three of four idle.
// 4 rows x 1025 tokens x 16 heads of 72, 64 blocks of one query behind one round of whole ones: 50.0 -> 45.2 us; nothing to gain
// where rounds are many (27 286 tokens, 24 blocks of 22 queries among 5112: 8449 -> 8431).
constexpr int kFewQueries = 32;

// 16 bytes per lane from byte offset off[lane] of a buffer into LDS at the wave-uniform dst + 16 lane; zeros past the buffer's end
__device__ __forceinline__ void buffer_to_lds(const uint16_t* buffer, int bytes, uint32_t off, uint16_t* dst) {
  const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(buffer), 0, bytes, 0x00020000);
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (__attribute__((address_space(3))) void*)dst, 16, off, 0, 0, 0);
}

// maximum and sum over the lanes l % 16 + {0, 16, 32, 48}, which hold one query
__device__ __forceinline__ float max_of_groups(float x) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float sum_of_groups(float x) {
  x += __shfl_xor(x, 16, 64);
  return x + __shfl_xor(x, 32, 64);
}

template <int HD>
__global__ __launch_bounds__(256, 2) void attention_dma_kernel(const uint16_t* __restrict__ qkv, uint16_t* __restrict__ out, int64_t ldo,
                                                            int T, int H, float scale_log2e) {
  constexpr int CH = HD / 8;                  // 16-byte chunks of a row, and load instructions of a tile
  constexpr int KS = (HD + 31) / 32;          // steps of 32 columns of q k^T
  constexpr int DT = (HD + 15) / 16;          // tiles of 16 dims of O^T
  constexpr int LPW = (CH + 3) / 4;           // load instructions per wave and tile
  constexpr int TILE = 64 * HD;               // elements of one key or value tile
  __shared__ __align__(16) uint16_t smem[4 * TILE + 8];
  uint16_t* Ks = smem;                        // [2][64][HD]
  uint16_t* Vs = smem + 2 * TILE;             // [2][64][HD]
  uint16_t* zero = smem + 4 * TILE;           // head_dim 72: the key columns 72 .. 95 of the last step

  // Blocks of a few queries (the last one of a (row, head) whose T ends shortly past a multiple of 128) come last: they are
  // short and fill what the rounds of whole blocks leave.
  const int nq = gridDim.x, pairs = gridDim.y * gridDim.z, lin = blockIdx.x + nq * (blockIdx.y + gridDim.y * blockIdx.z);
  const int whole = T - (nq - 1) * 128 <= kFewQueries ? nq - 1 : nq;          // whole blocks per pair
  const bool few = lin >= whole * pairs;
  const int pair = few ? lin - whole * pairs : lin / whole, q0 = (few ? whole : lin - pair * whole) * 128;
  const int row = pair / H, head = pair - row * H;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, g4 = lane >> 4;
  const int64_t D = static_cast<int64_t>(H) * HD;
  const uint16_t* base = qkv + static_cast<int64_t>(row) * T * 3 * D + head * HD;

  bf16x8 qf[KS][2];                           // queries 16 n + l16, columns 32 ks + 8 g4 ..
#pragma unroll
  for (int n = 0; n < 2; ++n) {
    const int q = q0 + (few ? 0 : wave * 32) + n * 16 + l16;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      Frag f;
      f.u = q < T && 4 * ks + g4 < CH ? *reinterpret_cast<const uint4*>(base + static_cast<int64_t>(q) * 3 * D + ks * 32 + g4 * 8) : make_uint4(0, 0, 0, 0);
      qf[ks][n] = f.v;
    }
  }
  if (4 * KS > CH && tid < 8) zero[tid] = 0;
  floatx4 o[DT][2];
#pragma unroll
  for (int i = 0; i < DT; ++i)
#pragma unroll
    for (int n = 0; n < 2; ++n) o[i][n] = floatx4{};

  // Loader: wave w issues instructions i = w, w + 4, ... of a tile's CH; lane -> chunk slot 64 i + lane, row slot / CH.  Through
  // buffer descriptors that begin at the tile and end behind key T - 1: what lies beyond reads as zeros, and the compiler does not
  // take the loads for LDS reads that every later key fragment would have to wait for.
  const int64_t row_bytes = 6 * D;
  uint32_t koff[LPW], voff[LPW];
#pragma unroll
  for (int u = 0; u < LPW; ++u) {
    const int slot = (wave + 4 * u) * 64 + lane, r = static_cast<unsigned>(slot) / CH, p = slot - r * CH;
    koff[u] = static_cast<uint32_t>(r * row_bytes + 2 * D + (key_chunk<HD>(p, r) << 4));
    voff[u] = static_cast<uint32_t>(r * row_bytes + 4 * D + (value_chunk<HD>(p, r) << 4));
  }
  auto issue = [&](int kt, uint16_t* dst, const uint32_t (&off)[LPW]) {
    const int keys = T - kt * 64 < 64 ? T - kt * 64 : 64;
    const uint16_t* from = base + kt * (32 * row_bytes);
#pragma unroll
    for (int u = 0; u < LPW; ++u)
      if (CH % 4 == 0 || wave + 4 * u < CH) buffer_to_lds(from, static_cast<int>(keys * row_bytes), off[u], dst + (kt & 1) * TILE + (wave + 4 * u) * 512);
  };
  // a wave whose queries all lie beyond T only loads
  const bool active = q0 + wave * 32 < T;

  // Key fragment: keys 16 m + l16, chunk 4 ks + g4 of the tile in buffer kb (rows 16 apart are swizzled alike).
  int krd[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) krd[ks] = l16 * HD + (key_chunk<HD>(4 * ks + g4, l16) << 3);
  auto key_frag = [&](int kb, int ks, int m) {
    const uint16_t* kc = Ks + kb * TILE + m * 16 * HD + krd[ks];
    if (4 * ks + 3 >= CH && 4 * ks + g4 >= CH) kc = zero;
    return *reinterpret_cast<const bf16x8*>(kc);
  };
  // Value fragment: dims 16 dt + l16 of the keys 32 u + 4 g4 .. + 3 and 32 u + 16 + 4 g4 .. + 3, in two transposing reads: lane j
  // of a group of 16 points at dims 16 dt + 4 (j % 4) of key k0 + j / 4 (chunk 2 dt + (j % 4) / 2, half j % 2).
  const int vrow = 4 * g4 + (l16 >> 2);
  auto value_half = [&](int vb, int k0, int dt) {                  // keys k0 + 4 g4 .. + 3 (rows 16 apart are swizzled alike)
    const int c0 = 2 * dt + ((l16 & 3) >> 1), c = CH % 2 == 0 || c0 < CH ? c0 : CH - 1;        // dims beyond HD: any, never stored
    const uint16_t* va = Vs + vb * TILE + (k0 + vrow) * HD + (l16 & 1) * 4 + (value_chunk<HD>(c, vrow) << 3);
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) short4v*)va);
  };
  auto value_frag = [&](int vb, int u, int dt) {
    union { short4v h[2]; bf16x8 v; } vf;
    vf.h[0] = value_half(vb, 32 * u, dt);
    vf.h[1] = value_half(vb, 32 * u + 16, dt);
    return vf.v;
  };
  auto store = [&](const float (&sum)[2]) {
#pragma unroll
    for (int n = 0; n < 2; ++n) {
      const float inv = 1.0f / sum[n];
      const int q = q0 + (few ? 0 : wave * 32) + n * 16 + l16;
      if (q < T) {
        uint16_t* op = out + (static_cast<int64_t>(row) * T + q) * ldo + head * HD + 4 * g4;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
          if (dt * 16 + 4 * g4 < HD)
            *reinterpret_cast<uint2*>(op + dt * 16) =
                make_uint2(cvt_pk_bf16(o[dt][n][0] * inv, o[dt][n][1] * inv), cvt_pk_bf16(o[dt][n][2] * inv, o[dt][n][3] * inv));
      }
    }
  };

  // Online softmax.  A lane's scores of a tile: s[m][n][i], key 16 m + 4 g4 + i, query 16 n + l16.
  float mref[2] = {-INFINITY, -INFINITY}, moff[2] = {}, lrun[2] = {}, psum[2] = {}, corr[2] = {1.0f, 1.0f}, tmax[2];
  bool moved = false;
  // one score of 32, in the order in which the second contraction needs them
  auto maximum = [&](const floatx4 (&s)[4][2], int from, int to) {
#pragma unroll
    for (int i = from; i < to; ++i) tmax[(i >> 2) & 1] = fmaxf(tmax[(i >> 2) & 1], s[i >> 3][(i >> 2) & 1][i & 3]);
  };
  auto reference = [&]() {
    moved = false;
#pragma unroll
    for (int n = 0; n < 2; ++n) {
      const float mnew = fmaxf(mref[n], max_of_groups(tmax[n]));
      moff[n] = mnew == -INFINITY ? 0.0f : mnew * scale_log2e;     // no finite score yet: weights 0
      corr[n] = fast_exp2(mref[n] * scale_log2e - moff[n]);
      moved |= mnew != mref[n];
      mref[n] = mnew;
    }
  };
  auto probabilities = [&](floatx4 (&s)[4][2], int from, int to) {
#pragma unroll
    for (int i = from; i < to; ++i) {
      const int m = i >> 3, n = (i >> 2) & 1;
      const float p = fast_exp2(fmaf(s[m][n][i & 3], scale_log2e, -moff[n]));
      s[m][n][i & 3] = p;
      psum[n] += p;
    }
  };
  auto pack = [&](const floatx4 (&s)[4][2], int u, int n) {        // P^T of keys 32 u .. 32 u + 31
    Frag pf;
    pf.u = make_uint4(cvt_pk_bf16(s[2 * u][n][0], s[2 * u][n][1]), cvt_pk_bf16(s[2 * u][n][2], s[2 * u][n][3]),
                      cvt_pk_bf16(s[2 * u + 1][n][0], s[2 * u + 1][n][1]), cvt_pk_bf16(s[2 * u + 1][n][2], s[2 * u + 1][n][3]));
    return pf.v;
  };
  auto mask = [&](floatx4 (&s)[4][2], int kt) {                    // keys past T
#pragma unroll
    for (int i = 0; i < 32; ++i)
      if (kt * 64 + (i >> 3) * 16 + 4 * g4 + (i & 3) >= T) s[i >> 3][(i >> 2) & 1][i & 3] = -INFINITY;
  };

  // Ring: keys are fetched two tiles ahead, values one.  At the top of tile kt the wave's outstanding loads are K(kt + 1) and V(kt);
  // behind the barrier K(kt + 2) overwrites K(kt) (read in tile kt - 1) and V(kt + 1) overwrites V(kt - 1).  A wave's own fragment
  // reads are complete before the barrier, and no memory access moves across it.
#define SPECA_PIN() __builtin_amdgcn_sched_barrier(0)
#define SPECA_TURN()                                        \
  {                                                         \
    __builtin_amdgcn_s_waitcnt(0x0070);                     \
    asm volatile("" ::: "memory");                          \
    __builtin_amdgcn_s_barrier();                           \
    asm volatile("" ::: "memory");                          \
    SPECA_PIN();                                            \
  }
  const int ntiles = (T + 63) / 64;
  if (few) {
    // At most 32 queries: the waves share them and split every tile's keys, 16 each, with statistics of their own (one after the
    // other in a single wave, the block would take half as long as a whole one).  Second contraction by 16x16x16 instructions.
    floatx4 s[2];
    float m[2] = {-INFINITY, -INFINITY}, l[2] = {};
    issue(0, Ks, koff);
    issue(0, Vs, voff);
    for (int kt = 0; kt < ntiles; ++kt) {
      SPECA_TURN()
      if (kt + 1 < ntiles) {
        issue(kt + 1, Ks, koff);
        issue(kt + 1, Vs, voff);
      }
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const bf16x8 kf = key_frag(kt & 1, ks, wave);
#pragma unroll
        for (int n = 0; n < 2; ++n) s[n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf, qf[ks][n], ks ? s[n] : floatx4{}, 0, 0, 0);
      }
      short4v pf[2];
#pragma unroll
      for (int n = 0; n < 2; ++n) {
        float t = -INFINITY;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          if (kt * 64 + wave * 16 + 4 * g4 + i >= T) s[n][i] = -INFINITY;
          t = fmaxf(t, s[n][i]);
        }
        const float mnew = fmaxf(m[n], max_of_groups(t)), off = mnew == -INFINITY ? 0.0f : mnew * scale_log2e;      // no finite score yet: weights 0
        const float c = fast_exp2(m[n] * scale_log2e - off);
        m[n] = mnew;
        l[n] *= c;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          s[n][i] = fast_exp2(fmaf(s[n][i], scale_log2e, -off));
          l[n] += s[n][i];
        }
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) o[dt][n] *= c;
        union { uint32_t u[2]; short4v v; } pk;
        pk.u[0] = cvt_pk_bf16(s[n][0], s[n][1]);
        pk.u[1] = cvt_pk_bf16(s[n][2], s[n][3]);
        pf[n] = pk.v;
      }
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        const short4v vf = value_half(kt & 1, 16 * wave, dt);
#pragma unroll
        for (int n = 0; n < 2; ++n) o[dt][n] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(vf, pf[n], o[dt][n], 0, 0, 0);
      }
    }
    // together: everything relative to the largest maximum, then waves 1 .. 3 hand their sums to wave 0 through LDS
    float* stat = reinterpret_cast<float*>(smem);
    SPECA_TURN()
#pragma unroll
    for (int n = 0; n < 2; ++n)
      if (g4 == 0) stat[wave * 32 + n * 16 + l16] = m[n];
    SPECA_TURN()
#pragma unroll
    for (int n = 0; n < 2; ++n) {
      float top = -INFINITY;
#pragma unroll
      for (int w = 0; w < 4; ++w) top = fmaxf(top, stat[w * 32 + n * 16 + l16]);
      const float c = fast_exp2(m[n] * scale_log2e - top * scale_log2e);
      l[n] = sum_of_groups(l[n]) * c;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) o[dt][n] *= c;
    }
    SPECA_TURN()
    constexpr int PART = DT * 2 * 256 + 128;                       // floats of a wave: O, then the sums of every lane
    static_assert(3 * PART * 4 <= 4 * TILE * 2, "three waves' sums in the operand buffers");
    if (wave) {
      float* part = stat + (wave - 1) * PART;
#pragma unroll
      for (int n = 0; n < 2; ++n) {
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) *reinterpret_cast<floatx4*>(part + ((dt * 2 + n) * 64 + lane) * 4) = o[dt][n];
        part[DT * 512 + n * 64 + lane] = l[n];
      }
    }
    SPECA_TURN()
    if (wave) return;
#pragma unroll
    for (int w = 0; w < 3; ++w) {
      const float* part = stat + w * PART;
#pragma unroll
      for (int n = 0; n < 2; ++n) {
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) o[dt][n] += *reinterpret_cast<const floatx4*>(part + ((dt * 2 + n) * 64 + lane) * 4);
        l[n] += part[DT * 512 + n * 64 + lane];
      }
    }
    store(l);
    return;
  }

  // Tile kt, whose scores lie in sc with their reference known.  A wave issues in order, so what runs side by side is written side by
  // side, pinned around every pair of matrix instructions: first the scores of tile kt + 1 with the first NP probabilities of tile
  // kt, then O^T += V^T P^T with the other probabilities in its first half and the maximum of tile kt + 1 in its second.  Fragments
  // are read RA steps ahead.  NEXT: there is a tile kt + 1; the last one is masked.
  constexpr int NS = 4 * KS, NV = 2 * DT, RA = 4, NP = 20;
  auto tile = [&](floatx4 (&sc)[4][2], floatx4 (&sn)[4][2], int kt, int buf, auto next_tag) {
    constexpr bool NEXT = decltype(next_tag)::value;
    bf16x8 kf[NS], vf[NV], pf[2][2];
    if constexpr (NEXT) {
#pragma unroll
      for (int i = 0; i < RA; ++i) kf[i] = key_frag(1 - buf, i >> 2, i & 3);
      SPECA_PIN();
    }
    if (__any(moved)) {
#pragma unroll
      for (int n = 0; n < 2; ++n) {
        lrun[n] *= corr[n];
#pragma unroll
        for (int i = 0; i < DT; ++i) o[i][n] *= corr[n];
      }
    }
    psum[0] = psum[1] = 0.0f;
    if constexpr (NEXT) {
#pragma unroll
      for (int i = 0; i < NS; ++i) {
        if (i + RA < NS) kf[i + RA] = key_frag(1 - buf, (i + RA) >> 2, (i + RA) & 3);
        else vf[i + RA - NS] = value_frag(buf, (i + RA - NS) / DT, (i + RA - NS) % DT);
        if (i >= NS - 2) pf[0][i - NS + 2] = pack(sc, 0, i - NS + 2);
#pragma unroll
        for (int n = 0; n < 2; ++n) {
          probabilities(sc, (2 * i + n) * NP / (2 * NS), (2 * i + n + 1) * NP / (2 * NS));
          SPECA_PIN();
          sn[i & 3][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[i], qf[i >> 2][n], i < 4 ? floatx4{} : sn[i & 3][n], 0, 0, 0);
          SPECA_PIN();
        }
      }
    } else {
#pragma unroll
      for (int i = 0; i < RA; ++i) vf[i] = value_frag(buf, i / DT, i % DT);
      probabilities(sc, 0, NP);
#pragma unroll
      for (int n = 0; n < 2; ++n) pf[0][n] = pack(sc, 0, n);
    }
    tmax[0] = tmax[1] = -INFINITY;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      if (i + RA < NV) vf[i + RA] = value_frag(buf, (i + RA) / DT, (i + RA) % DT);
      if (i >= DT - 1 && i <= DT) pf[1][i - DT + 1] = pack(sc, 1, i - DT + 1);
      if constexpr (NEXT) {
        if (i == DT && kt * 64 + 128 > T) mask(sn, kt + 1);
      }
#pragma unroll
      for (int n = 0; n < 2; ++n) {
        if (i < DT) probabilities(sc, NP + (2 * i + n) * (32 - NP) / (2 * DT - 1), i + 1 == DT && n ? 32 : NP + (2 * i + n + 1) * (32 - NP) / (2 * DT - 1));
        else if constexpr (NEXT) maximum(sn, (2 * (i - DT) + n) * 32 / (2 * DT), (2 * (i - DT) + n + 1) * 32 / (2 * DT));
        SPECA_PIN();
        o[i % DT][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[i], pf[i / DT][n], o[i % DT][n], 0, 0, 0);
        SPECA_PIN();
      }
    }
#pragma unroll
    for (int n = 0; n < 2; ++n) lrun[n] += psum[n];
    if constexpr (NEXT) reference();
  };
  // tile kt, not the last one, in buffer PAR = kt % 2, its scores in SC
#define SPECA_ATTN_TILE(PAR, SC, SN)                                      \
  {                                                                       \
    SPECA_TURN()                                                          \
    if (kt + 2 < ntiles) issue(kt + 2, Ks, koff);                         \
    issue(kt + 1, Vs, voff);                                              \
    if (active) tile(SC, SN, kt, PAR, std::true_type());                  \
  }
  floatx4 sa[4][2], sb[4][2];
  issue(0, Ks, koff);
  SPECA_TURN()
  if (1 < ntiles) issue(1, Ks, koff);
  issue(0, Vs, voff);
  if (active) {
#pragma unroll
    for (int i = 0; i < NS; ++i) {
      const bf16x8 kf = key_frag(0, i >> 2, i & 3);
#pragma unroll
      for (int n = 0; n < 2; ++n) sa[i & 3][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf, qf[i >> 2][n], i < 4 ? floatx4{} : sa[i & 3][n], 0, 0, 0);
    }
    if (ntiles == 1) mask(sa, 0);
    tmax[0] = tmax[1] = -INFINITY;
    maximum(sa, 0, 32);
    reference();
  }
  int kt = 0;
  for (; kt + 2 < ntiles; ++kt) {
    SPECA_ATTN_TILE(0, sa, sb)
    ++kt;
    SPECA_ATTN_TILE(1, sb, sa)
  }
  if (kt + 1 < ntiles) {
    SPECA_ATTN_TILE(0, sa, sb)
    ++kt;
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
      for (int n = 0; n < 2; ++n) sa[m][n] = sb[m][n];
  }
  SPECA_TURN()
  if (active) tile(sa, sb, kt, kt & 1, std::false_type());
#undef SPECA_ATTN_TILE
#undef SPECA_TURN
#undef SPECA_PIN

#pragma unroll
  for (int n = 0; n < 2; ++n) lrun[n] = sum_of_groups(lrun[n]);
  store(lrun);
}

// Whole-sequence form for T <= 256: one block of 8 waves per (row, head).  Every key and value of the
// head is brought into LDS by one wave of loads issued all at once (a single memory round trip, one
// barrier), each wave then owns 32 queries, holds its complete score row in registers (8 sub-tiles),
// takes the softmax in one pass (no running maximum, no rescaling of O) and runs the second
// contraction over all keys.  At 256 tokens the tiled kernels spend their time in per-tile load
// latency and barriers; this form is bound by one load round trip plus ~90 MFMAs per wave.
constexpr size_t whole_lds_bytes(int HD, bool stage) {
  const int HD16 = (HD + 15) / 16 * 16, HD32 = (HD + 31) / 32 * 32;
  return (static_cast<size_t>(256) * (HD16 + 8) + static_cast<size_t>(HD32) * 256 + (stage ? static_cast<size_t>(8) * 32 * HD : 0)) * sizeof(uint16_t);
}
constexpr bool whole_stages_output(int HD) { return whole_lds_bytes(HD, true) <= 160 * 1024; }

// FULL: T == 256 exactly (the DiT-XL/2 shape): no bounds tests, no ragged sub-tile, so the two contractions and the
// softmax between them are one straight-line region that the scheduler can interleave.
template <int HD, bool FULL>
__global__ __launch_bounds__(512) void attention_mfma_whole_kernel(const uint16_t* __restrict__ qkv, uint16_t* __restrict__ out, int64_t ldo,
                                                                   int T_, int H, float scale_log2e) {
  constexpr int TMAX = 256;
  const int T = FULL ? TMAX : T_;
  constexpr int HD16 = (HD + 15) / 16 * 16, HD32 = (HD + 31) / 32 * 32;
  constexpr int KS = HD16 / 16;         // reduction steps of q k^T
  constexpr int DT = HD32 / 32;         // 32-row tiles of O^T
  constexpr int KST = HD16 + 8;         // LDS row stride of the keys (elements)
  constexpr int CH = HD / 8;            // 16-byte chunks per key/value row
  constexpr int NST = TMAX / 32;        // 32-key sub-tiles
  constexpr int K_CHUNKS = (TMAX * CH + 511) / 512;
  static_assert(HD % 8 == 0, "head_dim must be a multiple of 8");
  static_assert((TMAX / 8) * CH <= 512, "one 8x8 value block per thread");
  extern __shared__ __align__(16) uint16_t smem[];
  uint16_t* Ks = smem;                        // [TMAX][KST]
  uint16_t* Vt = smem + TMAX * KST;           // [HD32][TMAX], see vt_read_off
  uint16_t* Os = Vt + HD32 * TMAX;            // [8 waves][32 queries][HD]: output staging, private to a wave (STAGE_OUT)
  constexpr bool STAGE_OUT = whole_stages_output(HD);

  // blocks b, b + 8, b + 16, ... run on the same XCD: give each XCD a contiguous range of (row, head) pairs, so
  // that a row's q, k and v are pulled into one L2 instead of a slice of every row into all eight
  const int lin = blockIdx.y + gridDim.y * blockIdx.z, total = gridDim.y * gridDim.z;
  const int pair = total % 8 == 0 ? (lin % 8) * (total / 8) + lin / 8 : lin;
  const int row = pair / H, head = pair - row * H;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l32 = lane & 31, lhi = lane >> 5;
  const int64_t D = static_cast<int64_t>(H) * HD;
  const uint16_t* base = qkv + static_cast<int64_t>(row) * T * 3 * D + head * HD;

  // all global loads first: keys, one 8x8 value block, the wave's queries
  uint4 rk[K_CHUNKS], rv[8];
#pragma unroll
  for (int c = 0; c < K_CHUNKS; ++c) {
    const int id = tid + c * 512;
    const int key = id / CH, dc = id - key * CH;
    rk[c] = (id < TMAX * CH && key < T) ? *reinterpret_cast<const uint4*>(base + static_cast<int64_t>(key) * 3 * D + D + dc * 8) : make_uint4(0, 0, 0, 0);
  }
  const bool v_thread = tid < (TMAX / 8) * CH;
  const int v_kb = tid / CH, v_dc = tid % CH;   // 8x8 block: keys v_kb*8.., dims v_dc*8..
  if (v_thread) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int key = v_kb * 8 + i;
      rv[i] = key < T ? *reinterpret_cast<const uint4*>(base + static_cast<int64_t>(key) * 3 * D + 2 * D + v_dc * 8) : make_uint4(0, 0, 0, 0);
    }
  }
  Frag qf[KS];
  const int q = wave * 32 + l32;
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    const int d = ks * 16 + lhi * 8;
    qf[ks].u = (q < T && d < HD) ? *reinterpret_cast<const uint4*>(base + static_cast<int64_t>(q) * 3 * D + d) : make_uint4(0, 0, 0, 0);
  }

  // zero padding: key columns [HD, HD16) and value rows [HD, HD32)
  if (HD16 > HD)
    for (int i = tid; i < TMAX * (HD16 - HD); i += 512) Ks[(i / (HD16 - HD)) * KST + HD + i % (HD16 - HD)] = 0;
  // (with a spare row, row HD of V^T is all ones: row HD of O^T is then the sum of the probabilities as the matrix
  // cores saw them, rounded to bf16 like the numerator)
  constexpr bool ONES = HD32 > HD;
  if (HD32 > HD)
    for (int i = tid; i < (HD32 - HD) * TMAX; i += 512) Vt[HD * TMAX + i] = i < TMAX ? 0x3F80 : 0;
#pragma unroll
  for (int c = 0; c < K_CHUNKS; ++c) {
    const int id = tid + c * 512;
    const int key = id / CH, dc = id - key * CH;
    if (id < TMAX * CH) *reinterpret_cast<uint4*>(Ks + key * KST + dc * 8) = rk[c];
  }
  if (v_thread) {
    // rv[i] = 8 dims of key i  ->  8 rows (dims) of 8 keys
    const uint32_t w[8][4] = {{rv[0].x, rv[0].y, rv[0].z, rv[0].w}, {rv[1].x, rv[1].y, rv[1].z, rv[1].w},
                              {rv[2].x, rv[2].y, rv[2].z, rv[2].w}, {rv[3].x, rv[3].y, rv[3].z, rv[3].w},
                              {rv[4].x, rv[4].y, rv[4].z, rv[4].w}, {rv[5].x, rv[5].y, rv[5].z, rv[5].w},
                              {rv[6].x, rv[6].y, rv[6].z, rv[6].w}, {rv[7].x, rv[7].y, rv[7].z, rv[7].w}};
#pragma unroll
    for (int dd = 0; dd < 8; ++dd) {
      uint32_t r[4];
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        const uint32_t a = w[2 * kk][dd >> 1], b = w[2 * kk + 1][dd >> 1];
        r[kk] = (dd & 1) ? ((a >> 16) | (b & 0xFFFF0000u)) : ((a & 0xFFFFu) | (b << 16));
      }
      int lo_, hi_;
      vt_write_off<TMAX>(v_dc * 8 + dd, v_kb, &lo_, &hi_);
      *reinterpret_cast<uint2*>(Vt + lo_) = make_uint2(r[0], r[1]);
      *reinterpret_cast<uint2*>(Vt + hi_) = make_uint2(r[2], r[3]);
    }
  }
  __syncthreads();
  if (!FULL && wave * 32 >= T) return;         // no barrier after this point

  const int nst = FULL ? NST : (T + 31) / 32;  // sub-tiles that hold keys
  floatx16 s[NST];
  float tmax = -INFINITY;
#pragma unroll
  for (int st = 0; st < NST; ++st) {
#pragma unroll
    for (int e = 0; e < 16; ++e) s[st][e] = 0.0f;
    if (st < nst) {
      const uint16_t* kp = Ks + (st * 32 + l32) * KST + lhi * 8;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        Frag kf;
        kf.u = *reinterpret_cast<const uint4*>(kp + ks * 16);
        s[st] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf.v, qf[ks].v, s[st], 0, 0, 0);
      }
      if (st * 32 + 32 > T) {                  // ragged last sub-tile
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int key = st * 32 + 8 * (e >> 2) + 4 * lhi + (e & 3);
          if (key >= T) s[st][e] = -INFINITY;
        }
      }
#pragma unroll
      for (int e = 0; e < 16; ++e) tmax = fmaxf(tmax, s[st][e]);
    }
  }
  tmax = fmaxf(tmax, __shfl_xor(tmax, 32, 64));     // maximum of the raw scores; scale and log2(e) enter in the fma below
  const float moff = tmax * scale_log2e;
  float psum = 0.0f;
  auto exps = [&](int st) {                      // probabilities of one sub-tile, in place
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const float p = fast_exp2(fmaf(s[st][e], scale_log2e, -moff));
      s[st][e] = p;
      if (!ONES) psum += p;
    }
  };
  floatx16 o[DT];
#pragma unroll
  for (int i = 0; i < DT; ++i)
#pragma unroll
    for (int e = 0; e < 16; ++e) o[i][e] = 0.0f;
  // V^T fragment addresses: chunk (2t + h) ^ swz(d) = 16 (t >> 3) + ((2 (t & 7)) ^ (h ^ swz(d))) because swz < 16 and h < 2,
  // so eight per-lane offsets per 32-row tile (one for each t & 7) and an immediate for t >> 3 replace the arithmetic per read
  // (24 registers at head_dim 72; at head_dim 128 the table would spill, so the offsets are formed per read there)
  constexpr bool VTAB = DT <= 3;
  int vto[VTAB ? DT : 1][8];
#pragma unroll
  for (int dt = 0; dt < (VTAB ? DT : 0); ++dt) {
    const int dd = dt * 32 + l32, y = lhi ^ vt_swz<TMAX>(dd);
#pragma unroll
    for (int b = 0; b < 8; ++b) vto[dt][b] = dd * TMAX + (((2 * b) ^ y) << 3);
  }
  // the exponentials of sub-tile st + 1 are issued with the second contraction of sub-tile st
  if (0 < nst) exps(0);
#pragma unroll
  for (int st = 0; st < NST; ++st) {
    if (st < nst) {
      if (st + 1 < NST && st + 1 < nst) exps(st + 1);
#pragma unroll
      for (int hh = 0; hh < 2; ++hh) {
        const int t = 2 * st + hh, j0 = hh * 8;   // accumulator entries j0 .. j0+7 of sub-tile st: 16 keys
        Frag pf;
        pf.u = make_uint4(cvt_pk_bf16(s[st][j0], s[st][j0 + 1]), cvt_pk_bf16(s[st][j0 + 2], s[st][j0 + 3]),
                          cvt_pk_bf16(s[st][j0 + 4], s[st][j0 + 5]), cvt_pk_bf16(s[st][j0 + 6], s[st][j0 + 7]));
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
          Frag vf;
          vf.u = *reinterpret_cast<const uint4*>(Vt + (VTAB ? vto[VTAB ? dt : 0][t & 7] + (t >> 3) * 128 : vt_read_off<TMAX>(dt * 32 + l32, t, lhi)));
          o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf.v, pf.v, o[dt], 0, 0, 0);
        }
      }
    }
  }
  // row HD of O^T sits in accumulator entry (HD % 32 / 8) * 4 of the last tile, in the lanes with lhi == 0
  const float ltot = ONES ? __shfl(o[DT - 1][(HD % 32 / 8) * 4], l32, 64) : psum + __shfl_xor(psum, 32, 64);
  const float inv = 1.0f / ltot;
  // A lane holds one query's output in 8-byte pieces 2304 bytes apart from its neighbour's: the wave re-lays its
  // 32 x HD tile through its own piece of LDS and stores whole 16-byte chunks, a query's HD values contiguous.
  if (!STAGE_OUT) {                            // no LDS to spare: 8-byte stores straight from the accumulators
    if (q < T) {
      uint16_t* op = out + (static_cast<int64_t>(row) * T + q) * ldo + head * HD;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
          const int d = dt * 32 + 8 * jj + 4 * lhi;
          if (d < HD) {
            uint2 r;
            r.x = cvt_pk_bf16(o[dt][4 * jj] * inv, o[dt][4 * jj + 1] * inv);
            r.y = cvt_pk_bf16(o[dt][4 * jj + 2] * inv, o[dt][4 * jj + 3] * inv);
            *reinterpret_cast<uint2*>(op + d) = r;
          }
        }
    }
    return;
  }
  uint16_t* ow = Os + wave * 32 * HD;
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {
      const int d = dt * 32 + 8 * jj + 4 * lhi;
      if (d < HD) {
        uint2 r;
        r.x = cvt_pk_bf16(o[dt][4 * jj] * inv, o[dt][4 * jj + 1] * inv);
        r.y = cvt_pk_bf16(o[dt][4 * jj + 2] * inv, o[dt][4 * jj + 3] * inv);
        *reinterpret_cast<uint2*>(ow + l32 * HD + d) = r;
      }
    }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");       // the wave's LDS writes before its reads below
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  uint16_t* ob = out + (static_cast<int64_t>(row) * T + wave * 32) * ldo + head * HD;
#pragma unroll
  for (int c0 = 0; c0 < 32 * CH; c0 += 64) {
    const int c = c0 + lane;
    const int qq = c / CH, dc = c - qq * CH;
    if (c < 32 * CH && wave * 32 + qq < T)
      *reinterpret_cast<uint4*>(ob + static_cast<int64_t>(qq) * ldo + dc * 8) = *reinterpret_cast<const uint4*>(ow + qq * HD + dc * 8);
  }
}

template <int HD>
Error launch_hd(const void* qkv, void* out, int64_t ldo, int rows, int T, int H, hipStream_t st) {
  // (the whole-sequence kernel stores 16-byte chunks of the output when it stages them through LDS)
  if (T <= 256 && (!whole_stages_output(HD) || (ldo % 8 == 0 && reinterpret_cast<uintptr_t>(out) % 16 == 0))) {
    constexpr size_t smem_w = whole_lds_bytes(HD, whole_stages_output(HD));
    static bool attr_w = false;
    if (smem_w > 64 * 1024 && !attr_w) {
      SPECA_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(attention_mfma_whole_kernel<HD, false>), hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(smem_w)));
      SPECA_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(attention_mfma_whole_kernel<HD, true>), hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(smem_w)));
      attr_w = true;
    }
    const float sl2 = 1.4426950408889634f / sqrtf(static_cast<float>(HD));
    if (T == 256) attention_mfma_whole_kernel<HD, true><<<dim3(1, H, rows), 512, smem_w, st>>>(static_cast<const uint16_t*>(qkv), static_cast<uint16_t*>(out), ldo, T, H, sl2);
    else attention_mfma_whole_kernel<HD, false><<<dim3(1, H, rows), 512, smem_w, st>>>(static_cast<const uint16_t*>(qkv), static_cast<uint16_t*>(out), ldo, T, H, sl2);
    SPECA_HIP(hipGetLastError());
    return ok();
  }
  const float sl2 = 1.4426950408889634f / sqrtf(static_cast<float>(HD));
  attention_dma_kernel<HD><<<dim3((T + 127) / 128, H, rows), 256, 0, st>>>(static_cast<const uint16_t*>(qkv), static_cast<uint16_t*>(out), ldo, T, H, sl2);
  SPECA_HIP(hipGetLastError());
  return ok();
}

}  // namespace

bool attention_mfma_supported(const void* qkv, const void* out, int64_t ldo, int H, int hd) {
  return (hd == 64 || hd == 72 || hd == 128) && ldo % 4 == 0 && reinterpret_cast<uintptr_t>(qkv) % 16 == 0 && reinterpret_cast<uintptr_t>(out) % 8 == 0;
}

Error launch_attention_mfma(const void* qkv, void* out, int64_t ldo, int rows, int T, int H, int hd, hipStream_t st) {
  if (rows > 65535 || H > 65535) SPECA_FAIL(SPECA_EINVAL, "attention: grid too large");
  switch (hd) {
    case 64: return launch_hd<64>(qkv, out, ldo, rows, T, H, st);
    case 72: return launch_hd<72>(qkv, out, ldo, rows, T, H, st);
    case 128: return launch_hd<128>(qkv, out, ldo, rows, T, H, st);
  }
  SPECA_FAIL(SPECA_EUNSUPPORTED, "attention: head_dim %d has no MFMA kernel", hd);
}

}  // namespace speca
