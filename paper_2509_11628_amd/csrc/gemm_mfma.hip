// The choice of the tile for every bf16 GEMM (256x256: gemm_phase.hip, others 128 wide: gemm_duo.hip, small and middle tiles and tails of
// K: gemm_ring.hip).
//
// What the kernels share.  Operand roles: the weight rows are the MFMA "A" operand and the token rows the "B" operand, i.e. the
// instruction produces a tile of C^T.  A lane then owns, for one token, consecutive output features, which is what the epilogues
// want (16-byte accesses to C, the cache and the residual stream).  K is walked in order by every tile shape, so an output element is
// the same fp32 sequence regardless of M, of the tile shape and of which rows share the launch.  Tiles are numbered so that the 8 XCDs
// (round-robin block dispatch) each work on a contiguous range of tiles that share activations in their own L2.
#include <algorithm>
#include <cmath>

#include "lane_epilogue.h"

namespace speca {

namespace {

constexpr int BK = 64;

}  // namespace

// Fourteen kernels can run a given problem; which is fastest depends on how the tile count falls on the chip's compute
// units more than on anything else (a 270-tile launch of one-block-per-CU tiles takes two rounds, a 252-tile one
// takes one), and the row count M varies from call to call: per-sample rejection sends any number of guidance pairs
// to the full pass.  So the choice is made by a small cost model instead of thresholds fitted to particular shapes:
//     time(kernel) = a + (c + b * ceil(K / 64)) * rounds,     depth = ceil(tiles / compute units),
//     rounds = 1 + r * (depth - 1), or with two blocks on a compute unit  floor(depth / 2) * (1 + r) + depth % 2
// a: launch; c: prologue and epilogue; b: one 64-wide K-step; r: what a further round, or the second block, costs.  Fitted to
// 800 problems with cold weights (16 to 27 286 rows, the layers of 384 to 3072 features and random sizes, K from 64 on, tails of K; layers below 10 us
// inside captured graphs, where the host's launch does not count), so that the time of the kernels picked is least (1.0 % above the best kernel of
// each on the mean) and the times themselves fit (7 to 13 % rms).
// c and r of the plain stores were then corrected on 1300 layers above 9.5 us, half of them with K below 800, for which that fit's picks had been
// up to 22 % slower than the kinds and table before it.  On 412 other layers 0.993 of the time on the mean (0.55 to 1.07, read-ahead's limits
// included), and those more than 5 % slower than before that fit are 7 instead of 14.  us, its pick / now:
// 1781 x 3456 x 384 13.7 / 11.1 (128x128 / 256x128), 5649 x 3456 x 256 30.1 / 24.9 (128x192 / split), 21616 x 3456 x 64 53.9 / 48.5 (128x192 / 256x256),
// 628 x 9216 x 384 13.8 / 11.3 (128x128 / 256x128), 6578 x 3072 x 96 23.7 / 22.2 (128x192 / 128x128).
// The branch epilogue (residual read and written in fp32, cache planes) is two to four times as long as a plain store, so c and r have
// second values for it, fitted to 170 reference steps of 4 blocks (384 to 3072 features, 200 to 51 200 rows, both cache layouts), each of
// them with its branch layers on every kind: the picks cost 0.4 % of a step on the mean (13 % at worst: planes of differences).
// 192x192 is not offered to it.
// Against the table, tiles and row groups before gemm_duo.hip, the loader waves and read_ahead: reference steps at 150 sizes take 0.92 of the time
// on the mean (0.76 to 1.06), 800 layers 0.91.
struct TileKind {
  int bm, bn;
  float a, c, b, r;    // three in microseconds, a ratio
  float cb, rb;        // c and r under the branch epilogue (cb = 0: not offered to it)
  bool two;            // two blocks fit on a compute unit
  bool whole_steps;    // K % 64 == 0
};
constexpr TileKind kTileKinds[] = {
    {256, 256, 3.5f, 5.86f, 1.096f, 1.12f, 16.4f, 0.76f, false, true},       // 0: phases (gemm_phase.hip)
    {256, 128, 5.3f, 3.34f, 0.597f, 1.23f, 7.6f, 1.05f, false, true},        // 1: two groups (gemm_duo.hip)
    {128, 128, 3.2f, 2.55f, 0.504f, 1.24f, 7.7f, 0.96f, false, false},       // 2: ring of 4 stages x 64 columns
    {128, 128, 3.8f, 2.54f, 0.760f, 0.36f, 8.5f, 0.11f, true, false},        // 3: ring of 2 x 64
    {128, 64, 0.6f, 2.88f, 0.348f, 1.02f, 5.5f, 0.92f, false, false},        // 4: ring of 3 x 128
    {64, 64, 1.0f, 2.12f, 0.216f, 1.03f, 4.4f, 0.88f, false, false},         // 5: ring of 3 x 128
    {32, 64, 0.6f, 2.54f, 0.208f, 0.91f, 4.4f, 0.77f, false, false},         // 6: ring of 4 x 128, two waves
    {192, 128, 2.7f, 4.12f, 0.669f, 1.11f, 17.7f, 0.95f, false, false},      // 7: ring of 3 x 64
    {128, 192, 2.3f, 4.20f, 1.025f, 0.33f, 9.4f, 0.11f, true, false},        // 8: ring of 2 x 64
    {192, 192, 4.6f, 7.16f, 0.900f, 1.12f, 0.0f, 0.00f, false, false},       // 9: ring of 3 x 64
    {96, 128, 0.4f, 4.40f, 0.476f, 1.03f, 11.4f, 0.78f, false, false},       // 10: ring of 4 x 64
    {64, 128, 0.5f, 2.46f, 0.361f, 1.00f, 3.5f, 0.90f, false, true},         // 11: two groups
    {128, 128, 0.0f, 3.15f, 0.455f, 1.30f, 6.9f, 0.96f, false, true},        // 12: two groups
    {192, 128, 3.2f, 3.82f, 0.522f, 1.20f, 8.2f, 1.04f, false, true},        // 13: two groups
};
constexpr int kKinds = sizeof(kTileKinds) / sizeof(kTileKinds[0]);

int compute_units() {
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

// Idle units read ahead (gemm_tile.h) where they are enough to stay ahead of the tiles; readers that fall behind fetch what the tiles have
// fetched already and take HBM from them.  A unit reads about 56 bytes per ns from HBM.  Tiles of 128 features pass 64 columns of all N rows
// of W in 0.36 to 0.6 us, 0.2 to 0.35 N bytes per ns: N / 128 units.  Those of 64 features take 0.21 to 0.35 us: N / 88 units, and N / 128 up to
// 4096 features, where tiles and readers together stay below what HBM gives.  32x64, with next to no activations to wait for, takes 0.13
// once its weights are near: N / 32, and N / 40 up to 4096 features (of 65 rows and more then: 3456 features with 88 idle units 0.98 on the mean of 15
// layers, 1536 with 40 0.97 of 11, 285 x 1536 x 7680 27.9 without and 25.5 with; 3072 with 64, N / 48, 1.01, 2304 with 40, N / 58, 1.07; 6144 with
// 160, N / 38, 1.08).  us with read-ahead / without, cold weights, out of 800 layers of 1 to 8192 rows: 32x64 39 x 6144 x 8192
// (64 idle units) 51.7 / 28.6, 94 x 4608 x 4608 (40) 34.2 / 19.3, 8 x 8192 x 4608 (128) 23.7 / 18.3, but 28 x 3072 x 4608 (208) 0.88 of the time,
// 91 x 3072 x 12288 (112) 0.77; 64x64 186 x 4608 x 8192 (40) 38.4 / 36.9, 162 x 3456 x 4392 (88) 0.82; 128x64 143 x 6144 x 8192 (64) 49.6 / 42.2,
// 332 x 3456 x 8192 (88) 0.88, 1280 x 1536 x 6144 (16) 0.89; 128x128 460 x 6144 x 4608 (64) 0.87.  Rows of exactly 16 KB gain least everywhere
// (0.87 to 1.1: all readers of a column meet in few channels).
// Below K = 768 the tiles have most of it on its way from the start; above N = 8192, for 128x128 above 6144, they draw what HBM gives
// (with / without 16 x 9216 x 3072 17.9 / 14.8, 298 x 8192 x 16384 on 128x128 142 / 124; twelve such layers of 7168 to 8192 features 1.04 on the mean).
// A launch of two streams reads two matrices with these units and the same limit: twice the units asked for would be 0.1 % faster on the mean
// over 70 reference steps of dual blocks where it matters (0.95 to 1.03).
unsigned launch_blocks(int bm, int bn, int tiles_m, int tiles_n, const Operands& o, const GemmEpi& epi) {
  const int held = tile_blocks(tiles_m, tiles_n), idle = compute_units() - held;
  const int64_t reach = static_cast<int64_t>(idle) * (bm == 32 ? (o.N > 4096 ? 32 : 40) : bn == 64 && o.N > 4096 ? 88 : 128);
  if (epi.beside || o.K < 768 || reach < o.N || o.N > (bm == 128 && bn == 128 ? 6144 : 8192)) return static_cast<unsigned>(held);
  return static_cast<unsigned>(held + std::min<int64_t>(idle, static_cast<int64_t>(o.N) * o.K >> 15));      // 64 KB each at least
}

// `paired`: two such layers run side by side, so their tiles fill each other's partial rounds
static double tile_cost(const TileKind& t, bool branch, double tiles, int K, bool paired) {
  if (paired) {
    const double depth = std::max(1.0, 2.0 * tiles / compute_units()), c = branch ? t.cb : t.c, r = branch ? t.rb : t.r;
    const double rounds = t.two && depth >= 2.0 ? depth / 2 * (1.0 + r) : 1.0 + r * (depth - 1.0);
    return t.a + (c + t.b * ((K + BK - 1) / BK)) * rounds;
  }
  const double depth = std::ceil(tiles / compute_units());
  const double odd = std::fmod(depth, 2.0);
  const double c = branch ? t.cb : t.c, r = branch ? t.rb : t.r;
  const double rounds = t.two ? (depth - odd) / 2 * (1.0 + r) + odd : 1.0 + r * (depth - 1.0);
  return t.a + (c + t.b * ((K + BK - 1) / BK)) * rounds;
}

static double tiles_of(const TileKind& t, int M, int N) { return static_cast<double>((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn); }

// Whether a kind can run the problem.  The rings hold a row's place inside the tile as a 32-bit byte offset, which bounds the
// stride of the rows (11 million elements for the tallest tile); the others hold it in 32 bits from a buffer's base.
static bool tile_fits(const TileKind& t, const Operands& o) {
  if (t.whole_steps) return gemm_phase_fits(o);
  constexpr int64_t kReach = (int64_t{1} << 31) - 128;               // elements, less a row's own 256 bytes
  return (std::min(t.bm, o.M) - 1) * o.lda < kReach && (std::min(t.bn, o.N) - 1) * o.ldw < kReach;
}

// cheapest eligible kernel for the problem (-1: none); *cost receives its modelled time
static int pick_tile(const Operands& o, bool branch, bool paired, double* cost) {
  int best = -1;
  double bc = 0.0;
  for (int k = 0; k < kKinds; ++k) {
    const TileKind& t = kTileKinds[k];
    if (!tile_fits(t, o) || (branch && t.cb == 0.0f)) continue;
    const double c = tile_cost(t, branch, tiles_of(t, o.M, o.N), o.K, paired);
    if (best < 0 || c < bc) { best = k; bc = c; }
  }
  *cost = bc;
  return best;
}

static Error launch_kind(int kind, const Operands& o, const GemmEpi& epi, hipStream_t st) {
  switch (kind) {
    case 0: return launch_gemm_phase(o, epi, st);
    case 1: return launch_gemm_duo(256, o, epi, st);
    case 11: case 12: case 13: return launch_gemm_duo(64 * (kind - 10), o, epi, st);
    default: return launch_gemm_ring(kind - 2, o, epi, st);
  }
}

bool gemm_mfma_supported(const Operands& o) {
  double cost = 0.0;
  return (o.K % 8 == 0) && (o.lda % 8 == 0) && (o.ldw % 8 == 0) && (o.N % 4 == 0) && (reinterpret_cast<uintptr_t>(o.a) % 16 == 0) &&
         (reinterpret_cast<uintptr_t>(o.w) % 16 == 0) && pick_tile(o, true, false, &cost) >= 0;     // the smallest tile, which fits whenever one does, serves every epilogue
}

// How a layer is run: all of it on one kind, or `head` columns ahead on the 256x256 tile and the rest on `kind`.
struct Choice {
  int kind;
  int head;
  double time;
};
// What a second launch costs beyond the two modelled times, in microseconds.  Over 220 layers that the model would split without it, splits of
// layers under 40 us lost 5 % on the mean (7000 x 3072 x 192 21.2 -> 23.1 us); with it 156 are split, 6 % faster on the mean and one of them
// slower by more than 2 %, and the choice lies 0.1 % above the better form of each on the mean (0.9 % without).  It is part of the layer's time, which
// the choices of row groups and of streams weigh: dual blocks of 34 sizes where that decides 0.5 % faster on the mean (4 % to -2.6 %; 2 rows x (1312 + 40)
// tokens x 3072 features, 4 blocks, 4440 -> 4267 us).
constexpr double kSecondLaunch = 4.0;
static Choice choose(const Operands& o, bool branch, bool paired) {
  Choice c{-1, 0, 0.0};
  c.kind = pick_tile(o, branch, paired, &c.time);
  if (paired) return c;
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
      const int kind = pick_tile(tail, false, false, &rest);
      rest += tile_cost(kTileKinds[0], false, tiles_of(kTileKinds[0], o.M, n1), o.K, false) + kSecondLaunch;
      if (rest < (c.head ? 1.0 : 0.96) * c.time) c = {kind, n1, rest};
    }
  }
  return c;
}

double layer_time(bool branch, int M, int N, int K, bool paired) {
  const Operands o{nullptr, K, nullptr, K, M, N, K};
  return choose(o, branch, paired).time;
}

Error launch_gemm_mfma(const Operands& o, const GemmEpi& epi, hipStream_t st) {
  const Choice c = choose(o, epi.mode == EPI_BRANCH, epi.beside);
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

// One launch for both streams against a launch per row and stream, us per pass: 2 rows x (768 + 77 tokens) x 3072 features, 6 blocks of which 2
// are dual, 8 steps 12 860 -> 11 330; 3 rows x (256 + 40) x 1024, 5 blocks, 3 dual, 6 steps 2962 -> 1939; 2 x (750 + 333) x 1536, 5 blocks, 4 dual,
// 6 steps 4751 -> 3597; 1 row x (4096 + 512) x 3072, 57 blocks, 19 dual, 10 steps 216.6 -> 212.6 ms; 1 x (27 030 + 256) x 3072 221.1 -> 221.6 ms.
int pick_streams(const Operands& o, const StreamLayer& y, bool branch) {
  const auto side_ok = [](const void* w) { return w && reinterpret_cast<uintptr_t>(w) % 16 == 0; };
  if (o.N % 4 || o.lda % 8 || o.ldw % 8 || reinterpret_cast<uintptr_t>(o.a) % 16 || !side_ok(y.w[0]) || !side_ok(y.w[1]) || !gemm_phase_fits(o) ||
      static_cast<int64_t>(y.rows) * y.tokens >= (int64_t{1} << 31) / o.lda)                 // byte offsets inside a tile: 32 bits
    return -1;
  double separate = 0.0, best = 0.0;
  for (int s = 0; s < 2; ++s) {
    Operands one = o;
    one.M = y.len[s];
    separate += y.rows * choose(one, branch, false).time;
  }
  int kind = -1;
  for (int k = 0; k < kKinds; ++k) {
    const TileKind& t = kTileKinds[k];
    if (!t.whole_steps) continue;
    const double c = tile_cost(t, branch, tiles_of(t, y.rows * y.len[0], o.N) + tiles_of(t, y.rows * y.len[1], o.N), o.K, false);
    if (kind < 0 || c < best) { kind = k; best = c; }
  }
  return best < separate ? kind : -1;
}

Error launch_gemm_mfma_streams(int kind, const Operands& o, const StreamLayer& y, const GemmEpi& epi, hipStream_t st) {
  Operands first = o;
  first.w = y.w[0];
  GemmEpi e = epi;
  e.bias = y.bias[0];
  e.gate = y.gate[0];
  const TwoStreams streams{y.w[1], y.bias[1], y.gate[1], 0, y.rows, y.tokens, y.len[0], y.off[0], y.len[1], y.off[1]};
  const TileKind& t = kTileKinds[kind];
  return t.bn == 256 ? launch_gemm_phase_streams(first, e, streams, st) : launch_gemm_duo_streams(t.bm, first, e, streams, st);
}

}  // namespace speca
