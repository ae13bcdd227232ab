// Projection GEMMs of the DiT block: tile-configuration table, planner and
// dispatch for the MFMA kernels of gemm_tile.h (bf16, and float32 for the
// float32 mode).
#include "gemm_tile.h"

namespace wam {

namespace {

using gemm::launch_tile;
using gemm::launch_tile_f32;

// ---------------------------------------------------------------- configs
// Tile shapes of the bf16 kernel and what a tile costs.  A CU that holds c
// blocks at once (c <= occ) finishes them in about K / 64 * per[c-1] +
// fix[c-1] us; the constants are least-squares fits to timings of every
// configuration at the four projections of 57 model sizes (64 to 12000 rows,
// D 256 to 2048), standard deviation 7-12%.  What they show: 256-column tiles
// over 8 waves do the most work per byte loaded and win where their blocks
// fill whole rounds of the 256 CUs; 128-column tiles over 4 waves leave room
// for two blocks per CU, whose barriers and epilogues overlap, and waste less
// in the last round; small tiles spread short sequences over the chip, where
// a launch costs ~3 us whatever it does.
struct TileCfg {
  int bm, bn, wgm, wgn, st, bk;  // rows x columns, waves (rows x columns), LDS stages, K per stage
  int occ;
  float per[3], fix[3];
};
constexpr TileCfg kCfgs[] = {
    {256, 256, 2, 4, 2, 64, 1, {1.38f}, {7.85f}},
    {320, 256, 2, 4, 2, 64, 1, {1.70f}, {8.28f}},
    {192, 256, 2, 4, 2, 64, 1, {1.10f}, {7.13f}},
    {160, 128, 2, 2, 2, 64, 2, {0.67f, 1.01f}, {4.73f, 8.28f}},
    {128, 128, 2, 2, 2, 64, 2, {0.56f, 0.87f}, {4.24f, 6.95f}},
    {96, 128, 2, 2, 2, 64, 2, {0.50f, 0.74f}, {3.74f, 5.40f}},
    {64, 128, 2, 2, 3, 64, 2, {0.33f, 0.57f}, {3.89f, 4.31f}},
    {96, 64, 2, 2, 3, 64, 2, {0.27f, 0.46f}, {3.38f, 3.56f}},
    {64, 64, 2, 2, 4, 64, 2, {0.19f, 0.37f}, {3.14f, 2.39f}},
    {32, 128, 2, 2, 4, 64, 2, {0.22f, 0.43f}, {3.45f, 2.77f}},
    {32, 64, 2, 2, 4, 64, 3, {0.14f, 0.24f, 0.39f}, {2.78f, 2.94f, 1.94f}},
    {32, 64, 2, 1, 4, 64, 3, {0.20f, 0.26f, 0.38f}, {3.18f, 3.62f, 2.20f}},
    {32, 32, 2, 2, 4, 128, 2, {0.10f, 0.16f}, {2.90f, 3.00f}},
};
constexpr int kNumCfgs = sizeof(kCfgs) / sizeof(kCfgs[0]);

template <int C>
hipError_t launch_c(const GemmArgs& a, hipStream_t s) {
  constexpr TileCfg t = kCfgs[C];
  return launch_tile<t.bm, t.bn, t.wgm, t.wgn, t.st, t.bk>(a, s);
}

template <int... C>
hipError_t launch_any(const GemmArgs& a, int cfg, hipStream_t s, std::integer_sequence<int, C...>) {
  hipError_t e = hipErrorInvalidValue;
  ((cfg == C ? (void)(e = launch_c<C>(a, s)) : (void)0), ...);
  return e;
}

double tile_cost(const TileCfg& t, int M, int N, int K) {
  const long blocks = (long)((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn);
  const long n = (blocks + 255) / 256;  // blocks of the busiest CU
  const double stages = K / 64.0;
  const int rem = (int)(n % t.occ);
  double c = (double)(n / t.occ) * (stages * t.per[t.occ - 1] + t.fix[t.occ - 1]);
  if (rem) c += stages * t.per[rem - 1] + t.fix[rem - 1];
  return c;
}

// Configuration of the smallest cost.  Over those sizes its choice is 1.3%
// slower than the fastest configuration on average (21% at worst, on a 5 us
// launch); the fixed rules it replaced, with tiles that had to divide N, were
// 22% slower on average, e.g. N = 1216, M = 5754: 41 -> 26 us (K = 1216) and
// 122 -> 74 us (K = 4864).
int plan_gemm(int M, int N, int K, int epi) {
  int best = -1;
  double bc = 0.0;
  for (int c = 0; c < kNumCfgs; ++c) {
    const TileCfg& t = kCfgs[c];
    // the QKV epilogue needs whole heads (64 columns) per wave
    if (K % t.bk || (epi == EPI_QKV && (t.bn / t.wgn) % 64)) continue;
    const double v = tile_cost(t, M, N, K);
    if (best < 0 || v < bc) best = c, bc = v;
  }
  return best;
}

// ---------------------------------------------------------------- fp32
// The fp32 matrix rate (157 TFLOP/s, a sixteenth of bf16) leaves loads and
// LDS far from their limits at any tile, so the tile only has to spread the
// work evenly: 64x64 where the last wave of blocks costs less than the better
// balance of 32-row or 32x32 tiles (counted as the tile area of the busiest
// CU; the small tiles pay ~10% for their shorter MFMA runs).  One wave column
// of 64 where a wave has to own whole heads (QKV epilogue).
// Small model, M = 864, against 64x64 tiles on the vector pipe (15-20
// TFLOP/s): QKV 65 -> 36 us, attention output 58 -> 16, MLP-up 79 -> 52,
// MLP-down 214 -> 52.
hipError_t launch_gemm_f32(const GemmArgs& a, hipStream_t s) {
  if (a.K % 32 || a.N % 64) return hipErrorInvalidValue;
  auto cost = [&](int bm, int bn, double per) {
    const long blocks = (long)((a.M + bm - 1) / bm) * (a.N / bn);
    return (double)((blocks + 255) / 256) * bm * bn * per;
  };
  const double c64 = cost(64, 64, 1.0);
  if (a.epi == EPI_QKV)
    return cost(32, 64, 1.05) < c64 ? launch_tile_f32<32, 64, 2, 1, 4, 32>(a, s)
                                    : launch_tile_f32<64, 64, 4, 1, 3, 32>(a, s);
  return cost(32, 32, 1.1) < c64 ? launch_tile_f32<32, 32, 2, 2, 4, 32>(a, s)
                                 : launch_tile_f32<64, 64, 2, 2, 3, 32>(a, s);
}

}  // namespace

hipError_t launch_gemm(const GemmArgs& a, bool bf16_mode, hipStream_t s) {
  if (a.M <= 0) return hipSuccess;
  if (bf16_mode) {
    if (a.N % 64) return hipErrorInvalidValue;  // ragged column tiles end on a wave's columns
    return launch_any(a, plan_gemm(a.M, a.N, a.K, a.epi), s, std::make_integer_sequence<int, kNumCfgs>{});
  }
  return launch_gemm_f32(a, s);
}

}  // namespace wam
