// Projection GEMMs of the DiT block: tile-configuration table, planner and
// dispatch for the MFMA kernels of gemm_tile.h (bf16, and float32 for the
// float32 mode).
#include "gemm_tile.h"

namespace wam {

namespace {

using gemm::launch_tile;
using gemm::launch_tile_f32;

// ---------------------------------------------------------------- configs
// Tile shapes and what a tile costs.  A CU that holds c
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
  float per[4], fix[4];
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

// float32 operands: the fp32 matrix rate (157 TFLOP/s, a sixteenth of bf16)
// leaves loads and LDS far from their limits at any tile, so the tile has to
// spread the work evenly; large ones run their MFMAs with fewer gaps (96x128
// at 80% of the rate, 32x32 at 60%).  Same cost form, fitted at 39 sizes (64
// to 6000 rows, D 64 to 1024; standard deviation 3-8%): the choice is 0.5%
// off the fastest on average.  M = 864, D = 768 on the vector pipe before:
// QKV 65 -> 31 us, attention output 58 -> 15, MLP-up 79 -> 43, MLP-down 214 ->
// 48.
constexpr TileCfg kF32Cfgs[] = {
    {128, 128, 2, 2, 2, 32, 1, {4.01f}, {4.4f}},
    {96, 128, 2, 2, 3, 32, 1, {3.04f}, {4.3f}},
    {64, 128, 2, 2, 3, 32, 2, {2.11f, 4.34f}, {4.0f, 6.4f}},
    {64, 64, 2, 4, 3, 32, 3, {1.11f, 2.13f, 3.37f}, {3.0f, 4.8f, 1.5f}},
    {32, 32, 2, 2, 4, 32, 3, {0.42f, 0.65f, 0.92f}, {2.5f, 2.9f, 1.6f}},
    {16, 64, 1, 1, 4, 32, 4, {1.10f, 1.14f, 1.21f, 1.27f}, {3.1f, 3.4f, 3.6f, 2.5f}},
};
constexpr int kNumF32Cfgs = sizeof(kF32Cfgs) / sizeof(kF32Cfgs[0]);

template <int C>
hipError_t launch_f32(const GemmArgs& a, hipStream_t s) {
  constexpr TileCfg t = kF32Cfgs[C];
  return launch_tile_f32<t.bm, t.bn, t.wgm, t.wgn, t.st, t.bk>(a, s);
}

template <int... C>
hipError_t launch_any(const GemmArgs& a, int cfg, hipStream_t s, std::integer_sequence<int, C...>) {
  hipError_t e = hipErrorInvalidValue;
  ((cfg == C ? (void)(e = launch_c<C>(a, s)) : (void)0), ...);
  return e;
}

template <int... C>
hipError_t launch_any_f32(const GemmArgs& a, int cfg, hipStream_t s, std::integer_sequence<int, C...>) {
  hipError_t e = hipErrorInvalidValue;
  ((cfg == C ? (void)(e = launch_f32<C>(a, s)) : (void)0), ...);
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

// Configuration of the smallest cost.  Over the bf16 sizes its choice is 1.3%
// slower than the fastest configuration on average (21% at worst, on a 5 us
// launch); the fixed rules it replaced, with tiles that had to divide N, were
// 22% slower on average, e.g. N = 1216, M = 5754: 41 -> 26 us (K = 1216) and
// 122 -> 74 us (K = 4864).
template <int NC>
int plan_gemm(const TileCfg (&cfgs)[NC], int M, int N, int K, int epi) {
  int best = -1;
  double bc = 0.0;
  for (int c = 0; c < NC; ++c) {
    const TileCfg& t = cfgs[c];
    // the QKV epilogue needs whole heads (up to 64 columns) per wave
    if (K % t.bk || (epi == EPI_QKV && (t.bn / t.wgn) % 64)) continue;
    const double v = tile_cost(t, M, N, K);
    if (best < 0 || v < bc) best = c, bc = v;
  }
  return best;
}

}  // namespace

hipError_t launch_gemm(const GemmArgs& a, bool bf16_mode, hipStream_t s) {
  if (a.M <= 0) return hipSuccess;
  if (a.N % 64) return hipErrorInvalidValue;  // ragged column tiles end on a wave's columns
  if (bf16_mode)
    return launch_any(a, plan_gemm(kCfgs, a.M, a.N, a.K, a.epi), s, std::make_integer_sequence<int, kNumCfgs>{});
  return launch_any_f32(a, plan_gemm(kF32Cfgs, a.M, a.N, a.K, a.epi), s,
                        std::make_integer_sequence<int, kNumF32Cfgs>{});
}

}  // namespace wam
