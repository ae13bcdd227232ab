// Which tile shape a projection and which form an attention launch takes: cost
// tables and the choice of the smallest cost.  Host arithmetic only (no HIP), so
// that a CPU test can ask for the choice at any size.
#pragma once

namespace wam {

// ---------------------------------------------------------------- projections
// bf16 tile shapes and what a tile costs.  A CU that holds c blocks at once
// (c <= occ) finishes them in about K / 64 * per[c-1] + fix[c-1] us; the
// constants are least-squares fits to timings of every configuration at the
// four projections of 57 model sizes (64 to 12000 rows, D 256 to 2048),
// standard deviation 7-12%.  What they show: 256-column tiles over 8 waves do
// the most work per byte loaded and win where their blocks fill whole rounds of
// the 256 CUs; 128-column tiles over 4 waves leave room for two blocks per CU,
// whose barriers and epilogues overlap, and waste less in the last round; small
// tiles spread short sequences over the chip, where a launch costs ~3 us
// whatever it does.
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

inline double tile_cost(const TileCfg& t, int M, int N, int K) {
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
int plan_gemm(const TileCfg (&cfgs)[NC], int M, int N, int K, bool qkv) {
  int best = -1;
  double bc = 0.0;
  for (int c = 0; c < NC; ++c) {
    const TileCfg& t = cfgs[c];
    // the QKV epilogue needs whole heads (up to 64 columns) per wave
    if (K % t.bk || (qkv && (t.bn / t.wgn) % 64)) continue;
    const double v = tile_cost(t, M, N, K);
    if (best < 0 || v < bc) best = c, bc = v;
  }
  return best;
}

// ---------------------------------------------------------------- attention
// bf16 kernel forms: running max; and with a bound on the scores the fixed
// reference in a software-pipelined loop, a plain loop (also with two wave
// groups that split the keys: 2 nw waves), or the ping-pong form.
enum AttnForm : int { ATTN_RUNNING = 0, ATTN_PIPELINED = 1, ATTN_PLAIN = 2, ATTN_PINGPONG = 3, ATTN_PLAIN_KSPLIT = 4 };

// Forms that the automatic choice picks from, and what a block costs: a CU
// that holds c of its blocks at once (c <= occ, set by their registers) takes
// about ceil(T / 64) * per[c-1] + fix[c-1] us, least-squares fits to timings
// of every form at 52 sizes (B 1 to 16, 4 to 32 heads, T 64 to 12000; standard
// deviation 4-10%).  More queries per wave share each K / V^T read but leave
// larger remainders in the last round; short sequences of few heads split the
// keys over two groups of four waves (T = 864, 12 heads: 8.4 us against 8.9).
struct AttnCfg {
  AttnForm form;
  int qt, nw, occ;
  float per[5], fix[5];
};
constexpr AttnCfg kBounded[] = {
    {ATTN_PLAIN, 4, 8, 1, {1.53f}, {5.0f}},
    {ATTN_PLAIN, 3, 4, 2, {0.84f, 1.19f}, {3.8f, 5.8f}},
    {ATTN_PLAIN, 2, 4, 3, {0.62f, 0.87f, 1.24f}, {3.6f, 5.2f, 5.8f}},
    {ATTN_PLAIN, 1, 4, 5, {0.41f, 0.60f, 0.78f, 1.07f, 1.29f}, {3.2f, 3.8f, 4.7f, 4.9f, 3.4f}},
    {ATTN_PLAIN_KSPLIT, 1, 4, 2, {0.31f, 0.51f}, {3.9f, 3.8f}},
};
constexpr AttnCfg kRunning[] = {
    {ATTN_RUNNING, 3, 8, 1, {1.37f}, {3.9f}},
    {ATTN_RUNNING, 3, 4, 2, {0.86f, 1.32f}, {4.4f, 6.9f}},
    {ATTN_RUNNING, 2, 4, 2, {0.61f, 0.94f}, {4.1f, 5.7f}},
    {ATTN_RUNNING, 1, 4, 4, {0.50f, 0.64f, 0.89f, 1.05f}, {3.3f, 4.2f, 4.7f, 4.8f}},
};

// Index of the form of the smallest cost for heads = B H (sample, head) pairs:
// over those sizes 1.7% (bounded) and 1.0% (running max) slower than the
// fastest form on average, where the fixed rules before were 5% and 10%.
template <int N>
int plan_attention(const AttnCfg (&cfgs)[N], int T, int heads) {
  int best = -1;
  double bc = 0.0;
  for (int i = 0; i < N; ++i) {
    const AttnCfg& c = cfgs[i];
    const int qb = c.qt * c.nw * 16;
    const long blocks = (long)((T + qb - 1) / qb) * heads, n = (blocks + 255) / 256;
    const int rem = (int)(n % c.occ), tiles = (T + 63) / 64;
    double v = (double)(n / c.occ) * (tiles * c.per[c.occ - 1] + c.fix[c.occ - 1]);
    if (rem) v += tiles * c.per[rem - 1] + c.fix[rem - 1];
    if (best < 0 || v < bc) best = i, bc = v;
  }
  return best;
}

// float32 attention: enough 16-query tiles for two waves per SIMD without a key
// split (2048 waves), else four waves split the keys of one tile; two tiles per
// wave (half the K / V^T traffic) once that still leaves four waves per SIMD.
enum AttnF32Form : int { ATTN_F32_KSPLIT = 0, ATTN_F32_ONE_TILE = 1, ATTN_F32_TWO_TILES = 2 };
inline AttnF32Form plan_attention_f32(int T, int heads) {
  const long units = (long)((T + 15) / 16) * heads;
  return units >= 8192 ? ATTN_F32_TWO_TILES : units >= 2048 ? ATTN_F32_ONE_TILE : ATTN_F32_KSPLIT;
}

}  // namespace wam
