// Projection GEMMs of the DiT block: tile-configuration table, planner and
// dispatch for the MFMA kernels of gemm_tile.h (bf16, and float32 for the
// float32 mode).
#include "gemm_tile.h"

namespace wam {

namespace {

using gemm::launch_tile;
using gemm::launch_tile_f32;

// ---------------------------------------------------------------- configs
struct TileCfg {
  int bm, bn, wgm, wgn, st, bk;
};
// index: tile rows x cols, waves (rows x cols), LDS stages, K per stage
constexpr TileCfg kCfgs[] = {
    {64, 64, 2, 2, 4, 32},    // 0
    {64, 128, 2, 2, 4, 32},   // 1
    {128, 64, 2, 2, 4, 32},   // 2
    {128, 128, 2, 2, 4, 32},  // 3
    {256, 256, 2, 4, 4, 32},  // 4
    {256, 256, 4, 2, 4, 32},  // 5
    {256, 128, 2, 4, 4, 32},  // 6
    {128, 256, 2, 4, 4, 32},  // 7
    {128, 128, 2, 4, 4, 32},  // 8
    {64, 256, 1, 4, 4, 32},   // 9
    {64, 64, 2, 2, 8, 32},    // 10
    {64, 128, 2, 2, 8, 32},   // 11
    {128, 64, 2, 2, 8, 32},   // 12
    {64, 64, 2, 2, 12, 32},   // 13
    {128, 128, 2, 2, 8, 32},  // 14
    {64, 64, 2, 2, 4, 128},   // 15
    {64, 128, 2, 2, 3, 128},  // 16
    {128, 64, 2, 2, 3, 128},  // 17
    {64, 64, 2, 2, 4, 64},    // 18
    {64, 128, 2, 2, 4, 64},   // 19
    {128, 128, 2, 4, 4, 64},  // 20
    {256, 256, 4, 2, 2, 64},  // 21
    {256, 256, 2, 4, 2, 64},  // 22
    {128, 128, 2, 2, 4, 64},  // 23
    {192, 256, 2, 4, 2, 64},  // 24
    {320, 256, 2, 4, 2, 64},  // 25
    {64, 64, 4, 1, 4, 32},    // 26 (QKV outputs of 64 mod 128 columns: odd head counts)
    {320, 128, 4, 2, 2, 64},  // 27
};
constexpr int kNumCfgs = sizeof(kCfgs) / sizeof(kCfgs[0]);

template <int C, int ROLE>
hipError_t launch_c(const GemmArgs& a, int splits, hipStream_t s) {
  constexpr TileCfg t = kCfgs[C];
  return launch_tile<t.bm, t.bn, t.wgm, t.wgn, t.st, t.bk, ROLE>(a, splits, s);
}

template <int ROLE>
hipError_t launch_role(const GemmArgs& a, int cfg, int splits, hipStream_t s) {
  switch (cfg) {
    case 0: return launch_c<0, ROLE>(a, splits, s);
    case 1: return launch_c<1, ROLE>(a, splits, s);
    case 2: return launch_c<2, ROLE>(a, splits, s);
    case 3: return launch_c<3, ROLE>(a, splits, s);
    case 4: return launch_c<4, ROLE>(a, splits, s);
    case 5: return launch_c<5, ROLE>(a, splits, s);
    case 6: return launch_c<6, ROLE>(a, splits, s);
    case 7: return launch_c<7, ROLE>(a, splits, s);
    case 8: return launch_c<8, ROLE>(a, splits, s);
    case 9: return launch_c<9, ROLE>(a, splits, s);
    case 10: return launch_c<10, ROLE>(a, splits, s);
    case 11: return launch_c<11, ROLE>(a, splits, s);
    case 12: return launch_c<12, ROLE>(a, splits, s);
    case 13: return launch_c<13, ROLE>(a, splits, s);
    case 14: return launch_c<14, ROLE>(a, splits, s);
    case 15: return launch_c<15, ROLE>(a, splits, s);
    case 16: return launch_c<16, ROLE>(a, splits, s);
    case 17: return launch_c<17, ROLE>(a, splits, s);
    case 18: return launch_c<18, ROLE>(a, splits, s);
    case 19: return launch_c<19, ROLE>(a, splits, s);
    case 20: return launch_c<20, ROLE>(a, splits, s);
    case 21: return launch_c<21, ROLE>(a, splits, s);
    case 22: return launch_c<22, ROLE>(a, splits, s);
    case 23: return launch_c<23, ROLE>(a, splits, s);
    case 24: return launch_c<24, ROLE>(a, splits, s);
    case 25: return launch_c<25, ROLE>(a, splits, s);
    case 26: return launch_c<26, ROLE>(a, splits, s);
    default: return launch_c<27, ROLE>(a, splits, s);
  }
}

bool qkv_ok(int c) { return (kCfgs[c].bn / kCfgs[c].wgn) % 64 == 0; }

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

int gemm_num_configs() { return kNumCfgs; }

GemmPlan plan_gemm(int M, int N, int K, int epi) {
  // From a sweep of every configuration at the workload shapes.  Large M:
  // tiles of 256 columns over 8 waves, K 64 per stage (two stages), with the
  // row count (192, 256 or 320) that minimises whole rounds of one block per
  // CU times rows per block, weighted by the per-row cost each tile height
  // measured (192-row tiles ~10% dearer per row, 320-row ~3% cheaper).  For
  // example M = 9224, N = 4096 (mid MLP-up): 592 blocks of 256 rows take 3
  // rounds, 464 of 320 rows take 2 (98 -> 82 us); M = 9224, N = 1024: 196
  // blocks of 192 rows fill one round that 148 of 256 leave a third idle
  // (97 -> 83 us).  256 rows with K 32 per stage (four stages) for outputs of
  // 1024 columns or fewer, or K not a multiple of 64.  Small M (under a few
  // blocks per CU): 64x64 tiles with K 64 per stage, 64x128 for the QKV
  // epilogue (whole heads per wave), 128x128 over 8 waves for wide, short-K
  // outputs; a K split only for grids under half a block per CU.
  GemmPlan p{0, 1};
  if (M >= 2048 && N % 256 == 0) {
    // outputs of at most 1024 columns whose 320x128 tiles fill one round
    // of 192-256 blocks (the mid model's attention output and MLP-down,
    // N = 1024: 232 blocks, against 196 of 192x256 that leave 60 CUs idle;
    // 34.4 -> 31.8 and 97.4 -> 89.0 us)
    const long b320x128 = (long)((M + 319) / 320) * (N / 128);
    if (K % 64 == 0 && N <= 1024 && b320x128 >= 192 && b320x128 <= 256) {
      p.cfg = 27;
      return p;
    }
    if (K % 64 == 0) {
      const long cols = N / 256;
      auto cost = [&](int bm, double per_row) {
        const long blocks = (M + bm - 1) / bm * cols;
        return (double)((blocks + 255) / 256) * bm * per_row;
      };
      const double c192 = cost(192, 1.10), c256 = cost(256, 1.0), c320 = cost(320, 0.97);
      if (c192 < c256 && c192 <= c320) {
        p.cfg = 24;
        return p;
      }
      if (c320 < c256) {
        p.cfg = 25;
        return p;
      }
    }
    if (N > 1024 && K % 64 == 0) p.cfg = 22;
    else p.cfg = N >= 3072 ? 5 : 4;
    return p;
  }
  if (epi == EPI_QKV) {
    // whole heads per wave: 64 columns per wave; an odd head count leaves
    // N = 192 H a multiple of 64 only, which takes one wave column of 64
    p.cfg = N % 128 != 0 ? 26 : K % 64 == 0 ? 19 : 1;
    return p;
  }
  if (N >= 2048 && N % 128 == 0 && K <= 1024) {
    p.cfg = 8;
    return p;
  }
  const long blocks = (long)((M + 63) / 64) * (N / 64);
  if (K % 64 == 0 && blocks >= 128) {
    p.cfg = 18;
    return p;
  }
  while (blocks * p.splits < 128 && K / (p.splits * 2) >= 768 && K % (gemm::kBK * p.splits * 2) == 0 &&
         p.splits < 8)
    p.splits *= 2;
  return p;
}

size_t gemm_partial_floats(int M, int N, int K, int epi) {
  const GemmPlan p = plan_gemm(M, N, K, epi);
  return p.splits > 1 ? (size_t)p.splits * M * N : 0;
}

hipError_t launch_gemm_cfg(const GemmArgs& a, int cfg, int splits, hipStream_t s) {
  if (a.M <= 0) return hipSuccess;
  if (cfg < 0 || cfg >= kNumCfgs || splits < 1) return hipErrorInvalidValue;
  if (a.K % (kCfgs[cfg].bk * splits) || a.N % kCfgs[cfg].bn || a.N % 4) return hipErrorInvalidValue;
  if (splits > 1 && (a.epi == EPI_QKV || !a.partial)) return hipErrorInvalidValue;
  if (a.epi == EPI_QKV && !qkv_ok(cfg)) return hipErrorInvalidValue;
  switch (a.role) {
    case 0: return launch_role<0>(a, cfg, splits, s);
    case 1: return launch_role<1>(a, cfg, splits, s);
    case 2: return launch_role<2>(a, cfg, splits, s);
    default: return launch_role<3>(a, cfg, splits, s);
  }
}

hipError_t launch_gemm(const GemmArgs& a, bool bf16_mode, hipStream_t s) {
  if (a.M <= 0) return hipSuccess;
  if (bf16_mode) {
    const GemmPlan p = plan_gemm(a.M, a.N, a.K, a.epi);
    return launch_gemm_cfg(a, p.cfg, p.splits, s);
  }
  return launch_gemm_f32(a, s);
}

}  // namespace wam
