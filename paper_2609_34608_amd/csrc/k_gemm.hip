// Projection GEMMs of the DiT block: dispatch for the MFMA kernels of
// gemm_tile.h (bf16, and float32 for the float32 mode) at the tile shape that
// plan.h chooses.
#include "gemm_tile.h"

namespace wam {

namespace {

using gemm::launch_tile;
using gemm::launch_tile_f32;

constexpr int kNumCfgs = sizeof(kCfgs) / sizeof(kCfgs[0]);

template <int C>
hipError_t launch_c(const GemmArgs& a, hipStream_t s) {
  constexpr TileCfg t = kCfgs[C];
  return launch_tile<t.bm, t.bn, t.wgm, t.wgn, t.st, t.bk>(a, s);
}

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

}  // namespace

hipError_t launch_gemm(const GemmArgs& a, bool bf16_mode, hipStream_t s) {
  if (a.M <= 0) return hipSuccess;
  if (a.N % 64) return hipErrorInvalidValue;  // ragged column tiles end on a wave's columns
  if (bf16_mode)
    return launch_any(a, plan_gemm(kCfgs, a.M, a.N, a.K, a.epi == EPI_QKV), s, std::make_integer_sequence<int, kNumCfgs>{});
  return launch_any_f32(a, plan_gemm(kF32Cfgs, a.M, a.N, a.K, a.epi == EPI_QKV), s,
                        std::make_integer_sequence<int, kNumF32Cfgs>{});
}

}  // namespace wam
