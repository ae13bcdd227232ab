// Tiled MFMA GEMM kernel template (gfx950), bf16 or float32 operands;
// instantiated by k_gemm.hip.
//
//   C[M][N] = A[M][K] . W[N][K]^T      (both operands K-contiguous)
//
// v_mfma_f32_16x16x32_bf16 takes the weight tile as its first operand and the
// activation tile as its second, so accumulator element r of a lane is
// C[m = lane%16][n = 4*(lane/16) + r]: each lane owns four consecutive output
// columns of one row and the epilogue stores 8 (bf16) or 16 (fp32) contiguous
// bytes.  A block of WGM x WGN waves owns a BM x BN tile.
//
// float32 operands use four v_mfma_f32_16x16x4_f32 where bf16 uses one MFMA:
// a lane's 16-byte chunk is then 4 values of K instead of 8, and MFMA r
// contracts value r of the four lanes' chunks (the order of K within a step
// does not matter as long as both operands share it), so the stages, the
// swizzle and the operand reads are the same bytes in both types.
//
// K advances BK elements (128 or 256 bytes) at a time through ST LDS stages.
// Each stage holds BM activation rows and BN weight rows, filled straight
// from global memory by global_load_lds_dwordx4 (16 bytes per lane, one 1 KiB
// run of LDS per instruction, no register staging): ST-1 stages are in flight
// while one is multiplied.  Inside a row the 16-byte chunks are XOR-swizzled
// (row & 7), which keeps the ds_read_b128 operand reads (16 rows x one chunk per
// 16 lanes) free of bank conflicts; the loads pick their global chunk so that
// the LDS image comes out swizzled.  The longer rows give each wave four MFMA
// k-steps per barrier instead of two, which is what the smallest tiles need.
// The compiler cannot follow the LDS writes of these loads, so the loop waits on
// vmcnt itself and uses a bare s_barrier (a workgroup fence would drain every
// load in flight).
// Blocks are renumbered so that each XCD (dispatch is round-robin over 8 XCDs)
// gets a contiguous run of a grouped tile order and shares A rows / W columns
// in its own L2.
#pragma once

#include "wam_internal.h"

namespace wam {
namespace gemm {

constexpr int kGroupM = 8;
constexpr int kXcd = 8;

typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(1))) void global_void;

// s_waitcnt immediate (gfx9 layout: vmcnt bits 3:0 and 15:14, expcnt 6:4,
// lgkmcnt 11:8): at most n vector-memory operations outstanding, no LDS or
// scalar-memory operation outstanding
constexpr int waitcnt_vm_lgkm0(int n) { return (n & 0xf) | ((n >> 4) << 14) | (0x7 << 4); }

// XOR swizzle of the 16-byte chunks of an LDS row (8 or 16 chunks)
__device__ __forceinline__ int chunk_swizzle(int row) { return row & 7; }

// Operand chunk (16 bytes) of one lane and the MFMA step that consumes a
// weight and an activation chunk.
template <typename E>
struct Operand;
template <>
struct Operand<bf16> {
  typedef bf16x8 frag;
  static constexpr int kSteps = 1;  // MFMAs per chunk pair
  static __device__ __forceinline__ f32x4 mma(frag w, frag a, f32x4 c, int) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, a, c, 0, 0, 0);
  }
};
template <>
struct Operand<float> {
  typedef f32x4 frag;
  static constexpr int kSteps = 4;
  static __device__ __forceinline__ f32x4 mma(frag w, frag a, f32x4 c, int r) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(w[r], a[r], c, 0, 0, 0);
  }
};

// compiler-only memory barrier: keeps LDS and global accesses on their side
__device__ __forceinline__ void compiler_fence() { asm volatile("" ::: "memory"); }

__device__ __forceinline__ void tile_coords(int bid, int nblocks, int tiles_m, int tiles_n, int& tm,
                                            int& tn) {
  const int per = nblocks / kXcd, rem = nblocks % kXcd;
  const int x = bid % kXcd, idx = bid / kXcd;
  const int logical = x * per + min(x, rem) + idx;
  const int width = kGroupM * tiles_n;
  const int group = logical / width;
  const int first_m = group * kGroupM;
  const int gsz = min(tiles_m - first_m, kGroupM);
  const int in = logical % width;
  tm = first_m + in % gsz;
  tn = in / gsz;
}

__device__ __forceinline__ void store4(bf16* p, f32x4 x) {
  bf16x4 v = {static_cast<bf16>(x[0]), static_cast<bf16>(x[1]), static_cast<bf16>(x[2]), static_cast<bf16>(x[3])};
  *reinterpret_cast<bf16x4*>(p) = v;
}
__device__ __forceinline__ void store4(float* p, f32x4 x) { *reinterpret_cast<f32x4*>(p) = x; }

__device__ __forceinline__ f32x4 gelu4(f32x4 v) {
  return f32x4{gelu_tanh_f(v[0]), gelu_tanh_f(v[1]), gelu_tanh_f(v[2]), gelu_tanh_f(v[3])};
}

// Epilogue of one wave's accumulators: acc[j][i] element r is the product at
// row mb + i*16 + lane%16, column nb + j*16 + 4*(lane/16) + r.
template <typename E, int EPI, int DH, int TN, int TM>
__device__ __forceinline__ void store_tile(const GemmArgs& a, const f32x4 (&acc)[TN][TM], int mb, int nb, int lane) {
  const int lr = lane % 16, lg = lane / 16;
  if constexpr (EPI == EPI_QKV) {
    constexpr int JH = DH / 16;  // column tiles per head
    const QkvOut& qo = a.qkv;
    const int D = qo.D;
    // per-lane constants hoisted out of the store loop: bias of the lane's
    // columns and the q / k gains of its head dims (d = jj*16 + 4*lg + r)
    f32x4 bias[TN], qg[JH], kg[JH];
#pragma unroll
    for (int j = 0; j < TN; ++j) bias[j] = *reinterpret_cast<const f32x4*>(a.bias + nb + j * 16 + lg * 4);
#pragma unroll
    for (int jj = 0; jj < JH; ++jj) {
      qg[jj] = kg[jj] = f32x4{1.f, 1.f, 1.f, 1.f};
      if (qo.qk_norm) {
        qg[jj] = *reinterpret_cast<const f32x4*>(qo.q_g + jj * 16 + lg * 4);
        kg[jj] = *reinterpret_cast<const f32x4*>(qo.k_g + jj * 16 + lg * 4);
      }
      qg[jj] *= q_log2_scale(DH);  // attention scores come out in log2 units
    }
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int m = mb + i * 16 + lr;
      const int b = m / qo.T, t = m % qo.T;
#pragma unroll
      for (int hs = 0; hs < TN / JH; ++hs) {
        const int nh = nb + hs * DH;  // first column of this head
        const int sec = nh / D, head = (nh % D) / DH;
        f32x4 v[JH];
        float ss = 0.f;
#pragma unroll
        for (int jj = 0; jj < JH; ++jj) {
          v[jj] = acc[hs * JH + jj][i] + bias[hs * JH + jj];
#pragma unroll
          for (int r = 0; r < 4; ++r) ss += v[jj][r] * v[jj][r];
        }
        if (sec < 2) {
          ss += __shfl_xor(ss, 16, 64);
          ss += __shfl_xor(ss, 32, 64);
          const f32x4* gain = sec == 0 ? qg : kg;
          const float rs = qo.qk_norm ? row_scale<E>(ss * (1.0f / DH) + qo.eps) : 1.0f;
          if (m < a.M) {
            E* dst = static_cast<E*>(sec == 0 ? qo.q : qo.k) + (((size_t)b * qo.H + head) * qo.Tpad + t) * DH;
#pragma unroll
            for (int jj = 0; jj < JH; ++jj) store4(dst + jj * 16 + lg * 4, v[jj] * rs * gain[jj]);
          }
        } else if (m < a.M) {
          // V^T row d; bf16: the tokens of each 64-key block in vt_key_pos order
          const int tp = sizeof(E) == 2 ? (t & ~63) + vt_key_pos(t & 63) : t;
          E* dst = static_cast<E*>(qo.vt) + ((size_t)b * qo.H + head) * DH * qo.Tpad + tp;
#pragma unroll
          for (int jj = 0; jj < JH; ++jj)
#pragma unroll
            for (int r = 0; r < 4; ++r)
              dst[(size_t)(jj * 16 + lg * 4 + r) * qo.Tpad] = static_cast<E>(v[jj][r]);
        }
      }
    }
  } else {
    // bias (and gate) of this lane's columns once, in registers: the output
    // may alias them as far as the compiler knows, so loads inside the store
    // loop would be repeated and serialised behind every store
    f32x4 bias[TN], gate[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int n = nb + j * 16 + lg * 4;
      bias[j] = *reinterpret_cast<const f32x4*>(a.bias + n);
      if constexpr (EPI == EPI_GATED_RES) gate[j] = *reinterpret_cast<const f32x4*>(a.gate + n);
    }
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int m = mb + i * 16 + lr;
      if (m >= a.M) continue;
      if constexpr (EPI == EPI_GATED_RES) {
        // residual stream plus gate * (acc + bias): all loads of the row first;
        // with a copy target the new values are stored there as well
        const size_t off = (size_t)m * a.N + nb + lg * 4;
        const f32x4* rrow = reinterpret_cast<const f32x4*>(a.res + off);
        f32x4* hrow = reinterpret_cast<f32x4*>(static_cast<float*>(a.out) + off);
        f32x4 hv[TN];
#pragma unroll
        for (int j = 0; j < TN; ++j) hv[j] = rrow[j * 4];
#pragma unroll
        for (int j = 0; j < TN; ++j) hv[j] = hv[j] + gate[j] * (acc[j][i] + bias[j]);
#pragma unroll
        for (int j = 0; j < TN; ++j) hrow[j * 4] = hv[j];
        if (a.copy) {
          f32x4* crow = reinterpret_cast<f32x4*>(a.copy + off);
#pragma unroll
          for (int j = 0; j < TN; ++j) crow[j * 4] = hv[j];
        }
      } else {
        E* orow = static_cast<E*>(a.out) + (size_t)m * a.N + nb + lg * 4;
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          const f32x4 v = acc[j][i] + bias[j];
          if constexpr (EPI == EPI_BIAS_GELU) store4(orow + j * 16, gelu4(v));
          else store4(orow + j * 16, v);
        }
      }
    }
  }
}

template <typename E, int BM, int BN, int WGM, int WGN, int ST, int BK, int EPI, int DH>
__device__ __forceinline__ void gemm_body(const GemmArgs& a) {
  typedef typename Operand<E>::frag frag;
  constexpr int EPC = 16 / sizeof(E);          // elements per 16-byte chunk
  constexpr int NW = WGM * WGN;
  constexpr int WM = BM / WGM, WN = BN / WGN;  // wave tile
  constexpr int TM = WM / 16, TN = WN / 16;
  constexpr int ROWS = BM + BN;                // LDS rows per stage: activations, then weights
  constexpr int CPR = BK / EPC;                // 16-byte chunks per LDS row
  constexpr int RPI = 64 / CPR;                // rows per 1 KiB load instruction
  constexpr int NI = ROWS / RPI;               // load instructions per stage
  constexpr int IPW = NI / NW;                 // ... per wave
  constexpr int KS = CPR / 4;                  // MFMA k-steps per stage (four chunks each)
  static_assert(CPR == 8 || CPR == 16, "stage depth");
  static_assert(TM >= 1 && TN >= 1, "wave tile too small");
  static_assert(IPW >= 1 && IPW * NW == NI, "stage rows / wave mismatch");
  static_assert(EPI != EPI_QKV || WN % DH == 0, "QKV epilogue needs whole heads per wave");
  static_assert(ST >= 2 && (ST - 2) * IPW < 64, "stage count");
  static_assert(64 % WN == 0, "ragged N: a wave's columns lie inside N or past it");
  if (a.skip && *a.skip) return;

  __shared__ __attribute__((aligned(1024))) E sm[ST][ROWS * BK];

  const int tiles_m = (a.M + BM - 1) / BM, tiles_n = (a.N + BN - 1) / BN;
  int tm, tn;
  tile_coords(blockIdx.x, gridDim.x, tiles_m, tiles_n, tm, tn);
  const int m0 = tm * BM, n0 = tn * BN;
  const int tid = threadIdx.x, lane = tid % 64, wid = tid / 64;
  const int wm = wid / WGN, wn = wid % WGN;
  const E* A = static_cast<const E*>(a.A);
  const E* W = static_cast<const E*>(a.W);
  const int K = a.K;
  const int nk = K / BK;

  // Load instruction j of this wave fills LDS rows RPI*(wid + NW*j) .. +RPI-1;
  // lane l writes LDS chunk l%CPR of row l/CPR, i.e. global chunk
  // (l%CPR) ^ swizzle.  Activation rows past M read row M-1 and weight rows
  // past N row N-1 (their products reach only outputs that are never stored).
  const E* src[IPW];
#pragma unroll
  for (int j = 0; j < IPW; ++j) {
    const int row = RPI * (wid + NW * j) + lane / CPR;
    const int col = ((lane % CPR) ^ chunk_swizzle(row)) * EPC;
    src[j] = row < BM ? A + (size_t)min(m0 + row, a.M - 1) * K + col
                      : W + (size_t)min(n0 + row - BM, a.N - 1) * K + col;
  }
  auto issue = [&](auto S, int kt) __attribute__((always_inline)) {
    constexpr int s = decltype(S)::value;
#pragma unroll
    for (int j = 0; j < IPW; ++j)
      __builtin_amdgcn_global_load_lds((const global_void*)(src[j] + kt * BK),
                                       (lds_void*)(&sm[s][(wid + NW * j) * RPI * BK]), 16, 0, 0);
  };

  f32x4 acc[TN][TM];
#pragma unroll
  for (int j = 0; j < TN; ++j)
#pragma unroll
    for (int i = 0; i < TM; ++i) acc[j][i] = f32x4{0.f, 0.f, 0.f, 0.f};

  // operand reads: for k-step ks, lane (lr, lg) takes chunk 4*ks + lg of row
  // lr of each 16-row tile (tile row offsets are multiples of 16, so the
  // swizzle depends on lr only)
  const int lr = lane % 16, lg = lane / 16;
  const int sw = chunk_swizzle(lr);
  const int arow = (wm * WM + lr) * BK;
  const int wrow = (BM + wn * WN + lr) * BK;
  auto compute = [&](auto S) __attribute__((always_inline)) {
    constexpr int s = decltype(S)::value;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const int ch = ((4 * ks + lg) ^ sw) * EPC;
      frag af[TM], wf[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) af[i] = *reinterpret_cast<const frag*>(&sm[s][arow + ch + i * 16 * BK]);
#pragma unroll
      for (int j = 0; j < TN; ++j) wf[j] = *reinterpret_cast<const frag*>(&sm[s][wrow + ch + j * 16 * BK]);
#pragma unroll
      for (int r = 0; r < Operand<E>::kSteps; ++r)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int i = 0; i < TM; ++i) acc[j][i] = Operand<E>::mma(wf[j], af[i], acc[j][i], r);
    }
  };
  // one K step on stage slot J: this wave's loads of stage kt have landed (the
  // ST-2 newer stages may still be in flight) and its LDS reads are done;
  // after the barrier everyone's are, and the slot read in the previous step
  // is free for stage kt+ST-1.  Past the last stage the loads repeat it into
  // slots nobody reads again, which keeps the wait counts uniform.
  auto step = [&](auto J, int kt) __attribute__((always_inline)) {
    constexpr int j = decltype(J)::value;
    __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0((ST - 2) * IPW));
    compiler_fence();
    __builtin_amdgcn_s_barrier();
    compiler_fence();
    issue(std::integral_constant<int, (j + ST - 1) % ST>{}, min(kt + ST - 1, nk - 1));
    // the loads must leave before the MFMAs: left to itself the scheduler
    // sinks them below the compute, next to the wait at the top of the next
    // step, which exposes their whole latency every stage
    __builtin_amdgcn_sched_barrier(0);
    compute(J);
  };

  static_for<ST - 1>([&](auto P) __attribute__((always_inline)) { issue(P, min((int)decltype(P)::value, nk - 1)); });
  const int nfull = nk / ST * ST;
  for (int kt0 = 0; kt0 < nfull; kt0 += ST)
    static_for<ST>([&](auto J) __attribute__((always_inline)) { step(J, kt0 + decltype(J)::value); });
  static_for<ST - 1>([&](auto J) __attribute__((always_inline)) {
    const int kt = nfull + decltype(J)::value;
    if (kt < nk) step(J, kt);
  });
  // no load may still be writing this block's LDS when the block retires
  __builtin_amdgcn_s_waitcnt(0);

  // N is a multiple of 64 and a wave's columns divide 64: a wave of the last
  // column tile lies either inside N or past it as a whole
  if (n0 + wn * WN >= a.N) return;
  store_tile<E, EPI, DH, TN, TM>(a, acc, m0 + wm * WM, n0 + wn * WN, lane);
}

template <int BM, int BN, int WGM, int WGN, int ST, int BK, int EPI, int ROLE>
__global__ __launch_bounds__(WGM* WGN * 64) void gemm_bf16_kernel(GemmArgs a) {
  gemm_body<bf16, BM, BN, WGM, WGN, ST, BK, EPI, 64>(a);
}

template <int BM, int BN, int WGM, int WGN, int ST, int BK, int EPI, int DH>
__global__ __launch_bounds__(WGM* WGN * 64) void gemm_f32_kernel(GemmArgs a) {
  gemm_body<float, BM, BN, WGM, WGN, ST, BK, EPI, DH>(a);
}

// The four projections: role 0 QKV, 1 attention output, 2 MLP-up, 3 MLP-down,
// each with its own epilogue.
template <int BM, int BN, int WGM, int WGN, int ST, int BK>
hipError_t launch_tile(const GemmArgs& a, hipStream_t s) {
  const int blocks = ((a.M + BM - 1) / BM) * ((a.N + BN - 1) / BN);
  constexpr int NT = WGM * WGN * 64;
  if (a.role == 0 && a.epi == EPI_QKV) {
    if constexpr ((BN / WGN) % 64 == 0)
      launch_k(gemm_bf16_kernel<BM, BN, WGM, WGN, ST, BK, EPI_QKV, 0>, blocks, NT, 0, s, a);
    else
      return hipErrorInvalidValue;
  } else if (a.role == 1 && a.epi == EPI_GATED_RES) {
    launch_k(gemm_bf16_kernel<BM, BN, WGM, WGN, ST, BK, EPI_GATED_RES, 1>, blocks, NT, 0, s, a);
  } else if (a.role == 2 && a.epi == EPI_BIAS_GELU) {
    launch_k(gemm_bf16_kernel<BM, BN, WGM, WGN, ST, BK, EPI_BIAS_GELU, 2>, blocks, NT, 0, s, a);
  } else if (a.role == 3 && a.epi == EPI_GATED_RES) {
    launch_k(gemm_bf16_kernel<BM, BN, WGM, WGN, ST, BK, EPI_GATED_RES, 3>, blocks, NT, 0, s, a);
  } else {
    return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int BM, int BN, int WGM, int WGN, int ST, int BK>
hipError_t launch_tile_f32(const GemmArgs& a, hipStream_t s) {
  const int blocks = ((a.M + BM - 1) / BM) * ((a.N + BN - 1) / BN);
  constexpr int NT = WGM * WGN * 64;
  switch (a.epi) {
    case EPI_BIAS_GELU:
      launch_k(gemm_f32_kernel<BM, BN, WGM, WGN, ST, BK, EPI_BIAS_GELU, 64>, blocks, NT, 0, s, a);
      break;
    case EPI_GATED_RES:
      launch_k(gemm_f32_kernel<BM, BN, WGM, WGN, ST, BK, EPI_GATED_RES, 64>, blocks, NT, 0, s, a);
      break;
    case EPI_QKV:
      if constexpr ((BN / WGN) % 64 == 0) {
        if (a.qkv.dh == 32) launch_k(gemm_f32_kernel<BM, BN, WGM, WGN, ST, BK, EPI_QKV, 32>, blocks, NT, 0, s, a);
        else launch_k(gemm_f32_kernel<BM, BN, WGM, WGN, ST, BK, EPI_QKV, 64>, blocks, NT, 0, s, a);
      } else {
        return hipErrorInvalidValue;
      }
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace gemm
}  // namespace wam
