// Bandwidth- and latency-bound kernels of the denoising step and of the
// state-adaptation operators (gfx950, wave64).
#include <math.h>

#include <algorithm>
#include <mutex>
#include <string>

#include "wam_internal.h"

namespace wam {

namespace {

__device__ __forceinline__ double block_sum_d(double v, double* sh) {
  v = wave_sum_d(v);
  const int w = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  const int nw = blockDim.x / kWave;
  __syncthreads();
  if (lane == 0) sh[w] = v;
  __syncthreads();
  double t = 0.0;
  for (int i = 0; i < nw; ++i) t += sh[i];
  return t;
}

// ------------------------------------------------------------- timestep MLP
// Small GEMV for the conditioning MLP: block = 64 outputs x 16 K-groups,
// y[n] = SiLU(sum_k x[k] W[k][n] + b[n]).  With FEATURES the input is
// computed in-kernel from sigma: x = [cos(t f_i), sin(t f_i)], t = 1000 sigma,
// f_i = 10000^(-i/128) (float64 arguments).
constexpr int kTimeDim = 256;
constexpr int kSgN = 64, kSgK = 16;
template <bool FEATURES>
__global__ __launch_bounds__(kSgN* kSgK) void small_gemv_silu_kernel(float sigma, const float* __restrict__ x,
                                                                    const float* __restrict__ W,
                                                                    const float* __restrict__ b,
                                                                    float* __restrict__ y, int K, int N) {
  __shared__ float xs[2048];
  __shared__ float part[kSgK][kSgN + 1];
  const int tid = threadIdx.x, nl = tid % kSgN, kg = tid / kSgN;
  for (int k = tid; k < K; k += blockDim.x) {
    if constexpr (FEATURES) {
      const int half = K / 2;
      const int j = k < half ? k : k - half;
      const double t = 1000.0 * (double)sigma;
      const double f = exp(-log(10000.0) * (double)j / (double)half);
      xs[k] = (float)(k < half ? cos(t * f) : sin(t * f));
    } else {
      xs[k] = x[k];
    }
  }
  __syncthreads();
  const int n = blockIdx.x * kSgN + nl;
  float acc = 0.f;
  if (n < N) {
#pragma unroll 4
    for (int k = kg; k < K; k += kSgK) acc += xs[k] * W[(size_t)k * N + n];
  }
  part[kg][nl] = acc;
  __syncthreads();
  if (kg == 0 && n < N) {
    float s = b[n];
    for (int g = 0; g < kSgK; ++g) s += part[g][nl];
    y[n] = s / (1.0f + __expf(-s));
  }
}

// ------------------------------------------------------------- GEMV
constexpr int kGemvKc = 32;   // input rows per split
constexpr int kGemvVec = 4;   // outputs per thread

__device__ __forceinline__ float act_apply(float v, int act) {
  return act == 1 ? v / (1.0f + __expf(-v)) : v;
}

template <typename TW>
__global__ void gemv_partial_kernel(const float* __restrict__ x, const TW* __restrict__ W,
                                    float* __restrict__ partial, int K, int N, int in_act) {
  const int n0 = (blockIdx.x * blockDim.x + threadIdx.x) * kGemvVec;
  const int k0 = blockIdx.y * kGemvKc;
  if (n0 >= N) return;
  float acc[kGemvVec] = {0.f, 0.f, 0.f, 0.f};
  const int k1 = min(K, k0 + kGemvKc);
  for (int k = k0; k < k1; ++k) {
    const float xv = act_apply(x[k], in_act);
    const TW* row = W + (size_t)k * N + n0;
#pragma unroll
    for (int j = 0; j < kGemvVec; ++j) acc[j] += xv * to_f32(row[j]);
  }
  float* p = partial + (size_t)blockIdx.y * N + n0;
#pragma unroll
  for (int j = 0; j < kGemvVec; ++j) p[j] = acc[j];
}

__global__ void gemv_reduce_kernel(const float* __restrict__ partial, const float* __restrict__ b,
                                   float* __restrict__ y, int nchunk, int N, int out_act) {
  const int n = blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= N) return;
  float s = 0.f;
  for (int c = 0; c < nchunk; ++c) s += partial[(size_t)c * N + n];
  y[n] = act_apply(s + b[n], out_act);
}

// ------------------------------------------------------------- embedding
// h[b,t,:] = token (video | action | obs) @ W_branch + b_branch + PE(t), PE a
// table built once at init
__global__ void embed_kernel(EmbedArgs a) {
  const int row = blockIdx.x;  // b*T + t
  const int b = row / a.T, t = row % a.T;
  __shared__ float tok[64];
  const float* w;
  const float* bias;
  int c;
  const int traj = a.Nv * a.Cv + a.Na * a.A;
  if (t < a.Nv) {
    c = a.Cv;
    w = a.wv;
    bias = a.bv;
    if (threadIdx.x < c) tok[threadIdx.x] = a.x[(size_t)b * traj + (size_t)t * a.Cv + threadIdx.x];
  } else if (t < a.Nv + a.Na) {
    c = a.A;
    w = a.wa;
    bias = a.ba;
    if (threadIdx.x < c)
      tok[threadIdx.x] = a.x[(size_t)b * traj + (size_t)a.Nv * a.Cv + (size_t)(t - a.Nv) * a.A + threadIdx.x];
  } else {
    c = a.Co;
    w = a.wo;
    bias = a.bo;
    if (threadIdx.x < c)
      tok[threadIdx.x] = a.cond[((size_t)b * a.No + (t - a.Nv - a.Na)) * a.Co + threadIdx.x];
  }
  __syncthreads();
  const float* pe = a.pe + (size_t)t * a.D;
  for (int d = threadIdx.x; d < a.D; d += blockDim.x) {
    float s = bias[d];
    for (int j = 0; j < c; ++j) s += tok[j] * w[(size_t)j * a.D + d];
    a.h[(size_t)row * a.D + d] = s + pe[d];
  }
}

// Vectorised form: a block takes up to R consecutive rows of one branch
// (video, action or observation tokens) of one sample, so that the branch's
// weight rows are read once for all of them (with one row per block the
// weight reads from L2 outweighed the HBM traffic of long sequences: 66 ->
// 33 us at T = 10176 with R = 8); thread i owns columns 4i..4i+3 (D / 4
// threads).  Every load a thread needs (bias, the up to kEmbedC weight rows,
// clamped to the branch's channel count against zero-padded token values,
// and the position-embedding rows) is issued before the sums.
constexpr int kEmbedC = 16;
__host__ __device__ inline int embed_blocks_per_sample(int Nv, int Na, int No, int R) {
  return (Nv + R - 1) / R + (Na + R - 1) / R + (No + R - 1) / R;
}
template <int R>
__global__ __launch_bounds__(512) void embed_v4_kernel(EmbedArgs a) {
  constexpr int kEmbedRows = R;
  const int per = embed_blocks_per_sample(a.Nv, a.Na, a.No, R);
  const int b = blockIdx.x / per, j = blockIdx.x % per;
  const int gv = (a.Nv + kEmbedRows - 1) / kEmbedRows, ga = (a.Na + kEmbedRows - 1) / kEmbedRows;
  const float* w;
  const float* bias;
  const float* src;  // token values of the block's first row
  int c, t0, n;      // channels, first row (within the sample), rows of this block
  const int traj = a.Nv * a.Cv + a.Na * a.A;
  if (j < gv) {
    t0 = j * kEmbedRows, n = min(kEmbedRows, a.Nv - t0), c = a.Cv, w = a.wv, bias = a.bv;
    src = a.x + (size_t)b * traj + (size_t)t0 * a.Cv;
  } else if (j < gv + ga) {
    const int i0 = (j - gv) * kEmbedRows;
    t0 = a.Nv + i0, n = min(kEmbedRows, a.Na - i0), c = a.A, w = a.wa, bias = a.ba;
    src = a.x + (size_t)b * traj + (size_t)a.Nv * a.Cv + (size_t)i0 * a.A;
  } else {
    const int i0 = (j - gv - ga) * kEmbedRows;
    t0 = a.Nv + a.Na + i0, n = min(kEmbedRows, a.No - i0), c = a.Co, w = a.wo, bias = a.bo;
    src = a.cond + ((size_t)b * a.No + i0) * a.Co;
  }
  __shared__ float tok[kEmbedRows][kEmbedC];
  for (int i = threadIdx.x; i < kEmbedRows * kEmbedC; i += blockDim.x) {
    const int r = i / kEmbedC, ch = i % kEmbedC;
    tok[r][ch] = r < n && ch < c ? src[(size_t)r * c + ch] : 0.f;
  }
  const int col = threadIdx.x * 4;
  const bool live = col < a.D;
  const int cc = live ? col : 0;
  const f32x4 b4 = *reinterpret_cast<const f32x4*>(bias + cc);
  f32x4 w4[kEmbedC], p4[kEmbedRows];
#pragma unroll
  for (int k = 0; k < kEmbedC; ++k) w4[k] = *reinterpret_cast<const f32x4*>(w + (size_t)min(k, c - 1) * a.D + cc);
#pragma unroll
  for (int r = 0; r < kEmbedRows; ++r)
    p4[r] = *reinterpret_cast<const f32x4*>(a.pe + (size_t)(t0 + min(r, n - 1)) * a.D + cc);
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kEmbedRows; ++r) {
    if (r >= n) break;
    f32x4 acc = b4;
#pragma unroll
    for (int k = 0; k < kEmbedC; ++k) acc += tok[r][k] * w4[k];
    if (live) *reinterpret_cast<f32x4*>(a.h + ((size_t)b * a.T + t0 + r) * a.D + col) = acc + p4[r];
  }
}

// ------------------------------------------------------------- LN + modulation
// One wave per row; lane holds elements 4 lane + 256 i .. +3 (16-byte loads,
// 8- or 16-byte stores), i < N4 = ceil(D / 256).  N4 is a template argument so
// that the row and the modulation are fetched by 3 N4 loads issued together,
// ahead of the reductions (with a run-time count the compiler emitted one load
// and one wait per chunk).  RAG: D is not a multiple of 256 (it is one of 64),
// and the lanes of the last chunk past D load the row's start again and count
// as zero.  HBM bound (6 bytes an element with bf16 results, 8 with float32);
// D = 1216, 5754 rows, bf16: 17.5 us with one element per lane and load, 8.8 us
// here.
template <int N4, bool RAG, typename TOut>
__global__ __launch_bounds__(256) void ln_modulate_kernel(const float* __restrict__ h, const float* __restrict__ shift,
                                                          const float* __restrict__ scale, TOut* __restrict__ u,
                                                          int rows, int D, float eps, const int* skip) {
  if (skip && *skip) return;
  if constexpr (!RAG) D = N4 * 256;
  const int row = blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave;
  const int lane = threadIdx.x % kWave;
  if (row >= rows) return;
  const int last = 4 * (lane + kWave * (N4 - 1));
  const bool live = !RAG || last < D;  // of the last chunk
  auto col = [&](int i) { return RAG && i == N4 - 1 && !live ? 0 : 4 * (lane + kWave * i); };
  const float* hr = h + (size_t)row * D;
  f32x4 v[N4], sc[N4], sh[N4];
#pragma unroll
  for (int i = 0; i < N4; ++i) v[i] = *reinterpret_cast<const f32x4*>(hr + col(i));
#pragma unroll
  for (int i = 0; i < N4; ++i) {
    sc[i] = *reinterpret_cast<const f32x4*>(scale + col(i));
    sh[i] = *reinterpret_cast<const f32x4*>(shift + col(i));
  }
  __builtin_amdgcn_sched_barrier(0);  // keep the modulation loads ahead of the reductions
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < N4; ++i) {
    const float t = (v[i].x + v[i].y) + (v[i].z + v[i].w);
    s += i < N4 - 1 || live ? t : 0.f;
  }
  const float mean = wave_sum(s) / (float)D;
  float q = 0.f;
#pragma unroll
  for (int i = 0; i < N4; ++i) {
    const float a = v[i].x - mean, b = v[i].y - mean, c = v[i].z - mean, d = v[i].w - mean;
    const float t = (a * a + b * b) + (c * c + d * d);
    q += i < N4 - 1 || live ? t : 0.f;
  }
  const float rstd = row_scale<TOut>(wave_sum(q) / (float)D + eps);
  TOut* ur = u + (size_t)row * D;
#pragma unroll
  for (int i = 0; i < N4; ++i) {
    if (i == N4 - 1 && !live) break;
    const f32x4 o = (v[i] - mean) * rstd * (1.0f + sc[i]) + sh[i];
    if constexpr (sizeof(TOut) == 2)
      *reinterpret_cast<bf16x4*>(ur + col(i)) = bf16x4{static_cast<bf16>(o[0]), static_cast<bf16>(o[1]),
                                                       static_cast<bf16>(o[2]), static_cast<bf16>(o[3])};
    else
      *reinterpret_cast<f32x4*>(ur + col(i)) = o;
  }
}

// ------------------------------------------------------------- final layer + Euler
// LayerNorm, modulation and the branch's head (up to 16 channels) on the fp32
// matrix cores, then the velocity and / or the Euler update x += dsigma v.  A
// block of four waves takes 16 consecutive trajectory rows of one branch of
// one sample, wave w their columns [w D/4, (w+1) D/4) in chunks of 16: lane
// (g, r) holds columns 4g .. 4g+3 of every chunk of row r, and of head row
// (output channel) r of W^T, which are the operands of four 16x16x4 MFMAs, so
// neither goes through LDS.  Row sums, squared
// deviations and the four waves' partial products meet in LDS, in wave order.
// HBM bound on long trajectories (D = 1536, 9664 rows, 59 MB: 38 us with
// the head in LDS and vector products, 26 us here), a chain of
// four short phases on short ones (D = 768, 800 rows: 12.0 -> 7.2 us).
constexpr int kFinalCout = 16;

template <int MAXC>
__global__ __launch_bounds__(256) void final_kernel(FinalArgs a) {
  constexpr int NW = 4, R = 16;
  __shared__ float rsum[NW][R], rsq[NW][R];
  __shared__ float part[NW][R][kFinalCout + 1];
  const int lane = threadIdx.x % kWave, wid = threadIdx.x / kWave;
  const int g = lane / 16, r = lane % 16;
  const int gv = (a.Nv + R - 1) / R, ga = (a.Na + R - 1) / R, per = gv + ga;
  const int b = blockIdx.x / per, j = blockIdx.x % per;
  const bool video = j < gv;
  const int t0 = video ? j * R : a.Nv + (j - gv) * R;
  const int tend = video ? a.Nv : a.Nv + a.Na;
  const int cout = video ? a.Cv : a.A;
  const int nc = a.D / 64;  // chunks of 16 columns per wave
  const int c0 = wid * (a.D / 4) + 4 * g;
  // rows past the branch and channels past the head read the last one of it;
  // what they give is never stored
  const float* hr = a.h + ((size_t)b * a.T + min(t0 + r, tend - 1)) * a.D + c0;
  const float* wr = (video ? a.wv : a.wa) + (size_t)min(r, cout - 1) * a.D + c0;
  // modulation and head: ahead of the reductions too where the registers
  // allow it, else (two waves per SIMD matter more) from L2 as they are used
  constexpr bool kAhead = MAXC <= 12;
  constexpr int MW = kAhead ? MAXC : 1;
  f32x4 u[MAXC], w[MW], sc[MW], sh[MW];
  auto load_mod = [&](int i, int at) {
    sc[at] = *reinterpret_cast<const f32x4*>(a.scale + c0 + 16 * i);
    sh[at] = *reinterpret_cast<const f32x4*>(a.shift + c0 + 16 * i);
    w[at] = *reinterpret_cast<const f32x4*>(wr + 16 * i);
  };
#pragma unroll
  for (int i = 0; i < MAXC; ++i)
    if (i < nc) u[i] = *reinterpret_cast<const f32x4*>(hr + 16 * i);
  if constexpr (kAhead) {
#pragma unroll
    for (int i = 0; i < MAXC; ++i)
      if (i < nc) load_mod(i, i);
  }
  __builtin_amdgcn_sched_barrier(0);  // keep these loads ahead of the reductions
  // sum over the columns of row r: lane, the row's four lanes, the four waves
  auto row_sum = [&](float v, float (*buf)[R]) {
    v += __shfl_xor(v, 16, 64);
    v += __shfl_xor(v, 32, 64);
    if (g == 0) buf[wid][r] = v;
    __syncthreads();
    return (buf[0][r] + buf[1][r]) + (buf[2][r] + buf[3][r]);
  };
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < MAXC; ++i)
    if (i < nc) s += (u[i].x + u[i].y) + (u[i].z + u[i].w);
  const float mean = row_sum(s, rsum) / (float)a.D;
  float q = 0.f;
#pragma unroll
  for (int i = 0; i < MAXC; ++i)
    if (i < nc) {
      u[i] -= mean;
      q += (u[i].x * u[i].x + u[i].y * u[i].y) + (u[i].z * u[i].z + u[i].w * u[i].w);
    }
  const float rstd = rsqrt_newton(row_sum(q, rsq) / (float)a.D + a.eps);
  // out^T = W^T u^T: lane (g, r) ends with channels 4g .. 4g+3 of row r
  // several accumulators: shorter sums, and no MFMA waits for the last
  f32x4 acc[2][4] = {};
#pragma unroll
  for (int i = 0; i < MAXC; ++i)
    if (i < nc) {
      const int at = kAhead ? i : 0;
      if constexpr (!kAhead) load_mod(i, 0);
      const f32x4 m = u[i] * rstd * (1.0f + sc[at]) + sh[at];
#pragma unroll
      for (int k = 0; k < 4; ++k) acc[i % 2][k] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[at][k], m[k], acc[i % 2][k], 0, 0, 0);
    }
  const f32x4 sum = ((acc[0][0] + acc[1][0]) + (acc[0][1] + acc[1][1])) +
                    ((acc[0][2] + acc[1][2]) + (acc[0][3] + acc[1][3]));
#pragma unroll
  for (int k = 0; k < 4; ++k) part[wid][r][4 * g + k] = sum[k];
  __syncthreads();
  const int row = threadIdx.x / kFinalCout, o = threadIdx.x % kFinalCout, t = t0 + row;
  if (t >= tend || o >= cout) return;
  const float vel = ((part[0][row][o] + part[1][row][o]) + (part[2][row][o] + part[3][row][o])) +
                    (video ? a.bv : a.ba)[o];
  const int traj = a.Nv * a.Cv + a.Na * a.A;
  const size_t idx = (size_t)b * traj + (video ? (size_t)t * a.Cv + o
                                               : (size_t)a.Nv * a.Cv + (size_t)(t - a.Nv) * a.A + o);
  if (a.v_out) a.v_out[idx] = vel;
  if (a.x) a.x[idx] += a.dsigma * vel;
}

// ------------------------------------------------------------- Residual Rescaling
// alpha (Eq. crr-alpha), cos and relative fit error (Eq. crr-gate) of one
// (sample, branch) from its float64 sums over nrows rows of D elements.
__device__ void rr_gate_stats(const RRGateArgs& a, int b, int br, int nrows, double sip, double sii, double saa) {
  const double n = (double)nrows * (double)a.D;
  const double den = fmax(saa / n, (double)a.eps);
  double alpha = (sip / n) / den;
  alpha = fmin(fmax(alpha, (double)a.alpha_min), (double)a.alpha_max);
  const bool ok_norm = sii > 0.0 && saa > 0.0;
  const double cosv = ok_norm ? sip / sqrt(sii * saa) : 0.0;
  const double r2 = fmax(sii - 2.0 * alpha * sip + alpha * alpha * saa, 0.0);
  const double fit = sii > 0.0 ? sqrt(r2) / sqrt(sii) : INFINITY;
  const bool pass = ok_norm && cosv >= (double)a.gamma_cos && fit <= (double)a.gamma_fit;
  const double v[8] = {sip, sii, saa, alpha, cosv, fit, pass ? 1.0 : 0.0, 0.0};
  const size_t at = ((size_t)b * 2 + br) * 8;
#pragma unroll
  for (int i = 0; i < 8; ++i) a.result[at + i] = v[i];
  // a host that decides reads them from its pinned buffer once the stream has
  // drained, without a copy command between the gate and that wait
  if (a.host)
#pragma unroll
    for (int i = 0; i < 8; ++i) a.host[at + i] = v[i];
}

// The gate in two launches, both in fixed summation orders.  Partials: blocks
// are laid out per (sample, branch): sample b owns gV = ceil(nV / 4) blocks
// over the rows of branch 0 (rows [0, Nv) then [Nv+Na, T), nV = T - Na of
// them) followed by gA = ceil(Na / 4) over branch 1 (rows [Nv, Nv+Na)).  Wave
// w of a block takes one row (all of its loads issued before any
// arithmetic; lanes past D, a multiple of 64, take no part in the last chunk),
// and the block adds its rows in wave order into one partial
// (row_sums[block][3]).  The second kernel, one block per (sample, branch),
// adds that pair's partials in block order and writes the statistics.
template <int MAXV>
__global__ __launch_bounds__(256) void rr_gate_partials_kernel(RRGateArgs a) {
  const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave;
  const int nV = a.T - a.Na;
  const int gV = (nV + 3) / 4, gA = (a.Na + 3) / 4, per = gV + gA;
  const int b = blockIdx.x / per, j = blockIdx.x % per;
  const bool br1 = j >= gV;
  const int i = (br1 ? j - gV : j) * 4 + w;  // row within the branch
  const bool valid = i < (br1 ? a.Na : nV);
  const int t = br1 ? a.Nv + i : (i < a.Nv ? i : i + a.Na);
  __shared__ double part[4][3];
  double sip = 0.0, sii = 0.0, saa = 0.0;
  if (valid) {
    const size_t off = ((size_t)b * a.T + t) * a.D;
    const f32x4* s4 = reinterpret_cast<const f32x4*>(a.hs + off);
    const f32x4* q4 = reinterpret_cast<const f32x4*>(a.hq + off);
    const f32x4* a4 = reinterpret_cast<const f32x4*>(a.pa + off);
    f32x4 sv[MAXV], qv[MAXV], av[MAXV];
#pragma unroll
    for (int k = 0; k < MAXV; ++k)
      if (4 * (lane + kWave * k) < a.D) {
        sv[k] = s4[lane + kWave * k];
        qv[k] = q4[lane + kWave * k];
        av[k] = a4[lane + kWave * k];
      }
#pragma unroll
    for (int k = 0; k < MAXV; ++k)
      if (4 * (lane + kWave * k) < a.D) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const double pi = (double)(sv[k][e] - qv[k][e]), pv = (double)av[k][e];
          sip += pi * pv;
          sii += pi * pi;
          saa += pv * pv;
        }
      }
    sip = wave_sum_d(sip);
    sii = wave_sum_d(sii);
    saa = wave_sum_d(saa);
  }
  if (lane == 0) {
    part[w][0] = sip;
    part[w][1] = sii;
    part[w][2] = saa;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double* out = a.row_sums + (size_t)blockIdx.x * 3;
    out[0] = (part[0][0] + part[1][0]) + (part[2][0] + part[3][0]);
    out[1] = (part[0][1] + part[1][1]) + (part[2][1] + part[3][1]);
    out[2] = (part[0][2] + part[1][2]) + (part[2][2] + part[3][2]);
  }
}

__global__ __launch_bounds__(256) void rr_gate_finish_kernel(RRGateArgs a) {
  const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave;
  const int b = blockIdx.x / 2, br = blockIdx.x % 2;
  const int nV = a.T - a.Na;
  const int gV = (nV + 3) / 4, gA = (a.Na + 3) / 4, per = gV + gA;
  const int first = b * per + (br ? gV : 0), cnt = br ? gA : gV;
  double s[3] = {0.0, 0.0, 0.0};
#pragma unroll 8
  for (int k = threadIdx.x; k < cnt; k += 256) {
    const double* p = a.row_sums + (size_t)(first + k) * 3;
    s[0] += p[0];
    s[1] += p[1];
    s[2] += p[2];
  }
  __shared__ double sh[3][4];
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const double v = wave_sum_d(s[c]);
    if (lane == 0) sh[c][w] = v;
  }
  __syncthreads();
  if (threadIdx.x == 0)
    rr_gate_stats(a, b, br, br ? a.Na : nV, (sh[0][0] + sh[0][1]) + (sh[0][2] + sh[0][3]),
                  (sh[1][0] + sh[1][1]) + (sh[1][2] + sh[1][3]), (sh[2][0] + sh[2][1]) + (sh[2][2] + sh[2][3]));
}

// h_e = h_s + alpha_{b,branch} R_a (Eq. residual-injection), in place on h.
// A thread updates kInjV float4 spaced one block width apart (all loads
// first; in the model one per thread measured fastest).  A float4 never
// straddles rows (D % 4 == 0); its sample and branch come from comparisons
// against the float4 offsets of the sample and branch boundaries (host:
// rows * D / 4 < 2^31).
constexpr int kInjV = 1;
__global__ __launch_bounds__(256) void rr_inject_kernel(float* __restrict__ h, const float* __restrict__ Ra,
                                                        const double* __restrict__ result, int B, int T, int D,
                                                        int Nv, int Na, const int* flag) {
  if (flag && *flag != 1) return;
  const int d4 = D / 4, td4 = T * d4, n4 = B * td4, lo = Nv * d4, hi = (Nv + Na) * d4;
  const int base = blockIdx.x * (256 * kInjV) + threadIdx.x;
  f32x4* h4 = reinterpret_cast<f32x4*>(h);
  const f32x4* r4 = reinterpret_cast<const f32x4*>(Ra);
  f32x4 hv[kInjV], rv[kInjV];
#pragma unroll
  for (int u = 0; u < kInjV; ++u) {
    const int i4 = base + 256 * u;
    if (i4 < n4) {
      hv[u] = h4[i4];
      rv[u] = r4[i4];
    }
  }
#pragma unroll
  for (int u = 0; u < kInjV; ++u) {
    const int i4 = base + 256 * u;
    if (i4 < n4) {
      int b = 0, r = i4;
      while (r >= td4) {
        r -= td4;
        ++b;
      }
      const int br = (r >= lo && r < hi) ? 1 : 0;
      const float al = (float)result[((size_t)b * 2 + br) * 8 + 3];
      h4[i4] = hv[u] + al * rv[u];
    }
  }
}

__global__ void rr_pre_middle_kernel(const float* __restrict__ h, float* __restrict__ hq,
                                     float* __restrict__ pa, int64_t n4, const int* flag) {
  if (flag && *flag != 0) return;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n4) return;
  const float4 hv = reinterpret_cast<const float4*>(h)[i];
  const float4 qv = reinterpret_cast<const float4*>(hq)[i];
  reinterpret_cast<float4*>(pa)[i] = make_float4(hv.x - qv.x, hv.y - qv.y, hv.z - qv.z, hv.w - qv.w);
  reinterpret_cast<float4*>(hq)[i] = hv;
}

__global__ void rr_refresh_kernel(const float* __restrict__ h, const float* __restrict__ hq,
                                  float* __restrict__ Ra, int64_t n4, const int* flag) {
  if (flag && *flag != 0) return;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n4) return;
  const float4 hv = reinterpret_cast<const float4*>(h)[i];
  const float4 qv = reinterpret_cast<const float4*>(hq)[i];
  reinterpret_cast<float4*>(Ra)[i] = make_float4(hv.x - qv.x, hv.y - qv.y, hv.z - qv.z, hv.w - qv.w);
}

// Device-side reuse decision: AND of the pass bits over samples and branches
// (or forced), written as a flag that predicates the following launches.
__global__ void rr_decide_kernel(const double* __restrict__ result, int B, int nbranch, int force_accept, int* flag,
                                 double* hist_stats, int* hist_flag) {
  if (threadIdx.x != 0) return;
  int all = 1;
  for (int i = 0; i < B * 2; ++i) {
    const double* r = result + (size_t)i * 8;
    if (i % 2 < nbranch) all &= r[6] != 0.0;
    hist_stats[i * 3 + 0] = r[3];
    hist_stats[i * 3 + 1] = r[4];
    hist_stats[i * 3 + 2] = r[5];
  }
  const int accept = force_accept ? 1 : all;
  *flag = accept;
  *hist_flag = accept;
}

// Condition of the action model of an independent pair: observation tokens,
// then context tokens (e.g. the video model's latent), zero-padded to Co.
__global__ void pack_condition_kernel(const float* __restrict__ obs, int n_obs, int c_obs,
                                      const float* __restrict__ ctx, int n_ctx, int c_ctx, int64_t ctx_stride,
                                      float* __restrict__ cond, int B, int Co) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int nt = n_obs + n_ctx;
  if (i >= (int64_t)B * nt * Co) return;
  const int c = (int)(i % Co);
  const int t = (int)((i / Co) % nt);
  const int b = (int)(i / ((int64_t)Co * nt));
  float v = 0.f;
  if (t < n_obs) {
    if (c < c_obs) v = obs[((int64_t)b * n_obs + t) * c_obs + c];
  } else if (c < c_ctx) {
    v = ctx[(int64_t)b * ctx_stride + (int64_t)(t - n_obs) * c_ctx + c];
  }
  cond[i] = v;
}

__global__ void copy_f32_kernel(const float* __restrict__ src, float* __restrict__ dst, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = src[i];
}

// float4 copy, four per thread spaced one block width apart (n4 float4)
__global__ __launch_bounds__(256) void copy_f32x4_kernel(const f32x4* __restrict__ src, f32x4* __restrict__ dst,
                                                         int64_t n4) {
  const int64_t base = (int64_t)blockIdx.x * 1024 + threadIdx.x;
  f32x4 v[4];
#pragma unroll
  for (int u = 0; u < 4; ++u)
    if (base + 256 * u < n4) v[u] = src[base + 256 * u];
#pragma unroll
  for (int u = 0; u < 4; ++u)
    if (base + 256 * u < n4) dst[base + 256 * u] = v[u];
}

// ------------------------------------------------------------- Trajectory Remapping
// Four consecutive floats p[0 .. cnt) (zeros past cnt): one 16-byte load when
// VEC (the caller has checked the alignment and cnt == 4), else scalar loads.
template <bool VEC>
__device__ __forceinline__ f32x4 load_group(const float* p, int64_t cnt) {
  if constexpr (VEC) {
    return *reinterpret_cast<const f32x4*>(p);
  } else {
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (u < cnt) v[u] = p[u];
    return v;
  }
}

// Float64 sum of ((p - q) * scale)^2 over elements [4 g0, min(4 g1, n)) of a
// run, by the 256 threads of a block: thread t takes the 4-element groups
// t, t + 256, ... (four groups in flight per step), and each group's elements
// in order.  Both instantiations add in exactly this order, so the result
// does not depend on whether the 16-byte path was taken.
template <bool VEC>
__device__ __forceinline__ double run_sq_sum(const float* p, const float* q, double scale, int64_t g0,
                                             int64_t g1, int64_t n) {
  const int64_t full = n / 4 < g1 ? n / 4 : g1;  // groups with all four elements
  double s = 0.0;
  int64_t g = g0 + threadIdx.x;
  for (; g + 3 * 256 < full; g += 4 * 256) {
    f32x4 x[4], y[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      x[u] = load_group<VEC>(p + 4 * (g + u * 256), 4);
      y[u] = load_group<VEC>(q + 4 * (g + u * 256), 4);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const double d = ((double)x[u][e] - (double)y[u][e]) * scale;
        s = fma(d, d, s);
      }
  }
  for (; g < g1; g += 256) {
    const int64_t cnt = n - 4 * g < 4 ? n - 4 * g : 4;
    const f32x4 x = load_group<VEC>(p + 4 * g, VEC ? 4 : cnt), y = load_group<VEC>(q + 4 * g, VEC ? 4 : cnt);
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (e < cnt) {
        const double d = ((double)x[e] - (double)y[e]) * scale;
        s = fma(d, d, s);
      }
  }
  return s;
}

// rms of (x^r - x_bar)/sigma_r per (sample, branch) over the whole branch: each
// branch is cut into reduce_chunks(n) runs of whole 4-element groups, one
// block per run sums its squares (float64); then the run sums are added in a
// fixed order (the same bits on every call) and turned into the remap
// coefficient sigma_b0 / (sigma_r rms) (0 for a zero direction).  Up to 2048
// blocks of the remap itself (one round of the chip) every one of them does
// that for the branches it touches while its loads are in flight, two launches
// in all: 4 x 154 K elements 12.4 -> 9.7 us.  Beyond, repeating the sum in
// every block costs more than the launch it saves (16 M elements: 55 us against
// 52) and one block per (sample, branch) does it in between.
template <bool VEC>
__global__ __launch_bounds__(256) void remap_partial_kernel(RemapArgs a) {
  __shared__ double sh[16];
  const int sb = blockIdx.y;  // sample * 2 + branch
  const int b = sb / 2, br = sb % 2;
  const int64_t traj = (int64_t)a.Nv * a.Cv + (int64_t)a.Na * a.A;
  const int64_t lo = br == 0 ? 0 : (int64_t)a.Nv * a.Cv;
  const int64_t n = br == 0 ? (int64_t)a.Nv * a.Cv : (int64_t)a.Na * a.A;
  const int nch = reduce_chunks(n);
  if ((int)blockIdx.x >= nch) return;
  const int64_t ng = (n + 3) / 4, per = (ng + nch - 1) / nch;
  const int64_t g0 = (int64_t)blockIdx.x * per;
  const int64_t g1 = g0 + per < ng ? g0 + per : ng;
  const size_t off = (size_t)b * traj + lo;
  double s = run_sq_sum<VEC>(a.x_r + off, a.x_bar + off, 1.0 / (double)a.sigma_r, g0, g1, n);
  s = block_sum_d(s, sh);
  if (threadIdx.x == 0) a.partial[(size_t)sb * kRemapChunks + blockIdx.x] = s;
}

// Fixed-order sum of run sums p[0 .. n): thread t adds runs t, t + 256, ...
// in turn, then the 256 thread sums combine as block_sum_d does.
__device__ __forceinline__ double runs_sum(const double* p, int n, double* sh) {
  double s = 0.0;
  for (int c = threadIdx.x; c < n; c += 256) s += p[c];
  return block_sum_d(s, sh);
}

// x = x_bar + sigma_b0 d with d = ((x^r - x_bar) / sigma_r) / rms
__device__ __forceinline__ double remap_coef(const RemapArgs& a, int sb, double* sh) {
  const int br = sb % 2;
  const int64_t n = br == 0 ? (int64_t)a.Nv * a.Cv : (int64_t)a.Na * a.A;
  const double s = runs_sum(a.partial + (size_t)sb * kRemapChunks, reduce_chunks(n), sh);
  const double rms = n > 0 ? sqrt(s / (double)n) : 0.0;
  return rms > 0.0 ? (double)a.sigma_b0 / ((double)a.sigma_r * rms) : 0.0;
}

__global__ __launch_bounds__(256) void remap_finish_kernel(RemapArgs a) {
  __shared__ double sh[16];
  const double c = remap_coef(a, blockIdx.x, sh);
  if (threadIdx.x == 0) a.coef[blockIdx.x] = c;
}

// x[j] = x_bar[j+shift] + sigma_b0 d[j+shift] on mapped slots, sigma_b0 eps[j]
// elsewhere.  Slot j of a branch of width w is mapped when j + shift < slots,
// i.e. when the element index within the branch plus shift * w stays inside
// the branch.  Grid (runs of 256 thread items, sample): with VEC an item is
// four consecutive elements with 16-byte loads and stores (the host has checked
// that the pointers, both branch lengths and both shifted offsets are multiples
// of four floats, so a group lies in one branch and is mapped or unmapped as a
// whole); otherwise one element.  Every element is computed by the same
// expression either way.
__device__ __forceinline__ float remap_value(float xb, float xr, double coef) {
  const double x = (double)xb;
  return (float)(x + ((double)xr - x) * coef);
}

template <bool VEC, bool FUSED>
__global__ __launch_bounds__(256) void remap_apply_kernel(RemapArgs a) {
  constexpr int E = VEC ? 4 : 1;
  typedef float item __attribute__((ext_vector_type(E)));
  __shared__ double sh[16];
  const int64_t traj = (int64_t)a.Nv * a.Cv + (int64_t)a.Na * a.A;
  const int64_t nv = (int64_t)a.Nv * a.Cv;
  const int b = blockIdx.y;
  const size_t base = (size_t)b * traj;
  const int64_t i0 = (int64_t)blockIdx.x * (256 * E), i = i0 + (int64_t)threadIdx.x * E;
  const bool live = i < traj, video = i < nv;
  if (!FUSED && !live) return;
  const int64_t src = i + (video ? (int64_t)a.shift_video * a.Cv : (int64_t)a.shift_action * a.A);
  const bool mapped = src < (video ? nv : traj);
  item xb{}, xr{};
  if (live && mapped) {
    xb = *reinterpret_cast<const item*>(a.x_bar + base + src);
    xr = *reinterpret_cast<const item*>(a.x_r + base + src);
  }
  double cv = 0.0, ca = 0.0;
  if constexpr (FUSED) {
    // branches this block touches (uniform over the block)
    if (i0 < nv) cv = remap_coef(a, b * 2, sh);
    if (i0 + 256 * E > nv) ca = remap_coef(a, b * 2 + 1, sh);
    if (!live) return;
  }
  item out;
  if (mapped) {
    const double c = FUSED ? (video ? cv : ca) : a.coef[b * 2 + (video ? 0 : 1)];
#pragma unroll
    for (int k = 0; k < E; ++k) out[k] = remap_value(xb[k], xr[k], c);
  } else {
    out = a.sigma_b0 * *reinterpret_cast<const item*>(a.noise + base + i);
  }
  *reinterpret_cast<item*>(a.x_out + base + i) = out;
}

// ------------------------------------------------------------- Observation Rebinding
struct OrSumArgs {
  const float* u_hat[WAM_MAX_COMPONENTS];
  const float* u[WAM_MAX_COMPONENTS];
  int64_t n[WAM_MAX_COMPONENTS];
  double inv_delta[WAM_MAX_COMPONENTS];
  int vec;  // bit m: component m takes 16-byte loads
  double* sums;
};

// Run sums of ((u_hat - u) / delta)^2 of component blockIdx.y, run blockIdx.x
// of reduce_chunks(n) runs of whole 4-element groups (float64, the order of
// run_sq_sum), stored straight into the host's pinned buffer; the host adds the
// runs in order.
__global__ __launch_bounds__(256) void or_sums_kernel(OrSumArgs a) {
  __shared__ double sh[16];
  const int m = blockIdx.y;
  const int64_t n = a.n[m];
  const int nch = reduce_chunks(n);
  if ((int)blockIdx.x >= nch) return;
  const int64_t ng = (n + 3) / 4, per = (ng + nch - 1) / nch;
  const int64_t g0 = (int64_t)blockIdx.x * per;
  const int64_t g1 = g0 + per < ng ? g0 + per : ng;
  double s = a.vec >> m & 1 ? run_sq_sum<true>(a.u_hat[m], a.u[m], a.inv_delta[m], g0, g1, n)
                            : run_sq_sum<false>(a.u_hat[m], a.u[m], a.inv_delta[m], g0, g1, n);
  s = block_sum_d(s, sh);
  if (threadIdx.x == 0) a.sums[(size_t)m * kRemapChunks + blockIdx.x] = s;
}

}  // namespace

// ================================================================ launchers
hipError_t launch_timestep_mlp(float sigma, const float* w1, const float* b1, const float* w2, const float* b2,
                               float* a1, float* silu_c, int D, hipStream_t s) {
  if (D > 2048) return hipErrorInvalidValue;
  const int grid = (D + kSgN - 1) / kSgN;
  launch_k(small_gemv_silu_kernel<true>, grid, kSgN * kSgK, 0, s, sigma, nullptr, w1, b1, a1, kTimeDim, D);
  launch_k(small_gemv_silu_kernel<false>, grid, kSgN * kSgK, 0, s, 0.f, a1, w2, b2, silu_c, D, D);
  return hipGetLastError();
}

hipError_t launch_gemv(const float* x, const void* W, bool w_bf16, const float* b, float* y,
                       float* partial, int K, int N, int in_act, int out_act, hipStream_t s) {
  if (N % kGemvVec) return hipErrorInvalidValue;
  const int nchunk = (K + kGemvKc - 1) / kGemvKc;
  dim3 grid((N / kGemvVec + 255) / 256, nchunk);
  if (w_bf16)
    launch_k(gemv_partial_kernel<bf16>, grid, 256, 0, s, x, (const bf16*)W, partial, K, N, in_act);
  else
    launch_k(gemv_partial_kernel<float>, grid, 256, 0, s, x, (const float*)W, partial, K, N, in_act);
  launch_k(gemv_reduce_kernel, (N + 255) / 256, 256, 0, s, partial, b, y, nchunk, N, out_act);
  return hipGetLastError();
}

hipError_t launch_embed(const EmbedArgs& a, hipStream_t s) {
  if (a.Cv > 64 || a.A > 64 || a.Co > 64) return hipErrorInvalidValue;
  // every branch present has at least one channel (the clamp reads row c-1)
  const bool chans = (a.Nv == 0 || a.Cv >= 1) && (a.Na == 0 || a.A >= 1) && (a.No == 0 || a.Co >= 1);
  if (a.D % 4 == 0 && a.D <= 2048 && a.Cv <= kEmbedC && a.A <= kEmbedC && a.Co <= kEmbedC && chans) {
    const int threads = (a.D / 4 + kWave - 1) / kWave * kWave;
    // rows per block: share the weight reads where the grid stays above
    // ~1000 blocks, one row per block for short sequences (latency)
    const long rows = (long)a.B * a.T;
    if (rows >= 8192)
      launch_k(embed_v4_kernel<8>, a.B * embed_blocks_per_sample(a.Nv, a.Na, a.No, 8), threads, 0, s, a);
    else if (rows >= 4096)
      launch_k(embed_v4_kernel<4>, a.B * embed_blocks_per_sample(a.Nv, a.Na, a.No, 4), threads, 0, s, a);
    else if (rows >= 2048)
      launch_k(embed_v4_kernel<2>, a.B * embed_blocks_per_sample(a.Nv, a.Na, a.No, 2), threads, 0, s, a);
    else
      launch_k(embed_v4_kernel<1>, a.B * embed_blocks_per_sample(a.Nv, a.Na, a.No, 1), threads, 0, s, a);
  } else {
    launch_k(embed_kernel, a.B * a.T, 256, 0, s, a);
  }
  return hipGetLastError();
}

template <int N4>
void launch_ln_t(const float* h, const float* shift, const float* scale, void* u, int rows, int D, float eps,
                 bool bf16_out, hipStream_t s, const int* skip) {
  const int grid = (rows + 3) / 4;
  bf16* ub = static_cast<bf16*>(u);
  float* uf = static_cast<float*>(u);
  if (D % 256 == 0) {
    if (bf16_out) launch_k(ln_modulate_kernel<N4, false, bf16>, grid, 256, 0, s, h, shift, scale, ub, rows, D, eps, skip);
    else launch_k(ln_modulate_kernel<N4, false, float>, grid, 256, 0, s, h, shift, scale, uf, rows, D, eps, skip);
  } else {
    if (bf16_out) launch_k(ln_modulate_kernel<N4, true, bf16>, grid, 256, 0, s, h, shift, scale, ub, rows, D, eps, skip);
    else launch_k(ln_modulate_kernel<N4, true, float>, grid, 256, 0, s, h, shift, scale, uf, rows, D, eps, skip);
  }
}

hipError_t launch_ln_modulate(const float* h, const float* shift, const float* scale, void* u,
                              int rows, int D, float eps, bool bf16_out, hipStream_t s, const int* skip) {
  if (D % kWave || D > 2048) return hipErrorInvalidValue;
  switch ((D + 255) / 256) {
    case 1: launch_ln_t<1>(h, shift, scale, u, rows, D, eps, bf16_out, s, skip); break;
    case 2: launch_ln_t<2>(h, shift, scale, u, rows, D, eps, bf16_out, s, skip); break;
    case 3: launch_ln_t<3>(h, shift, scale, u, rows, D, eps, bf16_out, s, skip); break;
    case 4: launch_ln_t<4>(h, shift, scale, u, rows, D, eps, bf16_out, s, skip); break;
    case 5: launch_ln_t<5>(h, shift, scale, u, rows, D, eps, bf16_out, s, skip); break;
    case 6: launch_ln_t<6>(h, shift, scale, u, rows, D, eps, bf16_out, s, skip); break;
    case 7: launch_ln_t<7>(h, shift, scale, u, rows, D, eps, bf16_out, s, skip); break;
    default: launch_ln_t<8>(h, shift, scale, u, rows, D, eps, bf16_out, s, skip); break;
  }
  return hipGetLastError();
}

hipError_t launch_final(const FinalArgs& a, hipStream_t s) {
  if (a.D % kWave || a.D > 2048 || a.Cv > kFinalCout || a.A > kFinalCout) return hipErrorInvalidValue;
  const int blocks = a.B * ((a.Nv + 15) / 16 + (a.Na + 15) / 16);
  if (blocks == 0) return hipSuccess;
  // registers for the chunks D needs
  const int nc = a.D / 64;
  if (nc <= 4) launch_k(final_kernel<4>, blocks, 256, 0, s, a);
  else if (nc <= 8) launch_k(final_kernel<8>, blocks, 256, 0, s, a);
  else if (nc <= 12) launch_k(final_kernel<12>, blocks, 256, 0, s, a);
  else if (nc <= 16) launch_k(final_kernel<16>, blocks, 256, 0, s, a);
  else if (nc <= 24) launch_k(final_kernel<24>, blocks, 256, 0, s, a);
  else launch_k(final_kernel<32>, blocks, 256, 0, s, a);
  return hipGetLastError();
}

hipError_t launch_rr_gate(const RRGateArgs& a, hipStream_t s) {
  if (a.D % kWave || a.D > 2048) return hipErrorInvalidValue;
  const int per = (a.T - a.Na + 3) / 4 + (a.Na + 3) / 4;
  launch_k(rr_gate_partials_kernel<8>, (unsigned)(a.B * per), 256, 0, s, a);
  launch_k(rr_gate_finish_kernel, (unsigned)(a.B * 2), 256, 0, s, a);
  return hipGetLastError();
}

hipError_t launch_rr_inject(float* h, const float* Ra, const double* result, int B, int T, int D,
                            int Nv, int Na, hipStream_t s, const int* flag) {
  const int64_t n4 = (int64_t)B * T * D / 4;
  if (D % 4 || n4 >= (int64_t)1 << 31) return hipErrorInvalidValue;
  const unsigned grid = (unsigned)((n4 + 256 * kInjV - 1) / (256 * kInjV));
  launch_k(rr_inject_kernel, grid, 256, 0, s, h, Ra, result, B, T, D, Nv, Na, flag);
  return hipGetLastError();
}

hipError_t launch_rr_pre_middle(const float* h, float* hq, float* pa, int64_t n, hipStream_t s,
                                const int* flag) {
  const int64_t n4 = n / 4;
  launch_k(rr_pre_middle_kernel, (unsigned)((n4 + 255) / 256), 256, 0, s, h, hq, pa, n4, flag);
  return hipGetLastError();
}

hipError_t launch_rr_refresh(const float* h, const float* hq, float* Ra, int64_t n, hipStream_t s,
                             const int* flag) {
  const int64_t n4 = n / 4;
  launch_k(rr_refresh_kernel, (unsigned)((n4 + 255) / 256), 256, 0, s, h, hq, Ra, n4, flag);
  return hipGetLastError();
}

hipError_t launch_rr_decide(const double* result, int B, int nbranch, int force_accept, int* flag,
                            double* hist_stats, int* hist_flag, hipStream_t s) {
  launch_k(rr_decide_kernel, 1, 64, 0, s, result, B, nbranch, force_accept, flag, hist_stats, hist_flag);
  return hipGetLastError();
}

hipError_t launch_pack_condition(const float* obs, int n_obs, int c_obs, const float* ctx, int n_ctx, int c_ctx,
                                 int64_t ctx_stride, float* cond, int B, int Co, hipStream_t s) {
  const int64_t n = (int64_t)B * (n_obs + n_ctx) * Co;
  if (n == 0) return hipSuccess;
  launch_k(pack_condition_kernel, (unsigned)((n + 255) / 256), 256, 0, s, obs, n_obs, c_obs, ctx, n_ctx, c_ctx,
           ctx_stride, cond, B, Co);
  return hipGetLastError();
}

hipError_t launch_copy_f32(const float* src, float* dst, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  if (n % 4 == 0 && reinterpret_cast<uintptr_t>(src) % 16 == 0 && reinterpret_cast<uintptr_t>(dst) % 16 == 0) {
    const int64_t n4 = n / 4;
    launch_k(copy_f32x4_kernel, (unsigned)((n4 + 1023) / 1024), 256, 0, s, reinterpret_cast<const f32x4*>(src),
             reinterpret_cast<f32x4*>(dst), n4);
  } else {
    launch_k(copy_f32_kernel, (unsigned)((n + 255) / 256), 256, 0, s, src, dst, n);
  }
  return hipGetLastError();
}

namespace {
bool aligned16(const void* p) { return reinterpret_cast<uintptr_t>(p) % 16 == 0; }
}  // namespace

hipError_t launch_remap(const RemapArgs& a, hipStream_t s) {
  const int64_t nv = (int64_t)a.Nv * a.Cv, na = (int64_t)a.Na * a.A, traj = nv + na;
  // 16-byte path: every group of four floats starts 16-byte aligned in each
  // array, in its branch and at its shifted source
  const bool sums_vec = aligned16(a.x_r) && aligned16(a.x_bar) && nv % 4 == 0 && na % 4 == 0;
  const bool apply_vec = sums_vec && aligned16(a.noise) && aligned16(a.x_out) &&
                         ((int64_t)a.shift_video * a.Cv) % 4 == 0 && ((int64_t)a.shift_action * a.A) % 4 == 0;
  const int nch = std::max(reduce_chunks(nv), reduce_chunks(na));
  if (sums_vec)
    launch_k(remap_partial_kernel<true>, dim3(nch, a.B * 2), 256, 0, s, a);
  else
    launch_k(remap_partial_kernel<false>, dim3(nch, a.B * 2), 256, 0, s, a);
  const int64_t items = apply_vec ? traj / 4 : traj;
  const dim3 grid((unsigned)((items + 255) / 256), a.B);
  if ((int64_t)grid.x * a.B <= 2048) {
    if (apply_vec) launch_k(remap_apply_kernel<true, true>, grid, 256, 0, s, a);
    else launch_k(remap_apply_kernel<false, true>, grid, 256, 0, s, a);
  } else {
    launch_k(remap_finish_kernel, a.B * 2, 256, 0, s, a);
    if (apply_vec) launch_k(remap_apply_kernel<true, false>, grid, 256, 0, s, a);
    else launch_k(remap_apply_kernel<false, false>, grid, 256, 0, s, a);
  }
  return hipGetLastError();
}

hipError_t launch_or_sums(int n_comp, const float* const* u_hat, const float* const* u,
                          const int64_t* n, const double* delta, double* sums, hipStream_t s) {
  if (n_comp < 1 || n_comp > WAM_MAX_COMPONENTS) return hipErrorInvalidValue;
  OrSumArgs a{};
  for (int m = 0; m < n_comp; ++m) {
    a.u_hat[m] = u_hat[m];
    a.u[m] = u[m];
    a.n[m] = n[m];
    a.inv_delta[m] = 1.0 / delta[m];
    if (aligned16(u_hat[m]) && aligned16(u[m]) && n[m] % 4 == 0) a.vec |= 1 << m;
  }
  a.sums = sums;
  int nch = 1;
  for (int m = 0; m < n_comp; ++m) nch = std::max(nch, reduce_chunks(n[m]));
  launch_k(or_sums_kernel, dim3(nch, n_comp), 256, 0, s, a);
  return hipGetLastError();
}

}  // namespace wam

// ================================================================ no-alloc remap
// Trajectory Remapping for callers that cannot allocate device memory (code
// under graph capture, tight serving loops): the rms and run-sum scratch of
// the remap kernels lives in this file-scope device array instead of a
// workspace.  Each GPU holds its own copy until the process ends; its device
// address is looked up once per device (with that device current) and only
// that address is ever handed to kernels or copies.
namespace wam {
namespace {

constexpr int kNoAllocScratchDoubles = WAM_MAX_BATCH * 2 * (1 + kRemapChunks);  // 256.3 KiB
constexpr int kMaxDevices = 64;

__device__ __align__(256) double scratch[kNoAllocScratchDoubles];

std::mutex g_scratch_mu;
double* g_scratch_ptr[kMaxDevices] = {};

thread_local std::string t_noalloc_err;

int noalloc_fail(int code, const char* msg) {
  t_noalloc_err = msg;
  return code;
}

// Device address of this GPU's copy of `scratch` (looked up on first use).
int scratch_for_current_device(double** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices)
    return noalloc_fail(WAM_E_HIP, "wam_remap_noalloc: no current device");
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p)
      return noalloc_fail(WAM_E_HIP, "wam_remap_noalloc: hipGetSymbolAddress of the scratch array failed");
    g_scratch_ptr[dev] = static_cast<double*>(p);
  }
  *out = g_scratch_ptr[dev];
  return WAM_OK;
}

}  // namespace
}  // namespace wam

extern "C" {

const char* wam_noalloc_last_error(void) { return wam::t_noalloc_err.c_str(); }

int wam_remap_noalloc(const wam_config* cfg, const wam_remap_args* a, void* hip_stream) {
  using namespace wam;
  if (!cfg || !a) return noalloc_fail(WAM_E_ARG, "wam_remap_noalloc: null argument");
  if (cfg->B < 1 || cfg->B > WAM_MAX_BATCH)
    return noalloc_fail(WAM_E_SHAPE, "wam_remap_noalloc: batch must be 1..WAM_MAX_BATCH (16): the static "
                                     "scratch holds 16 x 2 x 1025 float64 sums");
  if (cfg->Nv < 0 || cfg->Na < 0 || cfg->Cv < 1 || cfg->A < 1 || cfg->Nv + cfg->Na < 1)
    return noalloc_fail(WAM_E_SHAPE, "wam_remap_noalloc: need Nv, Na >= 0, Nv + Na >= 1, Cv, A >= 1");
  const int64_t traj = (int64_t)cfg->Nv * cfg->Cv + (int64_t)cfg->Na * cfg->A;
  if (traj * cfg->B > (int64_t)INT32_MAX)
    return noalloc_fail(WAM_E_SHAPE, "wam_remap_noalloc: B * traj must fit in 31 bits");
  if (!a->x_bar || !a->x_r || !a->noise || !a->x_out)
    return noalloc_fail(WAM_E_ARG, "wam_remap_noalloc: null remap argument");
  if (!(a->sigma_r > 0.f)) return noalloc_fail(WAM_E_ARG, "wam_remap_noalloc: sigma_r must be > 0");
  if (!(a->sigma_b0 >= 0.f)) return noalloc_fail(WAM_E_ARG, "wam_remap_noalloc: sigma_b0 must be >= 0");
  if (a->shift_action < 0 || a->shift_video < 0)
    return noalloc_fail(WAM_E_ARG, "wam_remap_noalloc: shifts must be >= 0");
  if (a->x_out == a->x_bar || a->x_out == a->x_r)
    return noalloc_fail(WAM_E_ARG, "wam_remap_noalloc: x_out must not alias inputs");
  double* sc = nullptr;
  int st = scratch_for_current_device(&sc);
  if (st) return st;
  RemapArgs r{a->x_bar, a->x_r, a->noise, a->x_out, sc, sc + 2 * cfg->B, a->sigma_r, a->sigma_b0,
              a->shift_action, a->shift_video, cfg->B, cfg->Nv, cfg->Cv, cfg->Na, cfg->A};
  if (launch_remap(r, static_cast<hipStream_t>(hip_stream)) != hipSuccess)
    return noalloc_fail(WAM_E_HIP, "wam_remap_noalloc: kernel launch failed");
  return WAM_OK;
}

}  // extern "C"
