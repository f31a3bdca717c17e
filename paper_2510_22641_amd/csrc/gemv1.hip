// One input row against a matrix, weight streaming (the batch-1 draft and greedy steps):
//  * gemv1_kernel - a wave holds the whole input row in registers and streams two weight rows.
//  * gemv1k_kernel - rows of 2048 and more: a block's four waves split K over its eight weight rows.
// Bound: HBM bytes of W, and a launch's fixed latency (arguments, inputs, weights, reduction).
#include "device.h"
#include "gemv_common.h"
#include "kernels.h"

#include <hip/hip_ext.h>

#include <climits>

namespace ssd {

namespace {

// One input row, K <= 512 * KP: the register path of the draft and greedy steps.  A wave's 64
// lanes hold the whole input row in registers (lane l owns elements p*512 + 8l .. +7 of every
// piece p), so the norm statistics are wave reductions and nothing is staged in LDS: each wave
// requests its inputs, then both weight rows, then the norm's gain (and shift), and computes the
// statistics while the weights are in flight.  NORM is the input transform (a template parameter
// so that rows without one keep no gain registers); NORM_SOFTMAX turns the row into per-group
// softmax probabilities (the folded cross-attention's second product).
template <typename WT, int KP, int NORM, int KIND>
__global__ __launch_bounds__(256) void gemv1_kernel(const LinearArgs a) {
  __shared__ float rv[GV_WAVES][1];
  __shared__ int ri[GV_WAVES][1];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int K = a.K;
  const bool gated = epi_gated<KIND>(a), qkv = epi_is<KIND>(a, EPI_QKV);
  const int n_total = qkv ? 3 * a.n_per : a.n_per;
  const int n_pairs = gated ? a.n_per : (n_total + 1) / 2;
  const int pr = blockIdx.x * GV_WAVES + wave;
  constexpr bool rms = NORM == NORM_RMS, ln = NORM == NORM_LN;

  // inputs first (the wait counter retires loads in issue order); clamped, never conditional
  float xv[KP][8];
#pragma unroll
  for (int p = 0; p < KP; ++p) {
    const int e = min(p * 512 + lane * 8, K - 8);
    const float4 x0 = *reinterpret_cast<const float4*>(a.x + e);
    const float4 x1 = *reinterpret_cast<const float4*>(a.x + e + 4);
    xv[p][0] = x0.x; xv[p][1] = x0.y; xv[p][2] = x0.z; xv[p][3] = x0.w;
    xv[p][4] = x1.x; xv[p][5] = x1.y; xv[p][6] = x1.z; xv[p][7] = x1.w;
  }
  // NORM_SOFTMAX with a pre-scale row: that row (at most 2048 floats) is requested with the
  // inputs, before the weights, so that its reduction and the softmax overlap the weight stream
  constexpr int PRE = NORM == NORM_SOFTMAX ? 8 : 1;
  float4 prev[PRE];
  if (NORM == NORM_SOFTMAX && a.pre_row) {
#pragma unroll
    for (int u = 0; u < PRE; ++u) {
      const int e = min(lane * 4 + u * 256, a.pre_len - 4);
      prev[u] = *reinterpret_cast<const float4*>(a.pre_row + e);
    }
  }
  const RowPair<WT> r = row_pair<WT, KIND>(a, n_total, pr < n_pairs ? pr : 0);
  const bool live = pr < n_pairs;
  // requested before the weights, as vector loads (the wait counter retires loads in issue order):
  // the sequence length, and the residual values this wave's epilogue adds
  int vzero;
  asm volatile("v_mov_b32 %0, 0" : "=v"(vzero));
  const int qlen = qkv ? a.kv.seq_len[vzero] : 0;
  float yold[2][1] = {{0.f}, {0.f}};
  if (epi_is<KIND>(a, EPI_RESID) || epi_is<KIND>(a, EPI_BIAS_RESID)) {
    const float* src = epi_is<KIND>(a, EPI_RESID) ? a.y : a.resid;
    const float* from = src ? src : a.x;  // no residual: a valid address, not used
    const float y0 = from[(src && r.ok0 ? r.n0 : 0) + vzero], y1 = from[(src && r.ok1 ? r.n1 : 0) + vzero];
    yold[0][0] = src ? y0 : 0.f;
    yold[1][0] = src ? y1 : 0.f;
  }
  Vec8<WT> w[2][KP];
  load_pieces<WT, KP>(w, r, 0, K, lane);
  QkvPre pre = {};
  if (qkv) {
    const int HD = a.n_per, mat = r.n0 >= HD ? (r.n0 >= 2 * HD ? 2 : 1) : 0;
    pre = qkv_pre(a, mat, r.n0 - mat * HD, 0, qlen + a.kv.pos_off);
  }
  Vec8<float> gv[rms || ln ? KP : 1], sv[ln ? KP : 1];
  if (rms || ln) {
#pragma unroll
    for (int p = 0; p < KP; ++p) gv[p].load(a.gain + min(p * 512 + lane * 8, K - 8));
  }
  if (ln) {
#pragma unroll
    for (int p = 0; p < KP; ++p) sv[p].load(a.shift + min(p * 512 + lane * 8, K - 8));
  }

  if (NORM == NORM_SOFTMAX) {
    // softmax over groups of a.group inputs: a group is a.group / 8 consecutive lanes of a piece
    // (512 is a multiple of the group, so groups never straddle pieces, and K of whole groups)
    const int gl = a.group >> 3;
    if (a.pre_row) {
      // scale by 1 / rms of the row the scores came from (every wave reads that row in full;
      // clamped re-reads past pre_len count as zero)
      float s2 = 0.f;
#pragma unroll
      for (int u = 0; u < PRE; ++u)
        if (lane * 4 + u * 256 < a.pre_len)
          s2 += (prev[u].x * prev[u].x + prev[u].y * prev[u].y) +
                (prev[u].z * prev[u].z + prev[u].w * prev[u].w);
      s2 = wave_sum(s2);
      const float sc = 1.0f / sqrtf(s2 / (float)a.pre_len + a.eps);
#pragma unroll
      for (int p = 0; p < KP; ++p)
#pragma unroll
        for (int e = 0; e < 8; ++e) xv[p][e] *= sc;
    }
#pragma unroll
    for (int p = 0; p < KP; ++p) {
      float m = xv[p][0];
#pragma unroll
      for (int e = 1; e < 8; ++e) m = fmaxf(m, xv[p][e]);
      for (int o = 1; o < gl; o <<= 1) m = fmaxf(m, __shfl_xor(m, o, SSD_WAVE));
      float sum = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        xv[p][e] = expf(xv[p][e] - m);
        sum += xv[p][e];
      }
      for (int o = 1; o < gl; o <<= 1) sum += __shfl_xor(sum, o, SSD_WAVE);
      const float inv = 1.0f / sum;
#pragma unroll
      for (int e = 0; e < 8; ++e) xv[p][e] *= inv;
    }
  }
  // pieces past K (clamped re-reads) count as zero
#pragma unroll
  for (int p = 0; p < KP; ++p)
    if (p * 512 + lane * 8 >= K) {
#pragma unroll
      for (int e = 0; e < 8; ++e) xv[p][e] = 0.f;
    }
  float rscale = 1.f;
  if (rms) {
    float s2 = 0.f;
#pragma unroll
    for (int p = 0; p < KP; ++p)
#pragma unroll
      for (int e = 0; e < 8; ++e) s2 = fmaf(xv[p][e], xv[p][e], s2);
    s2 = wave_sum(s2);
    rscale = 1.0f / sqrtf(s2 / (float)K + a.eps);
#pragma unroll
    for (int p = 0; p < KP; ++p) {
      float g[8];
      gv[p].to_f32(g);
#pragma unroll
      for (int e = 0; e < 8; ++e) xv[p][e] *= g[e];
    }
  } else if (ln) {
    float s1 = 0.f;
#pragma unroll
    for (int p = 0; p < KP; ++p)
#pragma unroll
      for (int e = 0; e < 8; ++e) s1 += xv[p][e];
    const float mean = wave_sum(s1) / (float)K;
    float s2 = 0.f;
#pragma unroll
    for (int p = 0; p < KP; ++p)
      if (p * 512 + lane * 8 < K) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float c = xv[p][e] - mean;
          s2 = fmaf(c, c, s2);
        }
      }
    const float rstd = 1.0f / sqrtf(wave_sum(s2) / (float)K + a.eps);
#pragma unroll
    for (int p = 0; p < KP; ++p) {
      float g[8], b[8];
      gv[p].to_f32(g);
      sv[p].to_f32(b);
#pragma unroll
      for (int e = 0; e < 8; ++e) xv[p][e] = (xv[p][e] - mean) * rstd * g[e] + b[e];
    }
  }

  float acc[2][1] = {{0.f}, {0.f}};
#pragma unroll
  for (int p = 0; p < KP; ++p) {
    if (p * 512 + lane * 8 < K) {
      float w0[8], w1[8];
      w[0][p].to_f32(w0);
      w[1][p].to_f32(w1);
      float t0 = acc[0][0], t1 = acc[1][0];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        t0 = fmaf(w0[e], xv[p][e], t0);
        t1 = fmaf(w1[e], xv[p][e], t1);
      }
      acc[0][0] = t0;
      acc[1][0] = t1;
    }
  }
  acc[0][0] = wave_sum(acc[0][0]) * rscale;
  acc[1][0] = wave_sum(acc[1][0]) * rscale;
  gemv_finish<WT, 1, KIND>(a, r, acc, yold, live, 0, 1, tid, lane, wave, rv, ri, pre,
                     qkv);
}

// One input row, 2048 <= K <= 2048 * KP (no LayerNorm): the K range is split
// over the block's four waves instead of its rows.  A block owns the four row pairs of gemv1
// (eight weight rows); wave w reads elements p * 2048 + 512 w + 8 lane .. +7 of the input, of the
// gain and of all eight rows, so that each wave requests a quarter of the input and gain bytes
// gemv1 does for the same weight bytes (those extra requests, not the weights, limit gemv1).  The
// eight partial dot products of a lane are reduced over the wave by halving exchanges (three
// swaps leave each group of eight lanes one row), then over the waves through LDS; RMSNorm is
// folded as in gemv1 with the sum of squares reduced the same way.  Wave w finishes row pair w
// with gemv1's epilogue.
template <typename WT, int KP, int NORM, int KIND>
__device__ __forceinline__ void gemv1k_body(const LinearArgs& a, const int blk) {
  static_assert(NORM != NORM_LN, "LayerNorm rows take gemv1_kernel");
  __shared__ float part[GV_WAVES][9];
  __shared__ float rv[GV_WAVES][1];
  __shared__ int ri[GV_WAVES][1];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int K = a.K;
  const bool gated = epi_gated<KIND>(a), qkv = epi_is<KIND>(a, EPI_QKV);
  const int n_total = qkv ? 3 * a.n_per : a.n_per;
  const int n_pairs = gated ? a.n_per : (n_total + 1) / 2;
  constexpr bool rms = NORM == NORM_RMS;

  // inputs first (the wait counter retires loads in issue order); clamped, never conditional
  float xv[KP][8];
#pragma unroll
  for (int p = 0; p < KP; ++p) {
    const int e = min(p * 2048 + wave * 512 + lane * 8, K - 8);
    const float4 x0 = *reinterpret_cast<const float4*>(a.x + e);
    const float4 x1 = *reinterpret_cast<const float4*>(a.x + e + 4);
    xv[p][0] = x0.x; xv[p][1] = x0.y; xv[p][2] = x0.z; xv[p][3] = x0.w;
    xv[p][4] = x1.x; xv[p][5] = x1.y; xv[p][6] = x1.z; xv[p][7] = x1.w;
  }
  const int pr = blk * GV_WAVES + wave;
  const RowPair<WT> r = row_pair<WT, KIND>(a, n_total, pr < n_pairs ? pr : 0);
  const bool live = pr < n_pairs;
  // requested before the weights, as vector loads (the wait counter retires loads in issue order):
  // the sequence length, and the residual values this wave's epilogue adds
  int vzero;
  asm volatile("v_mov_b32 %0, 0" : "=v"(vzero));
  const int qlen = qkv ? a.kv.seq_len[vzero] : 0;
  float yold[2][1] = {{0.f}, {0.f}};
  if (epi_is<KIND>(a, EPI_RESID) || epi_is<KIND>(a, EPI_BIAS_RESID)) {
    const float* src = epi_is<KIND>(a, EPI_RESID) ? a.y : a.resid;
    const float* from = src ? src : a.x;  // no residual: a valid address, not used
    const float y0 = from[(src && r.ok0 ? r.n0 : 0) + vzero], y1 = from[(src && r.ok1 ? r.n1 : 0) + vzero];
    yold[0][0] = src ? y0 : 0.f;
    yold[1][0] = src ? y1 : 0.f;
  }
  Vec8<WT> w[GV_WAVES][2][KP];
#pragma unroll
  for (int q = 0; q < GV_WAVES; ++q) {
    const int pq = blk * GV_WAVES + q;
    const RowPair<WT> rq = row_pair<WT, KIND>(a, n_total, pq < n_pairs ? pq : 0);
#pragma unroll
    for (int p = 0; p < KP; ++p) {
      const int e = min(p * 2048 + wave * 512 + lane * 8, K - 8);
      w[q][0][p].load(rq.w0 + e);
      w[q][1][p].load(rq.w1 + e);
    }
  }
  Vec8<float> gv[rms ? KP : 1];
  if (rms) {
#pragma unroll
    for (int p = 0; p < KP; ++p) gv[p].load(a.gain + min(p * 2048 + wave * 512 + lane * 8, K - 8));
  }
  QkvPre pre = {};
  if (qkv) {
    const int HD = a.n_per, mat = r.n0 >= HD ? (r.n0 >= 2 * HD ? 2 : 1) : 0;
    pre = qkv_pre(a, mat, r.n0 - mat * HD, 0, qlen + a.kv.pos_off);
  }

  // pieces past K (clamped re-reads) count as zero
#pragma unroll
  for (int p = 0; p < KP; ++p)
    if (p * 2048 + wave * 512 + lane * 8 >= K) {
#pragma unroll
      for (int e = 0; e < 8; ++e) xv[p][e] = 0.f;
    }
  float s2 = 0.f;
  if (rms) {
#pragma unroll
    for (int p = 0; p < KP; ++p)
#pragma unroll
      for (int e = 0; e < 8; ++e) s2 = fmaf(xv[p][e], xv[p][e], s2);
    s2 = wave_sum(s2);
#pragma unroll
    for (int p = 0; p < KP; ++p) {
      float g[8];
      gv[p].to_f32(g);
#pragma unroll
      for (int e = 0; e < 8; ++e) xv[p][e] *= g[e];
    }
  }

  // acc[2q + s]: row s of pair q
  float acc[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) acc[i] = 0.f;
#pragma unroll
  for (int q = 0; q < GV_WAVES; ++q)
#pragma unroll
    for (int p = 0; p < KP; ++p) {
      float w0[8], w1[8];
      w[q][0][p].to_f32(w0);
      w[q][1][p].to_f32(w1);
      float t0 = acc[2 * q], t1 = acc[2 * q + 1];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        t0 = fmaf(w0[e], xv[p][e], t0);
        t1 = fmaf(w1[e], xv[p][e], t1);
      }
      acc[2 * q] = t0;
      acc[2 * q + 1] = t1;
    }
  // halving exchanges: after the swaps over lane bits 5, 4, 3 lane l holds a partial of row
  // (l >> 3) & 7, summed over its group of eight lanes by the last three steps
  const bool b5 = lane & 32, b4 = lane & 16, b3 = lane & 8;
  float u[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float mine = b5 ? acc[i + 4] : acc[i], other = b5 ? acc[i] : acc[i + 4];
    u[i] = mine + __shfl_xor(other, 32, SSD_WAVE);
  }
  float t[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const float mine = b4 ? u[i + 2] : u[i], other = b4 ? u[i] : u[i + 2];
    t[i] = mine + __shfl_xor(other, 16, SSD_WAVE);
  }
  float sres = (b3 ? t[1] : t[0]) + __shfl_xor(b3 ? t[0] : t[1], 8, SSD_WAVE);
  sres += __shfl_xor(sres, 4, SSD_WAVE);
  sres += __shfl_xor(sres, 2, SSD_WAVE);
  sres += __shfl_xor(sres, 1, SSD_WAVE);
  if ((lane & 7) == 0) part[wave][lane >> 3] = sres;
  if (rms && lane == 0) part[wave][8] = s2;
  __syncthreads();
  float rscale = 1.f;
  if (rms) {
    const float tot = (part[0][8] + part[1][8]) + (part[2][8] + part[3][8]);
    rscale = 1.0f / sqrtf(tot / (float)K + a.eps);
  }
  float res[2][1];
  res[0][0] = ((part[0][2 * wave] + part[1][2 * wave]) + (part[2][2 * wave] + part[3][2 * wave])) * rscale;
  res[1][0] = ((part[0][2 * wave + 1] + part[1][2 * wave + 1]) + (part[2][2 * wave + 1] + part[3][2 * wave + 1])) * rscale;
  gemv_finish<WT, 1, KIND>(a, r, res, yold, live, 0, 1, tid, lane, wave, rv, ri, pre,
                     qkv);
}

template <typename WT, int KP, int NORM, int KIND>
__global__ __launch_bounds__(256) void gemv1k_kernel(const LinearArgs a) {
  gemv1k_body<WT, KP, NORM, KIND>(a, blockIdx.x);
}

// Two one-row GEMVs over the same inputs in one launch: blocks [0, na) run `a` (bf16 weights,
// K <= 2048 * KPA, bias / residual epilogue), the others `b` (float32 weights, K <= 2048 * KPB,
// stored); no input transform.
template <int KPA, int KPB>
__global__ __launch_bounds__(256) void gemv1k_pair_kernel(const LinearArgs a, const LinearArgs b,
                                                          const int na) {
  const int blk = blockIdx.x;
  if (blk < na) gemv1k_body<bf16_t, KPA, NORM_NONE, EPI_BIAS_RESID>(a, blk);
  else gemv1k_body<float, KPB, NORM_NONE, EPI_STORE>(b, blk - na);
}

template <typename WT, int KP, int NORM, int KIND>
void launch_gemv1_t(const LinearArgs& a, dim3 grid, hipStream_t s, LaunchTiming* t) {
  if (t) {
    hipExtLaunchKernelGGL((gemv1_kernel<WT, KP, NORM, KIND>), grid, dim3(256), 0u, s, t->start, t->stop, 0u, a);
    t->timed = true;
  } else {
    hipLaunchKernelGGL((gemv1_kernel<WT, KP, NORM, KIND>), grid, dim3(256), 0, s, a);
  }
}

template <typename WT, int KP, int NORM, int KIND>
void launch_gemv1k_t(const LinearArgs& a, dim3 grid, hipStream_t s, LaunchTiming* t) {
  if (t) {
    hipExtLaunchKernelGGL((gemv1k_kernel<WT, KP, NORM, KIND>), grid, dim3(256), 0u, s, t->start, t->stop, 0u, a);
    t->timed = true;
  } else {
    hipLaunchKernelGGL((gemv1k_kernel<WT, KP, NORM, KIND>), grid, dim3(256), 0, s, a);
  }
}

// The epilogue instances each input transform meets in a decoder; any other takes the run-time one.
#define SSD_KINDS(LAUNCH, NORM)                                                       \
  do {                                                                                \
    if constexpr (NORM == NORM_RMS) {                                                 \
      switch (a.epi) {                                                                \
        case EPI_QKV: LAUNCH(NORM, EPI_QKV); return;                                  \
        case EPI_GATED_GELU: LAUNCH(NORM, EPI_GATED_GELU); return;                    \
        case EPI_GATED_SILU: LAUNCH(NORM, EPI_GATED_SILU); return;                    \
        case EPI_ARGMAX: LAUNCH(NORM, EPI_ARGMAX); return;                            \
        case EPI_STORE: LAUNCH(NORM, EPI_STORE); return;                              \
        default: LAUNCH(NORM, GV_ANY); return;                                        \
      }                                                                               \
    } else if constexpr (NORM == NORM_LN) {                                           \
      if (a.epi == EPI_BIAS_GELU) { LAUNCH(NORM, EPI_BIAS_GELU); return; }            \
      LAUNCH(NORM, GV_ANY);                                                           \
    } else {                                                                          \
      switch (a.epi) {                                                                \
        case EPI_RESID: LAUNCH(NORM, EPI_RESID); return;                              \
        case EPI_BIAS_RESID: LAUNCH(NORM, EPI_BIAS_RESID); return;                    \
        default: LAUNCH(NORM, GV_ANY); return;                                        \
      }                                                                               \
    }                                                                                 \
  } while (0)

template <typename WT, int KP, int NORM>
void launch_gemv1(const LinearArgs& a, dim3 grid, hipStream_t s, LaunchTiming* t) {
#define SSD_L(N, E) launch_gemv1_t<WT, KP, N, E>(a, grid, s, t)
  SSD_KINDS(SSD_L, NORM);
#undef SSD_L
}

template <int KP, int NORM, typename WT = bf16_t>
void launch_gemv1k(const LinearArgs& a, dim3 grid, hipStream_t s, LaunchTiming* t) {
#define SSD_L(N, E) launch_gemv1k_t<WT, KP, N, E>(a, grid, s, t)
  SSD_KINDS(SSD_L, NORM);
#undef SSD_L
}

// Blocks of a one-row launch: four row pairs each.
int row_blocks(const LinearArgs& a) {
  const bool gated = (a.epi == EPI_GATED_GELU || a.epi == EPI_GATED_SILU);
  const int n_pairs = gated ? a.n_per : (a.n_per * a.n_mats + 1) / 2;
  return (n_pairs + GV_WAVES - 1) / GV_WAVES;
}

// One bf16 row with 2048 <= K <= 6144 and no LayerNorm, or up to 12288 without a norm (the
// LLaMA-7B down projection, K = 11008): the K-split kernel (same grid as gemv1).  float32
// weights at K = 2048 too (the folded cross-attention scores of a FlanT5-xl-sized layer).
bool use_gemv1k(const LinearArgs& a) {
  if (a.M != 1 || a.K < 2048 || a.K % 8) return false;
  if (a.wdtype != 1) return a.K == 2048 && (a.norm == NORM_RMS || a.norm == NORM_NONE);
  if (a.norm == NORM_RMS) return a.K <= 3 * 2048;
  return a.norm == NORM_NONE && a.K <= 6 * 2048;
}

hipError_t launch_gemv1k_any(const LinearArgs& a, hipStream_t s, LaunchTiming* t) {
  const dim3 grid(row_blocks(a));
  const bool timed = t && a.K == t->K && a.norm == t->norm && a.wdtype == t->wdtype && t->start &&
                     t->stop;
  LaunchTiming* tt = timed ? t : nullptr;
  const int kp = (a.K + 2047) / 2048;
  const bool rms = a.norm == NORM_RMS;
  if (a.wdtype != 1) {
    rms ? launch_gemv1k<1, NORM_RMS, float>(a, grid, s, tt)
        : launch_gemv1k<1, NORM_NONE, float>(a, grid, s, tt);
  } else if (kp == 1) rms ? launch_gemv1k<1, NORM_RMS>(a, grid, s, tt) : launch_gemv1k<1, NORM_NONE>(a, grid, s, tt);
  else if (kp == 2) rms ? launch_gemv1k<2, NORM_RMS>(a, grid, s, tt) : launch_gemv1k<2, NORM_NONE>(a, grid, s, tt);
  else if (kp == 3) rms ? launch_gemv1k<3, NORM_RMS>(a, grid, s, tt) : launch_gemv1k<3, NORM_NONE>(a, grid, s, tt);
  else if (kp == 4) launch_gemv1k<4, NORM_NONE>(a, grid, s, tt);
  else if (kp == 5) launch_gemv1k<5, NORM_NONE>(a, grid, s, tt);
  else launch_gemv1k<6, NORM_NONE>(a, grid, s, tt);
  return hipGetLastError();
}


template <typename WT, int KP>
void launch_gemv1_norm(const LinearArgs& a, hipStream_t s, LaunchTiming* t) {
  const dim3 grid(row_blocks(a));
  if (a.norm == NORM_RMS) launch_gemv1<WT, KP, NORM_RMS>(a, grid, s, t);
  else if (a.norm == NORM_LN) launch_gemv1<WT, 4, NORM_LN>(a, grid, s, t);
  else if (a.norm == NORM_SOFTMAX) launch_gemv1<WT, KP, NORM_SOFTMAX>(a, grid, s, nullptr);
  else launch_gemv1<WT, KP, NORM_NONE>(a, grid, s, t);
}

template <typename WT>
void launch_gemv1_any(const LinearArgs& a, hipStream_t s, LaunchTiming* t) {
  switch (gemv_pieces(a.K)) {
    case 2: return launch_gemv1_norm<WT, 2>(a, s, t);
    case 4: return launch_gemv1_norm<WT, 4>(a, s, t);
    case 12: return launch_gemv1_norm<WT, 12>(a, s, t);
    default: return launch_gemv1_norm<WT, 8>(a, s, t);
  }
}

}  // namespace

hipError_t launch_one_row(const LinearArgs& a, hipStream_t s, LaunchTiming* t, bool* taken) {
  *taken = false;
  if (a.M != 1 || (a.n_mats != 1 && a.epi != EPI_QKV && a.epi != EPI_GATED_GELU && a.epi != EPI_GATED_SILU))
    return hipSuccess;
  if (use_gemv1k(a)) {
    *taken = true;
    return launch_gemv1k_any(a, s, t);
  }
  if (a.norm == NORM_LN ? a.K > 2048 : a.K > 512 * gemv_pieces(a.K)) return hipSuccess;
  *taken = true;
  const bool timed = t && a.K == t->K && a.norm == t->norm && a.wdtype == t->wdtype && t->start && t->stop;
  if (a.wdtype == 1) launch_gemv1_any<bf16_t>(a, s, timed ? t : nullptr);
  else launch_gemv1_any<float>(a, s, timed ? t : nullptr);
  return hipGetLastError();
}

bool linear_pair_ok(const LinearArgs& a, const LinearArgs& b) {
  auto plain = [](const LinearArgs& x) {
    return x.M == 1 && x.norm == NORM_NONE && x.K >= 8 && x.K % 8 == 0 &&
           x.n_mats == 1 && x.n_per > 0;
  };
  return plain(a) && plain(b) && a.epi == EPI_BIAS_RESID && b.epi == EPI_STORE && a.wdtype == 1 && a.K <= 2048 && b.wdtype == 0 && b.K <= 4096;
}

hipError_t launch_linear_pair(const LinearArgs& a, const LinearArgs& b, hipStream_t s) {
  if (!linear_pair_ok(a, b)) return hipErrorInvalidValue;
  const int na = row_blocks(a), nb = row_blocks(b);
  hipLaunchKernelGGL((gemv1k_pair_kernel<1, 2>), dim3(na + nb), dim3(256), 0, s, a, b, na);
  return hipGetLastError();
}

}  // namespace ssd
