// Linear layers y = epilogue(W . norm(x)) for the decoder, the imitation network and the LM head.
//
// Paths:
//  * gemv_kernel — weight streaming in blocks of up to 8 float32 rows: float32 weights, the
//    imitation network's rows that dense_rows_kernel does not take, single rows past the limits of
//    gemv1.hip.  The input rows are staged in LDS with the gain applied, one row pair per wave.
//  * dense_rows_kernel — the imitation network on 2..8 rows (bf16 weights, rows up to 4096) on the
//    float32 matrix instruction.
//  * fold_rows_kernel — 2..8 rows of the folded cross-attention (float32 matrices) on matrix
//    products of bf16 hi / lo splits.
// One row takes the kernels of gemv1.hip, the decoder's layers on two rows and more with bf16
// weights those of gemm.hip.
//
// Every path accumulates in fp32 and ends in a fused epilogue (store, residual (+ stash), gated
// activation, bias + GELU, bias + residual, per-block (max, argmax) partials for the LM head, or
// QKV with rotary and the paged KV store).
#include "device.h"
#include "gemv_common.h"
#include "kernels.h"

#include <climits>

namespace ssd {

namespace {

// Weight-streaming GEMV for MB <= 8 input rows held in LDS (MB * K <= GV_LDS_FLOATS).
// One row pair per wave (blockIdx.x * 4 + wave); a wave requests a whole batch (GV_KP * 512
// elements of both rows; the whole row for K <= 6144) at once and the many resident waves of a CU
// hide the memory latency.
// RMSNorm is folded: LDS holds gain * x and the per-row 1/rms multiplies the dot products in the
// epilogue; LayerNorm inputs are staged as they are and normalised in place.
// (The wave index goes through readfirstlane in these kernels so that the compiler treats the
// wave's row choice as uniform: the matrix pointers then come from scalar registers instead of
// vector loads of the argument buffer that would wait for the inputs.)
template <typename WT, int MB, int GV_KP>
__global__ __launch_bounds__(256) void gemv_kernel(const LinearArgs a) {
  extern __shared__ float xs[];  // [MB][ldxs]
  __shared__ float red[GV_WAVES][2 * MB];
  __shared__ float rv[GV_WAVES][MB];
  __shared__ int ri[GV_WAVES][MB];

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int K = a.K;
  const int ldxs = (K + 7) & ~7;
  const int m0 = blockIdx.y * MB;
  const int mrows = min(MB, a.M - m0);
  const bool gated = (a.epi == EPI_GATED_GELU || a.epi == EPI_GATED_SILU);
  const int n_total = gated ? a.n_per : a.n_per * a.n_mats;
  const int n_pairs = gated ? a.n_per : (n_total + 1) / 2;
  const int pr = blockIdx.x * GV_WAVES + wave;
  const bool rms = a.norm == NORM_RMS, ln = a.norm == NORM_LN;

  // inputs first: the wait counter is in order, so they must be requested before the weights
  float p2[MB];
#pragma unroll
  for (int m = 0; m < MB; ++m) p2[m] = 0.f;
  if (ln) {
    // LayerNorm: the rows as they are and their means, the variances about the means (mean square
    // less squared mean would cancel where the mean is large against the spread), then the normalised
    // rows; a thread meets its own elements again
    auto row_sums = [&]() {
#pragma unroll
      for (int m = 0; m < MB; ++m) p2[m] = wave_sum(p2[m]);
      if (lane == 0) {
#pragma unroll
        for (int m = 0; m < MB; ++m) red[wave][m] = p2[m];
      }
      __syncthreads();
    };
    auto total = [&](int m) { return (red[0][m] + red[1][m]) + (red[2][m] + red[3][m]); };
    for (int idx = tid * 4; idx < MB * ldxs; idx += 1024) {
      const int m = idx / ldxs, k = idx - m * ldxs;
      float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
      if (m < mrows && k < K) v = *reinterpret_cast<const float4*>(a.x + (size_t)(m0 + m) * a.ldx + k);
#pragma unroll
      for (int mm = 0; mm < MB; ++mm)
        if (mm == m) p2[mm] += (v.x + v.y) + (v.z + v.w);
      *reinterpret_cast<float4*>(xs + m * ldxs + xs_off(k, ldxs)) = v;
    }
    row_sums();
    float mean[MB];
#pragma unroll
    for (int m = 0; m < MB; ++m) {
      mean[m] = total(m) / (float)K;
      p2[m] = 0.f;
    }
    __syncthreads();  // the means are read before the next sums take their place
    for (int idx = tid * 4; idx < MB * ldxs; idx += 1024) {
      const int m = idx / ldxs, k = idx - m * ldxs;
      if (k >= K) continue;
      float4 v = *reinterpret_cast<const float4*>(xs + m * ldxs + xs_off(k, ldxs));
#pragma unroll
      for (int mm = 0; mm < MB; ++mm)
        if (mm == m) {
          v.x -= mean[mm]; v.y -= mean[mm]; v.z -= mean[mm]; v.w -= mean[mm];
          p2[mm] += (v.x * v.x + v.y * v.y) + (v.z * v.z + v.w * v.w);
        }
      *reinterpret_cast<float4*>(xs + m * ldxs + xs_off(k, ldxs)) = v;
    }
    row_sums();
    for (int idx = tid * 4; idx < MB * ldxs; idx += 1024) {
      const int m = idx / ldxs, k = idx - m * ldxs;
      if (k >= K) continue;
      const float rstd = 1.0f / sqrtf(total(m) / (float)K + a.eps);
      float4 v = *reinterpret_cast<const float4*>(xs + m * ldxs + xs_off(k, ldxs));
      const float4 g = *reinterpret_cast<const float4*>(a.gain + k);
      const float4 b = *reinterpret_cast<const float4*>(a.shift + k);
      v.x = v.x * rstd * g.x + b.x;
      v.y = v.y * rstd * g.y + b.y;
      v.z = v.z * rstd * g.z + b.z;
      v.w = v.w * rstd * g.w + b.w;
      *reinterpret_cast<float4*>(xs + m * ldxs + xs_off(k, ldxs)) = v;
    }
  } else {
    // 8 float4 per thread requested together (a loop with one load per trip would pay one
    // memory round trip per trip)
    constexpr int SB = 8;
    for (int base = tid * 4; base < MB * ldxs; base += 1024 * SB) {
      float4 v[SB], g[SB];
#pragma unroll
      for (int u = 0; u < SB; ++u) {
        const int idx = base + u * 1024;
        const int m = idx / ldxs, k = idx - m * ldxs;
        v[u] = g[u] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (idx < MB * ldxs && m < mrows && k < K) {
          v[u] = *reinterpret_cast<const float4*>(a.x + (size_t)(m0 + m) * a.ldx + k);
          if (rms) g[u] = *reinterpret_cast<const float4*>(a.gain + k);
        }
      }
#pragma unroll
      for (int u = 0; u < SB; ++u) {
        const int idx = base + u * 1024;
        if (idx >= MB * ldxs) break;
        const int m = idx / ldxs, k = idx - m * ldxs;
        float4 x4 = v[u];
        if (rms) {
#pragma unroll
          for (int mm = 0; mm < MB; ++mm)
            if (mm == m) p2[mm] += (x4.x * x4.x + x4.y * x4.y) + (x4.z * x4.z + x4.w * x4.w);
          x4.x *= g[u].x; x4.y *= g[u].y; x4.z *= g[u].z; x4.w *= g[u].w;
        }
        *reinterpret_cast<float4*>(xs + m * ldxs + xs_off(k, ldxs)) = x4;
      }
    }
    if (rms) {
#pragma unroll
      for (int m = 0; m < MB; ++m) p2[m] = wave_sum(p2[m]);
      if (lane == 0) {
#pragma unroll
        for (int m = 0; m < MB; ++m) red[wave][2 * m + 1] = p2[m];
      }
    }
  }

  // the residual values this wave's epilogue adds (lane 0), then the first weights
  const RowPair<WT> r = row_pair<WT, GV_ANY>(a, n_total, pr < n_pairs ? pr : 0);
  const bool live = pr < n_pairs;
  float yold[2][MB];
  if (lane == 0 && live && (a.epi == EPI_RESID || a.epi == EPI_BIAS_RESID)) {
    const float* src = a.epi == EPI_RESID ? a.y : a.resid;
    const int ld = a.epi == EPI_RESID ? a.ldy : a.ldr;
#pragma unroll
    for (int m = 0; m < MB; ++m) {
      yold[0][m] = (src && r.ok0 && m < mrows) ? src[(size_t)(m0 + m) * ld + r.n0] : 0.f;
      yold[1][m] = (src && r.ok1 && m < mrows) ? src[(size_t)(m0 + m) * ld + r.n1] : 0.f;
    }
  }
  Vec8<WT> w[2][GV_KP];
  load_pieces<WT, GV_KP>(w, r, 0, K, lane);
  __syncthreads();

  float rscale[MB];  // per input row: 1/rms (RMSNorm folded into the epilogue) or 1
#pragma unroll
  for (int m = 0; m < MB; ++m) {
    rscale[m] = 1.f;
    if (rms) {
      const float s2 = (red[0][2 * m + 1] + red[1][2 * m + 1]) + (red[2][2 * m + 1] + red[3][2 * m + 1]);
      rscale[m] = 1.0f / sqrtf(s2 / (float)K + a.eps);
    }
  }

  float acc[2][MB];
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int m = 0; m < MB; ++m) acc[s][m] = 0.f;
  for (int e0 = 0; e0 < K; e0 += 512 * GV_KP) {
    if (e0 > 0) load_pieces<WT, GV_KP>(w, r, e0, K, lane);
    fma_pieces<WT, MB, GV_KP>(w, xs, ldxs, e0, K, lane, acc);
  }
#pragma unroll
  for (int m = 0; m < MB; ++m) {
    acc[0][m] = wave_sum(acc[0][m]) * rscale[m];
    acc[1][m] = wave_sum(acc[1][m]) * rscale[m];
  }
  gemv_finish<WT, MB, GV_ANY>(a, r, acc, yold, live, m0, mrows, tid, lane, wave, rv, ri);
}

constexpr int SKW = 8;  // waves of a block of the folded cross-attention kernel
constexpr int SSQ_MAX = 256;  // partial sums of squares it reads

// The folded cross-attention of a verify chunk (at most 8 rows, float32 weights) on half tiles.  A
// half tile is 8 features: the A operand holds them twice, A row i being feature i & 7 over elements
// 0..31 (i < 8) or 32..63 (i >= 8) of a 64-element step, and the B operand's columns are the 8 input
// rows over the same two halves; D[f][t] + D[f + 8][t + 8] is the step's dot product (the other two
// quadrants are cross terms and are dropped).  A step's weights are read as 256 contiguous bytes of a
// row, eight lanes each, split into bf16 hi / lo and passed through the wave's own LDS to the operand
// order (a row per lane is 64 accesses of the vector memory path a load instead of 16).  With eight
// waves to split K instead of four: 6.2 -> 6.0 us for the scores and 7.2 -> 6.5 for the output of 6 rows
// at the FlanT5-xl shape, 4.4 -> 3.6 and 4.8 -> 4.2 at FlanT5-base; what is left is the launch, one round
// trip of loads and the reduction.  A step takes the products hi.hi, hi.lo and lo.hi (about 16 mantissa
// bits on both sides).  The epilogue runs on 64 threads (feature tid / 8, row tid % 8).
// RMS: the scores, fold_q . rms(x) from input planes, stored.  Else the output, y += fold_o .
// softmax(scores): the input is float32 rows (in_f32) turned into softmax probabilities over groups of
// a.group consecutive inputs (8, 16 or 32: the group of a lane's 8 elements spans the 1, 2 or 4 lanes
// l, l ^ 16, l ^ 32, l ^ 48 of one row and step half), split into hi / lo as the B operand; it leaves
// the next planes and one partial sum of squares per half tile.
template <bool RMS, int SK>
__global__ __launch_bounds__(64 * SKW) void fold_rows_kernel(const LinearArgs a) {
  constexpr bool SMX = !RMS;
  constexpr int NG = 4 * SKW;  // groups of 16 threads
  __shared__ float part[SKW][8][9];
  __shared__ float rs[16];
  __shared__ float ssq_red[4 * SKW][16];
  __shared__ __attribute__((aligned(16))) unsigned char staged[SKW][2][1024];  // hi, lo: [8 rows][64]

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int K = a.K, M = a.M, n_out = a.n_per, h = blockIdx.x;
  const int steps = K / 64;
  const int s_beg = (steps * wave) / SKW, s_end = (steps * (wave + 1)) / SKW;
  // this lane's weights of a step: row lane / 8, elements 4 (lane % 8) .. and 32 + 4 (lane % 8) ..
  const float* wrow = reinterpret_cast<const float*>(a.w[0]) + (size_t)min(h * 8 + (lane >> 3), n_out - 1) * K + (lane & 7) * 4;
  // staging: 16-byte chunk k of row r at position k ^ r
  unsigned char* st_w = staged[wave][0] + (lane >> 3) * 128 + (lane & 1) * 8;
  const int wp0 = (((lane & 7) >> 1) ^ (lane >> 3)) << 4, wp1 = ((4 + ((lane & 7) >> 1)) ^ (lane >> 3)) << 4;
  const unsigned char* st_r = staged[wave][0] + (lane & 7) * 128 + (((4 * ((lane >> 3) & 1) + (lane >> 4)) ^ (lane & 7)) << 4);
  const int kq = ((lane >> 3) & 1) * 32 + (lane >> 4) * 8;  // this lane's 8 elements of a step
  const int tok = lane & 7;
  const bool tok_ok = tok < M;
  // input fragments: rows of the K block this lane's elements lie in; or this lane's float32 row
  const bf16_t* brow = a.in_planes + ((lane >> 3) & 1) * PLANE_FRAG + ((lane >> 4) * 16 + tok) * 8;
  const float* frow = SMX ? a.in_f32 + (size_t)(tok_ok ? tok : 0) * a.in_ld : nullptr;
  const int gsh = SMX ? (a.group >= 32 ? 2 : (a.group >= 16 ? 1 : 0)) : 0;  // exchanges per group
  const int ef = (tid >> 3) & 7, et = tid & 7, en = h * 8 + ef;  // epilogue thread: feature, row

  // values the epilogue needs, requested before the main batch (the wait counter retires loads in
  // issue order): the producer's partial sums of squares (thread: row tid % 16, partials
  // tid / 16 + NG j) and the old residual value of this thread's output
  float sv[RMS ? SSQ_MAX / NG : 1];
  if (RMS) {
#pragma unroll
    for (int j = 0; j < SSQ_MAX / NG; ++j)
      sv[j] = a.in_ssq[(size_t)min((tid >> 4) + NG * j, a.in_nssq - 1) * 16 + (tid & 15)];
  }
  float y_old = 0.f;
  if (SMX) y_old = a.y[(size_t)min(et, M - 1) * a.ldy + min(en, n_out - 1)];

  f32x4_t acc = f32x4_t{0.f, 0.f, 0.f, 0.f};
  for (int s0 = s_beg; s0 < s_end; s0 += SK) {
    uint4 bv[SK][2];   // the hi and lo planes' 16 bytes, or 32 bytes of the float32 row
    f32x4_t wf[SK][2];
    // inputs first (L2-resident, they arrive early), then the weights in step order
#pragma unroll
    for (int u = 0; u < SK; ++u) {
      const int st = max(min(s0 + u, s_end - 1), 0);
      if (SMX) {
        const float4 f0 = *reinterpret_cast<const float4*>(frow + st * 64 + kq);
        const float4 f1 = *reinterpret_cast<const float4*>(frow + st * 64 + kq + 4);
        bv[u][0] = make_uint4(__float_as_uint(f0.x), __float_as_uint(f0.y), __float_as_uint(f0.z), __float_as_uint(f0.w));
        bv[u][1] = make_uint4(__float_as_uint(f1.x), __float_as_uint(f1.y), __float_as_uint(f1.z), __float_as_uint(f1.w));
      } else {
        const bf16_t* bp = brow + (size_t)st * (2 * PLANE_FRAG);
        bv[u][0] = *reinterpret_cast<const uint4*>(bp);
        bv[u][1] = *reinterpret_cast<const uint4*>(bp + PLANE_LO);
      }
    }
#pragma unroll
    for (int u = 0; u < SK; ++u) {
      const int k0 = max(min(s0 + u, s_end - 1), 0) * 64;
      wf[u][0] = *reinterpret_cast<const f32x4_t*>(wrow + k0);
      wf[u][1] = *reinterpret_cast<const f32x4_t*>(wrow + k0 + 32);
    }
    __builtin_amdgcn_sched_barrier(0);  // keep the whole batch in flight before the first MFMA
#pragma unroll
    for (int u = 0; u < SK; ++u) {
      // a step past this wave's range, or a row past M, re-read valid data: zero operands
      const bool use = tok_ok && (s0 + u < s_end);
      const uint4 z = make_uint4(0, 0, 0, 0);
      uint4 b0 = bv[u][0], b1 = bv[u][1];
      if constexpr (SMX) {
        // softmax over the lane's group: max and sum over its 8 elements and the group's other
        // lanes (every lane takes part in the exchanges), then hi / lo of the probabilities
        float f[8] = {__uint_as_float(b0.x), __uint_as_float(b0.y), __uint_as_float(b0.z), __uint_as_float(b0.w),
                      __uint_as_float(b1.x), __uint_as_float(b1.y), __uint_as_float(b1.z), __uint_as_float(b1.w)};
        float m = f[0];
#pragma unroll
        for (int e = 1; e < 8; ++e) m = fmaxf(m, f[e]);
        const float m16 = fmaxf(m, __shfl_xor(m, 16, SSD_WAVE));
        const float m32 = fmaxf(m16, __shfl_xor(m16, 32, SSD_WAVE));
        m = gsh == 0 ? m : (gsh == 1 ? m16 : m32);
        float sum = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          f[e] = expf(f[e] - m);
          sum += f[e];
        }
        const float s16 = sum + __shfl_xor(sum, 16, SSD_WAVE);
        const float s32 = s16 + __shfl_xor(s16, 32, SSD_WAVE);
        sum = gsh == 0 ? sum : (gsh == 1 ? s16 : s32);
        const float inv = 1.0f / sum;
        split_bf16x8_v(make_float4(f[0] * inv, f[1] * inv, f[2] * inv, f[3] * inv),
                       make_float4(f[4] * inv, f[5] * inv, f[6] * inv, f[7] * inv), b0, b1);
      }
      // operands as values (no address taken, so that nothing of the batch lives in memory)
      const bf16x8_t B0 = __builtin_bit_cast(bf16x8_t, use ? b0 : z);
      const bf16x8_t B1 = __builtin_bit_cast(bf16x8_t, use ? b1 : z);
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const f32x4_t f = wf[u][q];
        const uint32_t h0 = pack_bf16x2(f[0], f[1]), h1 = pack_bf16x2(f[2], f[3]);
        unsigned char* p = st_w + (q ? wp1 : wp0);
        *reinterpret_cast<uint2*>(p) = make_uint2(h0, h1);
        *reinterpret_cast<uint2*>(p + 1024) =
            make_uint2(pack_bf16x2(f[0] - __uint_as_float(h0 << 16), f[1] - __uint_as_float(h0 & 0xffff0000u)),
                       pack_bf16x2(f[2] - __uint_as_float(h1 << 16), f[3] - __uint_as_float(h1 & 0xffff0000u)));
      }
      const bf16x8_t Ah = *reinterpret_cast<const bf16x8_t*>(st_r), Al = *reinterpret_cast<const bf16x8_t*>(st_r + 1024);
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Ah, B0, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Ah, B1, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Al, B0, acc, 0, 0, 0);
    }
  }
  // lane holds D rows 4 (lane / 16) + e, column lane % 16: the useful quadrants are rows 0..7 x
  // columns 0..7 (lanes 0..7 and 16..23) and rows 8..15 x columns 8..15 (those lanes + 40)
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float v = acc[e] + __shfl_down(acc[e], 40, SSD_WAVE);
    if (lane < 24 && !(lane & 8)) part[wave][4 * (lane >> 4) + e][lane & 7] = v;
  }
  if (RMS) {
    float sp = 0.f;
#pragma unroll
    for (int j = 0; j < SSQ_MAX / NG; ++j) sp += ((tid >> 4) + NG * j < a.in_nssq) ? sv[j] : 0.f;
    ssq_red[tid >> 4][tid & 15] = sp;
  }
  __syncthreads();
  if (RMS && tid < 16) {
    float s2 = 0.f;
#pragma unroll
    for (int g = 0; g < NG; ++g) s2 += ssq_red[g][tid];
    rs[tid] = 1.0f / sqrtf(s2 / (float)K + a.eps);
  }
  __syncthreads();

  if (tid >= 64) return;  // whole waves
  float v = 0.f;
#pragma unroll
  for (int w = 0; w < SKW; ++w) v += part[w][ef][et];
  const bool ok = et < M && en < n_out;
  if (RMS) {
    if (ok) a.y[(size_t)et * a.ldy + en] = v * rs[et];
    return;
  }
  float y2 = 0.f;
  if (ok) {
    const float t = y_old + v;
    a.y[(size_t)et * a.ldy + en] = t;
    if (a.out_planes) store_planes1(a.out_planes + plane_at(et, en, 1), a.out_gain ? a.out_gain[en] * t : t);
    y2 = t * t;
  }
  if (a.out_ssq) {
    // the half tile's 8 features of row et: lanes et + 8 f of this wave
    y2 += __shfl_xor(y2, 8, SSD_WAVE);
    y2 += __shfl_xor(y2, 16, SSD_WAVE);
    y2 += __shfl_xor(y2, 32, SSD_WAVE);
    if (lane < 8) a.out_ssq[(size_t)h * 16 + et] = y2;
  }
}

// The imitation network's two layers on 2..8 rows: bf16 weights against float32 rows (LN: normalised
// first) on the float32 matrix instruction, so that inputs and accumulation stay float32.  Half tiles
// of 8 features as in fold_rows_kernel: A rows 0..7 and 8..15 are the features over the two halves of a
// 64-element step, the B columns the rows over the same halves, so a row's eight lanes read its whole
// 128 bytes.  Matrix element e of a lane's group of 8 takes the group's elements in any order as long
// as A and B agree, so both are read as contiguous 16-byte loads and no operand is rearranged.  Eight
// waves split K, all loads of a block in flight at once; the rows' LayerNorm statistics come from the
// same registers.  Bound by launch and one round trip.  The vector kernel stages the rows in LDS in
// every block and multiplies each weight row by row: 26.6 -> 7.8 us (LN) and 13.5 -> 5.4 us for 8
// rows of 2048 x 2048.
template <bool LN, int SK>
__global__ __launch_bounds__(64 * SKW) void dense_rows_kernel(const LinearArgs a) {
  __shared__ float part[SKW][8][9];
  __shared__ float st[SKW][2][8];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int K = a.K, M = a.M, n_out = a.n_per, h = blockIdx.x;
  const int steps = K / 64;
  const int s_beg = (steps * wave) / SKW, s_end = (steps * (wave + 1)) / SKW;  // at most SK steps
  const int kq = ((lane >> 3) & 1) * 32 + (lane >> 4) * 8;  // this lane's 8 elements of a step
  const float* xrow = a.x + (size_t)min(lane & 7, M - 1) * a.ldx + kq;
  const bf16_t* wrow = reinterpret_cast<const bf16_t*>(a.w[0]) + (size_t)min(h * 8 + (lane & 7), n_out - 1) * K + kq;
  const int ef = (tid & 63) >> 3, et = tid & 7, en = h * 8 + ef, ec = min(en, n_out - 1), em = min(et, M - 1);

  f32x4_t xv[SK][2], gv[LN ? SK : 1][2], bv[LN ? SK : 1][2];
  uint4 wv[SK];
#pragma unroll
  for (int u = 0; u < SK; ++u) {
    const float* p = xrow + max(min(s_beg + u, s_end - 1), 0) * 64;
    xv[u][0] = *reinterpret_cast<const f32x4_t*>(p);
    xv[u][1] = *reinterpret_cast<const f32x4_t*>(p + 4);
  }
#pragma unroll
  for (int u = 0; u < SK; ++u)
    wv[u] = *reinterpret_cast<const uint4*>(wrow + max(min(s_beg + u, s_end - 1), 0) * 64);
  if constexpr (LN) {
#pragma unroll
    for (int u = 0; u < SK; ++u) {
      const int k0 = max(min(s_beg + u, s_end - 1), 0) * 64 + kq;
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        gv[u][q] = *reinterpret_cast<const f32x4_t*>(a.gain + k0 + 4 * q);
        bv[u][q] = *reinterpret_cast<const f32x4_t*>(a.shift + k0 + 4 * q);
      }
    }
  }
  const float bias = a.bias ? a.bias[ec] : 0.f;
  const float y_old = !LN && a.resid ? a.resid[(size_t)em * a.ldr + ec] : 0.f;
  __builtin_amdgcn_sched_barrier(0);

  if constexpr (LN) {
    // mean, then the variance about it (mean square less squared mean would cancel where the mean is
    // large against the spread)
    float p1 = 0.f, p2 = 0.f;
#pragma unroll
    for (int u = 0; u < SK; ++u) {
      if (s_beg + u >= s_end) break;  // the same for the whole wave
#pragma unroll
      for (int e = 0; e < 8; ++e) p1 += xv[u][e >> 2][e & 3];
    }
#pragma unroll
    for (int o = 8; o < SSD_WAVE; o <<= 1) p1 += __shfl_xor(p1, o, SSD_WAVE);
    if (lane < 8) st[wave][0][lane] = p1;
    __syncthreads();
    p1 = 0.f;
#pragma unroll
    for (int w = 0; w < SKW; ++w) p1 += st[w][0][lane & 7];
    const float mean = p1 / (float)K;
#pragma unroll
    for (int u = 0; u < SK; ++u) {
      if (s_beg + u >= s_end) break;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float v = xv[u][e >> 2][e & 3] - mean;
        p2 = fmaf(v, v, p2);
      }
    }
#pragma unroll
    for (int o = 8; o < SSD_WAVE; o <<= 1) p2 += __shfl_xor(p2, o, SSD_WAVE);
    if (lane < 8) st[wave][1][lane] = p2;
    __syncthreads();
    p2 = 0.f;
#pragma unroll
    for (int w = 0; w < SKW; ++w) p2 += st[w][1][lane & 7];
    const float rstd = 1.0f / sqrtf(p2 / (float)K + a.eps);
#pragma unroll
    for (int u = 0; u < SK; ++u)
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int e = 0; e < 4; ++e) xv[u][q][e] = (xv[u][q][e] - mean) * rstd * gv[u][q][e] + bv[u][q][e];
  }
  f32x4_t acc = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int u = 0; u < SK; ++u) {
    if (s_beg + u >= s_end) break;
    const uint32_t w4[4] = {wv[u].x, wv[u].y, wv[u].z, wv[u].w};
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float wf = __uint_as_float(e & 1 ? w4[e >> 1] & 0xffff0000u : w4[e >> 1] << 16);
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(wf, xv[u][e >> 2][e & 3], acc, 0, 0, 0);
    }
  }
  // the useful quadrants, as in fold_rows_kernel
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float v = acc[e] + __shfl_down(acc[e], 40, SSD_WAVE);
    if (lane < 24 && !(lane & 8)) part[wave][4 * (lane >> 4) + e][lane & 7] = v;
  }
  __syncthreads();
  if (tid >= 64 || et >= M || en >= n_out) return;
  float v = 0.f;
#pragma unroll
  for (int w = 0; w < SKW; ++w) v += part[w][ef][et];
  a.y[(size_t)et * a.ldy + en] = LN ? gelu_tanh(v + bias) : y_old + (v + bias);
}

// The rows of K a block's eight waves hold in registers: at most 8 steps of 64 each
bool dense_rows_ok(const LinearArgs& a) {
  return a.wdtype == 1 && a.M >= 2 && a.M <= 8 && a.n_mats == 1 && a.K % 64 == 0 && a.K <= 64 * SKW * 8 &&
         a.ldx % 4 == 0 && a.bias &&
         ((a.norm == NORM_LN && a.epi == EPI_BIAS_GELU) || (a.norm == NORM_NONE && a.epi == EPI_BIAS_RESID));
}

template <bool LN>
hipError_t launch_dense_rows(const LinearArgs& a, hipStream_t s) {
  const dim3 grid((a.n_per + 7) / 8), block(64 * SKW);
  const int spw = (a.K / 64 + SKW - 1) / SKW;
  if (spw <= 2) hipLaunchKernelGGL((dense_rows_kernel<LN, 2>), grid, block, 0, s, a);
  else if (spw <= 4) hipLaunchKernelGGL((dense_rows_kernel<LN, 4>), grid, block, 0, s, a);
  else hipLaunchKernelGGL((dense_rows_kernel<LN, 8>), grid, block, 0, s, a);
  return hipGetLastError();
}

// Vector-path launch shape: MB input rows per block (grid.y = row blocks), blocks over row groups.
struct GvPlan {
  int mb, blocks;
};

GvPlan gv_plan(const LinearArgs& a) {
  GvPlan p;
  const int kpad = (a.K + 7) & ~7;
  int mb = a.M < 1 ? 1 : (a.M > 8 ? 8 : a.M);
  while (mb > 1 && mb * kpad > GV_LDS_FLOATS) --mb;
  p.mb = mb;
  const bool gated = (a.epi == EPI_GATED_GELU || a.epi == EPI_GATED_SILU);
  const int n_total = gated ? a.n_per : a.n_per * a.n_mats;
  const int n_pairs = gated ? a.n_per : (n_total + 1) / 2;
  const int groups = (n_pairs + GV_WAVES - 1) / GV_WAVES;
  p.blocks = groups;
  return p;
}

template <typename WT, int MB, int KP>
hipError_t launch_gemv_kp(const LinearArgs& a, const GvPlan& p, hipStream_t s) {
  static bool attr = false;
  if (!attr) {
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&gemv_kernel<WT, MB, KP>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, GV_LDS_FLOATS * 4);
    attr = true;
  }
  dim3 grid(p.blocks, (a.M + MB - 1) / MB);
  if (a.norm == NORM_SOFTMAX) return hipErrorInvalidValue;
  const size_t shm = (size_t)MB * ((a.K + 7) & ~7) * sizeof(float);
  hipLaunchKernelGGL((gemv_kernel<WT, MB, KP>), grid, dim3(256), shm, s, a);
  return hipGetLastError();
}

}  // namespace

// whole rows up to 12 pieces of 512 elements (6144) in one batch (2 or 4 pieces for short rows),
// else batches of 8
int gemv_pieces(int K) {
  const int pieces = (K + 511) / 512;
  if (pieces <= 2) return 2;
  if (pieces <= 4) return 4;
  if (pieces <= 8 || pieces > 12) return 8;
  return 12;
}

namespace {

template <typename WT, int MB>
hipError_t launch_gemv_mb(const LinearArgs& a, const GvPlan& p, hipStream_t s) {
  switch (gemv_pieces(a.K)) {
    case 2: return launch_gemv_kp<WT, MB, 2>(a, p, s);
    case 4: return launch_gemv_kp<WT, MB, 4>(a, p, s);
    case 12: return launch_gemv_kp<WT, MB, 12>(a, p, s);
    default: return launch_gemv_kp<WT, MB, 8>(a, p, s);
  }
}

template <typename WT>
hipError_t launch_gemv_t(const LinearArgs& a, hipStream_t s) {
  const GvPlan p = gv_plan(a);
  switch (p.mb) {
    case 1: return launch_gemv_mb<WT, 1>(a, p, s);
    case 2: return launch_gemv_mb<WT, 2>(a, p, s);
    case 3: return launch_gemv_mb<WT, 3>(a, p, s);
    case 4: return launch_gemv_mb<WT, 4>(a, p, s);
    case 5: return launch_gemv_mb<WT, 5>(a, p, s);
    case 6: return launch_gemv_mb<WT, 6>(a, p, s);
    case 7: return launch_gemv_mb<WT, 7>(a, p, s);
    default: return launch_gemv_mb<WT, 8>(a, p, s);
  }
}

}  // namespace

int argmax_parts_max(int n_out) {
  const int groups = ((n_out + 1) / 2 + GV_WAVES - 1) / GV_WAVES;
  const int tiles = n_out > 16 ? (n_out + 15) / 16 : 2;  // the many-row kernel: two a column tile
  return groups > tiles ? groups : tiles;
}

// Steps per batch of loads of the folded cross-attention: as many as the registers allow (12), then
// balanced so that the wave's last batch is not a short one padded with clamped re-reads.
// Instantiated depths: 1, 2, 4, 8, 10, 12.
int fold_depth(int K) {
  const int spw = (K / 64 + SKW - 1) / SKW, batches = (spw + 11) / 12, want = (spw + batches - 1) / batches;
  const int opts[6] = {1, 2, 4, 8, 10, 12};
  for (int i = 0; i < 6; ++i)
    if (opts[i] >= want) return opts[i];
  return 12;
}

bool fold_rows_ok(int d_model, int n_fold, int group, int M) {
  // the consumer of the output's partial sums of squares reads at most SSQ_MAX of them, and so does
  // the scores product, after a residual projection on half tiles
  return M >= 2 && M <= 8 && d_model % 64 == 0 && d_model / 8 <= SSQ_MAX && n_fold % 64 == 0 &&
         (group == 8 || group == 16 || group == 32) && n_fold % group == 0;
}

template <bool RMS>
void launch_fold_sk(const LinearArgs& b, hipStream_t s) {
  const dim3 grid((b.n_per + 7) / 8), block(64 * SKW);
  switch (fold_depth(b.K)) {
    case 1: hipLaunchKernelGGL((fold_rows_kernel<RMS, 1>), grid, block, 0, s, b); break;
    case 2: hipLaunchKernelGGL((fold_rows_kernel<RMS, 2>), grid, block, 0, s, b); break;
    case 4: hipLaunchKernelGGL((fold_rows_kernel<RMS, 4>), grid, block, 0, s, b); break;
    case 8: hipLaunchKernelGGL((fold_rows_kernel<RMS, 8>), grid, block, 0, s, b); break;
    case 10: hipLaunchKernelGGL((fold_rows_kernel<RMS, 10>), grid, block, 0, s, b); break;
    default: hipLaunchKernelGGL((fold_rows_kernel<RMS, 12>), grid, block, 0, s, b); break;
  }
}

hipError_t launch_fold_rows(const LinearArgs& a, hipStream_t s, int* n_ssq) {
  const bool smx = a.norm == NORM_SOFTMAX;
  if (a.wdtype != SSD_F32 || a.n_mats != 1 || a.M < 2 || a.M > 8 || a.K % 64 || a.n_per < 1)
    return hipErrorInvalidValue;
  if (smx) {
    if (a.epi != EPI_RESID || !a.in_f32 || a.in_ld % 4 || a.stash ||
        (a.group != 8 && a.group != 16 && a.group != 32) || a.K % a.group)
      return hipErrorInvalidValue;
    if (n_ssq) *n_ssq = (a.n_per + 7) / 8;
    launch_fold_sk<false>(a, s);
  } else {
    if (a.norm != NORM_RMS || a.epi != EPI_STORE || !a.in_planes || !a.in_ssq || a.in_nssq < 1 ||
        a.in_nssq > SSQ_MAX)
      return hipErrorInvalidValue;
    launch_fold_sk<true>(a, s);
  }
  return hipGetLastError();
}

double linear_bytes(const LinearArgs& a) {
  const bool gated = (a.epi == EPI_GATED_GELU || a.epi == EPI_GATED_SILU);
  const double n_w = (double)a.n_per * (gated ? 2 : a.n_mats);
  const double n_out = gated ? a.n_per : n_w;
  const double welem = a.wdtype == 1 ? 2.0 : 4.0;
  double bytes = n_w * a.K * welem + (double)a.M * a.K * 4.0;
  if (a.epi == EPI_ARGMAX) bytes += a.logits ? (double)a.M * n_out * 4.0 : 0.0;
  else bytes += (double)a.M * n_out * 4.0 * (a.epi == EPI_RESID || a.epi == EPI_BIAS_RESID ? 2.0 : 1.0);
  return bytes;
}

hipError_t launch_linear(LinearArgs a, hipStream_t s, int* n_parts, LaunchTiming* timing) {
  if (a.M <= 0) return hipSuccess;
  // the softmax input transform exists on the one-row register path only
  if (a.norm == NORM_SOFTMAX &&
      (a.M != 1 || a.K > 6144 || (a.group != 8 && a.group != 16 && a.group != 32 && a.group != 64) ||
       a.K % a.group))
    return hipErrorInvalidValue;
  if (a.epi == EPI_ARGMAX) a.n_parts = gv_plan(a).blocks;
  if (n_parts) *n_parts = a.n_parts;
  bool one = false;
  const hipError_t e = launch_one_row(a, s, timing, &one);
  if (one) return e;
  if (dense_rows_ok(a)) return a.norm == NORM_LN ? launch_dense_rows<true>(a, s) : launch_dense_rows<false>(a, s);
  return a.wdtype == 1 ? launch_gemv_t<bf16_t>(a, s) : launch_gemv_t<float>(a, s);
}

}  // namespace ssd
