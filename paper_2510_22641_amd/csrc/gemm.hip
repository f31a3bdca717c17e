// Linear layers over two rows and more with bf16 weights (verify chunks, batched draft steps, prefill
// blocks).  The inputs arrive as two bf16 planes hi = bf16(v), lo = bf16(v - hi) of
// v = g * x (g the RMSNorm gain, or 1), written once by their producer, so both planes against the
// weights keep the activations at about 16 mantissa bits; 1/rms of a row comes from the partial
// sums of squares its producer left and scales the outputs.
//
//  * gemv_rows_kernel (gemm_rows.h) - up to 128 rows: weights and planes go straight from memory
//    into registers, K split over a block's eight waves.  Bound: HBM bytes of W, and the loads a
//    compute unit issues.
//  * gemm_ring_kernel - long row blocks: LDS tiles filled by direct global-to-LDS loads in a ring
//    of K steps.  Bound: the matrix cores and the LDS reads that feed them.
//
// Both end in the epilogues of the one-row kernels: store, residual (+ stash, next planes, partial
// sums of squares), gated activation to planes, bias + GELU, bias + residual, per-block argmax
// partials, and QKV with rotary and the paged KV store.
#include "device.h"
#include "gemv_common.h"
#include "gemm_rows.h"
#include "kernels.h"

#include <climits>

namespace ssd {

int cu_count() {
  static const int cus = [] {
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
      n = 256;
    return n;
  }();
  return cus;
}

namespace {

// Planes of a pass's first rows, one block per row: gain * x and the row's sum of squares (ssq[m],
// one partial), or with `shift` the LayerNorm (x - mean) / sqrt(var + eps) * gain + shift.
__global__ __launch_bounds__(256) void rows_prep_kernel(const float* __restrict__ x, int ldx, int K,
                                                        const float* __restrict__ gain,
                                                        const float* __restrict__ shift, float eps,
                                                        bf16_t* __restrict__ out, int ng,
                                                        float* __restrict__ ssq) {
  __shared__ float red[2][4];
  const int m = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const float* xr = x + (size_t)m * ldx;
  float mean = 0.f, rstd = 1.f;
  if (shift) {
    float s1 = 0.f;
    for (int k = tid * 4; k < K; k += 1024) {
      const float4 v = *reinterpret_cast<const float4*>(xr + k);
      s1 += (v.x + v.y) + (v.z + v.w);
    }
    s1 = wave_sum(s1);
    if (lane == 0) red[0][wave] = s1;
    __syncthreads();
    mean = ((red[0][0] + red[0][1]) + (red[0][2] + red[0][3])) / (float)K;
    float s2 = 0.f;
    for (int k = tid * 4; k < K; k += 1024) {
      const float4 v = *reinterpret_cast<const float4*>(xr + k);
      const float a = v.x - mean, b = v.y - mean, c = v.z - mean, d = v.w - mean;
      s2 += (a * a + b * b) + (c * c + d * d);
    }
    s2 = wave_sum(s2);
    if (lane == 0) red[1][wave] = s2;
    __syncthreads();
    rstd = 1.0f / sqrtf(((red[1][0] + red[1][1]) + (red[1][2] + red[1][3])) / (float)K + eps);
  }
  float s2 = 0.f;
  for (int k = tid * 4; k < K; k += 1024) {
    float4 v = *reinterpret_cast<const float4*>(xr + k);
    const float4 g = gain ? *reinterpret_cast<const float4*>(gain + k) : make_float4(1.f, 1.f, 1.f, 1.f);
    if (shift) {
      const float4 t = *reinterpret_cast<const float4*>(shift + k);
      v = make_float4((v.x - mean) * rstd * g.x + t.x, (v.y - mean) * rstd * g.y + t.y,
                      (v.z - mean) * rstd * g.z + t.z, (v.w - mean) * rstd * g.w + t.w);
    } else {
      s2 += (v.x * v.x + v.y * v.y) + (v.z * v.z + v.w * v.w);
      v = make_float4(v.x * g.x, v.y * g.y, v.z * g.z, v.w * g.w);
    }
    store_planes4(out + plane_at(m, k, ng), v.x, v.y, v.z, v.w);
  }
  if (!ssq || shift) return;
  s2 = wave_sum(s2);
  if (lane == 0) red[0][wave] = s2;
  __syncthreads();
  if (tid == 0) ssq[m] = (red[0][0] + red[0][1]) + (red[0][2] + red[0][3]);
}

// y[m] += p_0[m] + ... + p_{S-1}[m] over the K-range partials of a residual projection, in range
// order; the next projection's planes and partial sums of squares (one per column slice) with it.
// Block (16-row group, slice of KSUM_COLS columns); a lane owns eight elements as the plane
// fragments lay them out, so that a wave writes whole fragments and reads 128 bytes a row.
constexpr int KSUM_COLS = 256;

__global__ __launch_bounds__(256) void ksum_rows_kernel(const LinearArgs a, int n_out) {
  __shared__ float red[4][16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int row = lane & 15, m = blockIdx.x * 16 + row;
  const bool ok = m < a.M;
  float s2 = 0.f;
#pragma unroll
  for (int u = 0; u < KSUM_COLS / 128; ++u) {
    const int n = blockIdx.y * KSUM_COLS + (u * 4 + wave) * 32 + (lane >> 4) * 8;
    if (!ok || n >= n_out) continue;  // n_out is a multiple of 8
    float* yp = a.y + (size_t)m * a.ldy + n;
    float4 y[2], p[4][2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      y[q] = reinterpret_cast<const float4*>(yp)[q];
#pragma unroll
      for (int s = 0; s < 4; ++s)
        if (s < a.ksplit)
          p[s][q] = reinterpret_cast<const float4*>(a.kpart + ((size_t)s * a.kpart_rows + m) * a.kpart_ld + n)[q];
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      float4 t = p[0][q];
#pragma unroll
      for (int s = 1; s < 4; ++s)
        if (s < a.ksplit) { t.x += p[s][q].x; t.y += p[s][q].y; t.z += p[s][q].z; t.w += p[s][q].w; }
      y[q].x += t.x; y[q].y += t.y; y[q].z += t.z; y[q].w += t.w;
      reinterpret_cast<float4*>(yp)[q] = y[q];
      if (a.stash) reinterpret_cast<float4*>(a.stash + (size_t)m * a.lds + n)[q] = y[q];
      s2 += (y[q].x * y[q].x + y[q].y * y[q].y) + (y[q].z * y[q].z + y[q].w * y[q].w);
      if (a.out_gain) {
        const float4 g = reinterpret_cast<const float4*>(a.out_gain + n)[q];
        y[q].x *= g.x; y[q].y *= g.y; y[q].z *= g.z; y[q].w *= g.w;
      }
    }
    if (a.out_planes) {
      uint4 hi, lo;
      split_bf16x8_v(y[0], y[1], hi, lo);
      bf16_t* pp = a.out_planes + plane_at(m, n, a.row_groups);
      *reinterpret_cast<uint4*>(pp) = hi;
      *reinterpret_cast<uint4*>(pp + PLANE_LO) = lo;
    }
  }
  if (!a.out_ssq) return;
  s2 += __shfl_xor(s2, 16, SSD_WAVE);
  s2 += __shfl_xor(s2, 32, SSD_WAVE);
  if (lane < 16) red[wave][lane] = s2;
  __syncthreads();
  if (tid < 16 && ok)
    a.out_ssq[(size_t)blockIdx.y * 16 * a.row_groups + m] = (red[0][tid] + red[1][tid]) + (red[2][tid] + red[3][tid]);
}

// QKV column tiles: tiles 2u and 2u + 1 of 16 features are columns c .. c + 15 and c + dh/2 ..
// c + dh/2 + 15 of one head of one matrix (the rotary pairs; d_head is 64 or 128); returns the
// matrix and c.
__device__ __forceinline__ void qkv_pair_tile(const LinearArgs& a, int u, int& mat, int& c) {
  const int sh = __builtin_ctz(a.d_head >> 5), per_mat = a.n_heads << sh;
  mat = u >= 2 * per_mat ? 2 : (u >= per_mat ? 1 : 0);
  const int rem = u - mat * per_mat, h = rem >> sh;
  c = h * a.d_head + 16 * (rem - (h << sh));
}

// ---------------------------------------------------------------------------------------------
// LDS ring: a block of four waves (2 x 2) owns 32 MI rows x 32 NJ features (a gated block: 16 NJ
// features of both matrices), each wave 16 MI rows x 16 NJ features.  K advances in steps of KB
// blocks of 32: a step's plane fragments and weight rows go from memory into one of NS LDS stages
// by 16-byte direct loads, NS - 1 steps ahead, with one barrier a step; the 16-byte chunks of a
// weight row are permuted by its row number on the way in, so that eight rows of a fragment
// read lie in different banks (the planes lie in fragment order already).  The weights are the A operand: a
// lane then holds four consecutive features of a row.
template <int MI, int NJ, int KB, int NS>
constexpr int ring_lds() { return NS * KB * (4 * MI + 2 * NJ) * 1024; }

enum RingKind { RING_PLAIN = 0, RING_GATED = 1, RING_QKV = 2, RING_CROSS = 3 };

template <int KIND, int MI, int NJ, int KB, int NS>
__global__ __launch_bounds__(256, 2) void gemm_ring_kernel(const LinearArgs a) {
  constexpr bool GATED = KIND == RING_GATED, qkv = KIND == RING_QKV;
  constexpr int BM = 32 * MI, BN = 32 * NJ;
  constexpr int RGS = 2 * MI;                  // row groups of 16
  constexpr int RK = 32 * KB;                  // elements of a step
  constexpr int PR = 16 / KB;                  // weight rows of a 1 KB piece
  constexpr int AP = KB * 2 * RGS, WP = BN / PR;  // 1 KB pieces of a stage: plane fragments [K block]
                                                  // [row group][hi, lo], then PR weight rows each
  static_assert(KB == 1 || KB == 2, "rows of 64 or 128 bytes");
  constexpr int STAGE = (AP + WP) * 1024;      // bytes
  constexpr int PW = (AP + WP) / 4;            // pieces a wave loads per stage
  static_assert((AP + WP) % 4 == 0, "whole pieces per wave");
  static_assert(NS >= 2 && NS <= 4, "the waits below count at most two later steps");
  extern __shared__ __attribute__((aligned(16))) unsigned char ring[];
  __shared__ float rs[BM];

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1, g = lane >> 4, c = lane & 15;
  const int K = a.K, M = a.M, ng = a.row_groups, ssq_ld = 16 * ng;
  const bool rms = a.norm == NORM_RMS;
  const int n_out = GATED ? a.n_per : a.n_per * a.n_mats;
  // Workgroups are dealt to the 8 XCDs round-robin by linear id, and each XCD has its own L2: the
  // id is mapped to a contiguous range of tiles per XCD (row tiles fastest, then K ranges, then
  // weight tiles), so the blocks that share a weight tile read it through one L2.
  int rt, zs, ct;
  {
    const int nx = gridDim.x, nz = gridDim.z, T = nx * gridDim.y * nz;
    const int id = blockIdx.x + nx * (blockIdx.y + gridDim.y * blockIdx.z);
    const int xcd = id & 7, slot = id >> 3;
    const int t = xcd * (T >> 3) + min(xcd, T & 7) + slot;
    rt = t % nx;
    const int rest = t / nx;
    zs = rest % nz;
    ct = rest / nz;
  }
  const int m0 = rt * BM;
  int nk = K / RK, kb = 0;
  if (KIND != RING_CROSS && a.ksplit > 1) {  // K range zs of a.ksplit (whole steps each)
    const int per = (nk + a.ksplit - 1) / a.ksplit;
    kb = zs * per;
    nk = min(per, nk - kb);
  }

  // this wave's pieces; of a weight piece a lane fills chunk l % (4 KB) of its row l / (4 KB) with the
  // row's chunk (l % 4) ^ ((row / 2) % 4) (KB 1) or (l % 8) ^ (row % 8).  Rows past the matrix repeat its last one and are never stored.
  const char* src[PW];  // uniform: the piece's fragment or matrix row
  uint32_t off[PW];     // this lane's bytes from it
#pragma unroll
  for (int q = 0; q < PW; ++q) {
    const int pc = wave * PW + q;  // uniform over the wave
    if (pc < AP) {
      const int kblk = pc / (2 * RGS), fr = pc % (2 * RGS);
      src[q] = reinterpret_cast<const char*>(
          a.in_planes + ((size_t)(KB * kb + kblk) * ng + min((m0 >> 4) + (fr >> 1), ng - 1)) * PLANE_FRAG + (fr & 1) * PLANE_LO);
      off[q] = lane * 16u;
    } else {
      const int n = (pc - AP) * PR, prow = KB == 1 ? lane >> 2 : lane >> 3;  // local weight rows of the piece
      const uint32_t pch = KB == 1 ? (lane & 3) ^ ((lane >> 3) & 3) : (lane & 7) ^ (lane >> 3);
      int mat = 0, row0, row;    // matrix, its row at the piece's start (uniform), row of this lane
      if (GATED) {
        const int w2 = n / (16 * NJ), r = n - w2 * (16 * NJ);
        mat = r >= 8 * NJ;
        const int first = ct * (BN / 2) + w2 * (8 * NJ) + (r - mat * 8 * NJ);
        row0 = min(first, a.n_per - 1);
        row = min(first + prow, a.n_per - 1);
      } else if (qkv) {
        const int tile = min((ct * BN + n) >> 4, n_out / 16 - 1);
        int c0;
        qkv_pair_tile(a, tile >> 1, mat, c0);
        row0 = c0 + (tile & 1) * (a.d_head >> 1) + (n & 8);
        row = row0 + prow;
      } else {
        row0 = min(ct * BN + n, n_out - 1);
        row = min(ct * BN + n + prow, n_out - 1);
      }
      const bf16_t* wm = KIND == RING_CROSS ? reinterpret_cast<const bf16_t*>(a.wtab[zs]) : mat_ptr(a, mat);
      src[q] = reinterpret_cast<const char*>(wm + (size_t)row0 * K + (size_t)kb * RK);
      off[q] = (uint32_t)(row - row0) * (uint32_t)K * 2u + pch * 16u;
    }
  }
  const uint32_t lds0 = (uint32_t)(size_t)(__attribute__((address_space(3))) unsigned char*)ring;
  auto fetch = [&](int kt) {  // step kt into stage kt % NS
    const uint32_t st = lds0 + (uint32_t)(kt % NS) * STAGE + (uint32_t)wave * PW * 1024;
#pragma unroll
    for (int q = 0; q < PW; ++q) {
      const bool plane = wave * PW + q < AP;
      const char* p = src[q] + (size_t)kt * (plane ? (size_t)ng * (PLANE_FRAG * 2 * KB) : (size_t)(RK * 2));
      // LDS-direct load: lane l's 16 bytes land at M0 + 16 l (one wait state after the M0 write).  (The
      // compiler reserves M0, so it warns of the clobber; it is named all the same, so that no value
      // of its own is expected to live there across the statement.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                   :: "s"(st + q * 1024), "v"(off[q]), "s"(p) : "memory", "m0");
#pragma clang diagnostic pop
    }
  };
#pragma unroll
  for (int s = 0; s < NS - 1; ++s)
    if (s < nk) fetch(s);

  // 1 / rms of the block's rows from the producer's partial sums of squares
  if (rms) {
    constexpr int TP = 256 / BM;  // threads per row
    const int row = tid / TP, p0 = tid % TP, m = min(m0 + row, M - 1);
    float s2 = 0.f;
    for (int p = p0; p < a.in_nssq; p += 16 * TP) {  // 16 requested together
      float v[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) v[u] = a.in_ssq[(size_t)min(p + u * TP, a.in_nssq - 1) * ssq_ld + m];
#pragma unroll
      for (int u = 0; u < 16; ++u) s2 += p + u * TP < a.in_nssq ? v[u] : 0.f;
    }
#pragma unroll
    for (int o = 1; o < TP; o <<= 1) s2 += __shfl_xor(s2, o, SSD_WAVE);
    if (p0 == 0) rs[row] = 1.0f / sqrtf(s2 / (float)K + a.eps);
  }

  f32x4_t acc[NJ][MI];
#pragma unroll
  for (int j = 0; j < NJ; ++j)
#pragma unroll
    for (int i = 0; i < MI; ++i) acc[j][i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  // fragments: planes as they lie; weights row 16 j + c, chunk 4 kb2 + g at its permuted position
  const unsigned char* fa = ring + (size_t)(wm * 2 * MI) * 1024 + lane * 16;
  const unsigned char* fw = ring + AP * 1024 + (size_t)(wn * 16 * NJ + c) * (RK * 2);
  const int wpos[2] = {KB == 1 ? (g ^ ((c >> 1) & 3)) << 4 : (g ^ (c & 7)) << 4, ((4 + g) ^ (c & 7)) << 4};
  // step kt has landed (this wave's own loads; with the barrier everyone's), and everyone is done with
  // the stage the next fetch overwrites (up to NS - 2 later steps, as many as there are, stay in flight)
  auto land = [&](int kt) {
    if (NS >= 4 && kt + 2 < nk) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"(2 * PW) : "memory");
    else if (NS >= 3 && kt + 1 < nk) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"(PW) : "memory");
    else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if (kt + NS - 1 < nk) fetch(kt + NS - 1);
  };
  struct Frags {
    bf16x8_t h[MI], l[MI], w[NJ];
  };
  auto read = [&](Frags& f, int kt, int kb2) {
    const size_t st = (size_t)(kt % NS) * STAGE;
#pragma unroll
    for (int j = 0; j < NJ; ++j) f.w[j] = *reinterpret_cast<const bf16x8_t*>(fw + st + j * (16 * RK * 2) + wpos[kb2]);
#pragma unroll
    for (int i = 0; i < MI; ++i) f.h[i] = *reinterpret_cast<const bf16x8_t*>(fa + st + kb2 * (RGS * 2048) + i * 2048);
#pragma unroll
    for (int i = 0; i < MI; ++i) f.l[i] = *reinterpret_cast<const bf16x8_t*>(fa + st + kb2 * (RGS * 2048) + i * 2048 + 1024);
  };
  auto mul = [&](const Frags& f) {
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int i = 0; i < MI; ++i) acc[j][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.w[j], f.h[i], acc[j][i], 0, 0, 0);
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int i = 0; i < MI; ++i) acc[j][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.w[j], f.l[i], acc[j][i], 0, 0, 0);
  };
  if constexpr (KB == 2) {
    // a K block's operands are read ahead of the products of the one before
    Frags f0, f1;
    land(0);
    read(f0, 0, 0);
    for (int kt = 0; kt < nk; ++kt) {
      read(f1, kt, 1);
      __builtin_amdgcn_sched_barrier(0);
      mul(f0);
      __builtin_amdgcn_sched_barrier(0);
      if (kt + 1 < nk) {
        land(kt + 1);
        read(f0, kt + 1, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
      mul(f1);
      __builtin_amdgcn_sched_barrier(0);
    }
  } else {
    for (int kt = 0; kt < nk; ++kt) {
      Frags f;
      land(kt);
      read(f, kt, 0);
      mul(f);
    }
  }
  if (rms) __syncthreads();

  // epilogue: lane holds features 4 g + e of tile j for row 16 i + c
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    const int ml = wm * 16 * MI + 16 * i + c, m = m0 + ml;
    const bool rok = m < M;
    const float rsc = rms ? rs[ml] : 1.f;
    if constexpr (qkv) {
      const int pos = qkv_pos(a, rok ? m : M - 1), half = a.d_head >> 1;
      const int pg_i = pos >= 0 ? pos / a.kv.page_size : 0;
      const int bq = (rok ? m : M - 1) / a.C;
      const int page = a.kv.page_table[(size_t)bq * a.kv.max_pages + min(pg_i, a.kv.max_pages - 1)];
      const bool cap = pos < 0 || pos >= a.max_seq || pg_i >= a.kv.max_pages;
      const bool bad = page < 0 || page >= a.kv.n_pages;
      const int tp = pos < 0 ? 0 : (pos >= a.max_seq ? a.max_seq - 1 : pos);
#pragma unroll
      for (int u = 0; u < NJ / 2; ++u) {
        const int tile = (ct * BN + wn * 16 * NJ) / 16 + 2 * u;
        if (!rok || tile * 16 >= n_out) continue;
        int mat, c0;
        qkv_pair_tile(a, tile >> 1, mat, c0);
        const int hh = c0 >> __builtin_ctz(a.d_head), d = (c0 & (a.d_head - 1)) + 4 * g;
        float v0[4], v1[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) { v0[e] = acc[2 * u][i][e] * rsc; v1[e] = acc[2 * u + 1][i][e] * rsc; }
        if (mat < 2 && a.rope_cos) {
          const float4 cs4 = *reinterpret_cast<const float4*>(a.rope_cos + (size_t)tp * half + d);
          const float4 sn4 = *reinterpret_cast<const float4*>(a.rope_sin + (size_t)tp * half + d);
          const float cs[4] = {cs4.x, cs4.y, cs4.z, cs4.w}, sn[4] = {sn4.x, sn4.y, sn4.z, sn4.w};
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float r0 = v0[e] * cs[e] - v1[e] * sn[e], r1 = v1[e] * cs[e] + v0[e] * sn[e];
            v0[e] = r0;
            v1[e] = r1;
          }
        }
        if (mat == 0) {
          float* yp = a.y + (size_t)m * a.ldy + c0 + 4 * g;
          *reinterpret_cast<float4*>(yp) = make_float4(v0[0], v0[1], v0[2], v0[3]);
          *reinterpret_cast<float4*>(yp + half) = make_float4(v1[0], v1[1], v1[2], v1[3]);
          continue;
        }
        if (cap || bad) {  // the same bits as qkv_store_pre, and no store
          atomicOr(a.status, cap ? SSD_DEV_CAPACITY : SSD_DEV_BAD_PAGE);
          continue;
        }
        const size_t o = (((size_t)page * a.n_heads + hh) * a.kv.page_size + pos % a.kv.page_size) * a.d_head + d;
        void* base = mat == 2 ? a.kv.v : a.kv.k;
        if (a.kvdtype == 1) {
          bf16_t* p = reinterpret_cast<bf16_t*>(base) + o;
          *reinterpret_cast<uint2*>(p) = make_uint2(pack_bf16x2(v0[0], v0[1]), pack_bf16x2(v0[2], v0[3]));
          *reinterpret_cast<uint2*>(p + half) = make_uint2(pack_bf16x2(v1[0], v1[1]), pack_bf16x2(v1[2], v1[3]));
        } else {
          float* p = reinterpret_cast<float*>(base) + o;
          *reinterpret_cast<float4*>(p) = make_float4(v0[0], v0[1], v0[2], v0[3]);
          *reinterpret_cast<float4*>(p + half) = make_float4(v1[0], v1[1], v1[2], v1[3]);
        }
      }
      continue;
    }
    if constexpr (GATED) {
#pragma unroll
      for (int j = 0; j < NJ / 2; ++j) {
        const int n = ct * (BN / 2) + wn * 8 * NJ + 16 * j + 4 * g;
        float t[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) t[e] = apply_epi_act(a.epi, acc[j][i][e] * rsc, acc[j + NJ / 2][i][e] * rsc);
        if (rok && n < n_out)  // n_per is a multiple of 64
          store_planes4(a.out_planes + plane_at(m, n, ng), t[0], t[1], t[2], t[3]);
      }
      continue;
    }
    float best = -INFINITY, y2 = 0.f;
    int besti = INT_MAX;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int n = ct * BN + wn * 16 * NJ + 16 * j + 4 * g;
      float v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = acc[j][i][e] * rsc;
      if (!rok || n >= n_out) continue;
      if constexpr (KIND == RING_CROSS) {  // matrix zs of the table
        const size_t o = cross_at(a, zs >> 1, m, n);
        void* dst = zs & 1 ? a.cross_v : a.cross_k;
        if (a.kvdtype == 1)
          *reinterpret_cast<uint2*>(reinterpret_cast<bf16_t*>(dst) + o) =
              make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]));
        else
          *reinterpret_cast<float4*>(reinterpret_cast<float*>(dst) + o) = make_float4(v[0], v[1], v[2], v[3]);
        continue;
      }
      if (a.ksplit > 1) {
        *reinterpret_cast<float4*>(a.kpart + ((size_t)zs * a.kpart_rows + m) * a.kpart_ld + n) =
            make_float4(v[0], v[1], v[2], v[3]);
        continue;
      }
      if (a.epi == EPI_ARGMAX) {  // any vocabulary size: one feature at a time
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (n + e < n_out) {
            argmax_merge(best, besti, v[e], n + e);
            if (a.logits) a.logits[(size_t)m * a.ldl + n + e] = v[e];
          }
        continue;
      }
      float4* yp = reinterpret_cast<float4*>(a.y + (size_t)m * a.ldy + n);
      if (a.epi == EPI_RESID) {
        const float4 o = *yp;
        v[0] += o.x; v[1] += o.y; v[2] += o.z; v[3] += o.w;
        *yp = make_float4(v[0], v[1], v[2], v[3]);
        if (a.stash) *reinterpret_cast<float4*>(a.stash + (size_t)m * a.lds + n) = make_float4(v[0], v[1], v[2], v[3]);
        if (a.out_planes) {
          float4 gn = make_float4(1.f, 1.f, 1.f, 1.f);
          if (a.out_gain) gn = *reinterpret_cast<const float4*>(a.out_gain + n);
          store_planes4(a.out_planes + plane_at(m, n, ng), v[0] * gn.x, v[1] * gn.y, v[2] * gn.z, v[3] * gn.w);
        }
        y2 += (v[0] * v[0] + v[1] * v[1]) + (v[2] * v[2] + v[3] * v[3]);
        continue;
      }
      if (a.epi == EPI_BIAS_GELU || a.epi == EPI_BIAS_RESID) {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] += a.bias[n + e];  // (the caller's biases: any alignment)
        if (a.epi == EPI_BIAS_GELU) {
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = gelu_tanh(v[e]);
          if (a.out_planes)
            store_planes4(a.out_planes + plane_at(m, n, ng), v[0], v[1], v[2], v[3]);
        } else if (a.resid) {
          const float4 r = *reinterpret_cast<const float4*>(a.resid + (size_t)m * a.ldr + n);
          v[0] += r.x; v[1] += r.y; v[2] += r.z; v[3] += r.w;
        }
      }
      *yp = make_float4(v[0], v[1], v[2], v[3]);
    }
    // the row's four lanes: the wave's argmax partial, or its partial sum of squares
    if (a.epi == EPI_ARGMAX) {
#pragma unroll
      for (int o = 16; o <= 32; o <<= 1) {
        const float v2 = __shfl_xor(best, o, SSD_WAVE);
        const int i2 = __shfl_xor(besti, o, SSD_WAVE);
        argmax_merge(best, besti, v2, i2);
      }
      if (g == 0 && rok) {
        a.part_val[(size_t)m * a.n_parts + 2 * ct + wn] = best;
        a.part_idx[(size_t)m * a.n_parts + 2 * ct + wn] = besti;
      }
    } else if (a.epi == EPI_RESID && a.ksplit == 1 && a.out_ssq) {
      y2 += __shfl_xor(y2, 16, SSD_WAVE);
      y2 += __shfl_xor(y2, 32, SSD_WAVE);
      if (g == 0 && rok) a.out_ssq[(size_t)(2 * ct + wn) * ssq_ld + m] = y2;
    }
  }
}

// Launch shape of gemv_rows_kernel: NT tiles and RG row groups a block that minimise (blocks per
// compute unit, rounded up) x (16-byte loads a lane and K step): the loads a compute unit issues
// bound the kernel.
RowsShape rows_shape(int n_out, int M, int epi) {
  const bool gated = epi == EPI_GATED_GELU || epi == EPI_GATED_SILU;
  const int tiles = (n_out + (gated ? 7 : 15)) / (gated ? 8 : 16), groups = (M + 15) / 16;
  const long long cus = cu_count();
  RowsShape best = {GR_FULL, 1, 1};
  long long best_cost = -1;
  auto consider = [&](int mode, int nt, int rg, long long blocks) {
    const long long cost = ((blocks + cus - 1) / cus) * (gr_wloads(mode, nt) + gr_aloads(mode, rg));
    if (best_cost < 0 || cost < best_cost) {
      best = {mode, nt, rg};
      best_cost = cost;
    }
  };
  for (int nt = 1; nt <= 4; ++nt) {
    if (M <= 8) {
      consider(GR_PACK, nt, 1, (tiles + nt - 1) / nt);
      continue;
    }
    for (int r = 1; r <= 4; ++r) {
      const int blocks_y = (groups + r - 1) / r, rg = (groups + blocks_y - 1) / blocks_y;
      if (gr_fits(nt, rg)) consider(GR_FULL, nt, rg, (long long)((tiles + nt - 1) / nt) * blocks_y);
    }
  }
  if (M <= 8 && (epi == EPI_RESID || epi == EPI_STORE)) consider(GR_HALF, 1, 1, (n_out + 7) / 8);
  return best;
}

// Forms of gemm_ring_kernel and their measured time (us) per 32-element K step of a compute unit that
// holds 1, 2, ... of their blocks at once (as many as fit its LDS): a lone block's waves wait for
// each other at every step, so small grids want small tiles, and the large tile pays only where two
// of its blocks share a unit.  (Measured over 160..1216 rows, 2048..12288 features, K 2048..11008;
// against 128 x 128 tiles alone: QKV of 488 rows at the FlanT5-xl shape 45 -> 28 us, W_o 25 -> 17,
// gate/up 77 -> 57.)
struct RingForm {
  int mi, nj, kb, ns, fit;
  double us[4];
};
constexpr RingForm RING_FORMS[5] = {
    {4, 8, 1, 2, 2, {1.0, 1.42, 0, 0}},      // 128 x 256
    {4, 4, 1, 2, 3, {0.61, 0.85, 1.27, 0}},  // 128 x 128
    {2, 4, 1, 4, 2, {0.36, 0.52, 0, 0}},     // 64 x 128, four stages (with two stages, and four blocks a unit,
                                             // it never was the cheapest)
    {2, 2, 2, 2, 3, {0.31, 0.40, 0.50, 0}},  // 64 x 64, steps of 64
    {2, 2, 1, 4, 3, {0.25, 0.38, 0.51, 0}},  // 64 x 64, four stages
};

struct RingShape {
  int form, ksplit;
};

// The form, and for residual projections the number of K ranges, with the least estimated time.
RingShape ring_shape(int width, int M, int K, bool can_split, int kpart_max) {
  const int cus = cu_count(), steps = K / 32;
  RingShape best = {0, 1};
  double best_t = -1.0;
  for (int f = 0; f < 5; ++f) {
    const RingForm& rf = RING_FORMS[f];
    const long long tiles = (long long)((M + 32 * rf.mi - 1) / (32 * rf.mi)) * ((width + 32 * rf.nj - 1) / (32 * rf.nj));
    for (int S = 1; S <= (can_split ? (kpart_max < 4 ? kpart_max : 4) : 1); ++S) {
      const int nk = steps / rf.kb, per = (nk + S - 1) / S;
      if ((long long)per * (S - 1) >= nk) break;  // every range holds a step
      const long long r = (tiles * S + cus - 1) / cus, full = r / rf.fit, rest = r % rf.fit;
      double t = (double)(per * rf.kb) * (full * rf.us[rf.fit - 1] + (rest ? rf.us[rest - 1] : 0.0));
      // the second launch: its latency, the partials and the residual
      if (S > 1) t += 3.0 + (double)M * width * (S + 4) * 4.0 / 6.0e6;
      if (best_t < 0.0 || t < best_t) {
        best = {f, S};
        best_t = t;
      }
    }
  }
  return best;
}

template <int KIND, int F>
hipError_t launch_ring_t(const LinearArgs& a, int n_out, hipStream_t s) {
  constexpr int MI = RING_FORMS[F].mi, NJ = RING_FORMS[F].nj, KB = RING_FORMS[F].kb, NS = RING_FORMS[F].ns;
  constexpr int shm = ring_lds<MI, NJ, KB, NS>();
  if constexpr (shm > 60 * 1024) {
    static bool attr = false;
    if (!attr) {
      (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_ring_kernel<KIND, MI, NJ, KB, NS>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, shm);
      attr = true;
    }
  }
  const int width = KIND == RING_GATED ? 2 * n_out : n_out;
  const dim3 grid((a.M + 32 * MI - 1) / (32 * MI), (width + 32 * NJ - 1) / (32 * NJ), KIND == RING_CROSS ? a.n_tab : a.ksplit);
  hipLaunchKernelGGL((gemm_ring_kernel<KIND, MI, NJ, KB, NS>), grid, dim3(256), shm, s, a);
  return hipGetLastError();
}

template <int KIND>
hipError_t launch_ring(const LinearArgs& a, int form, int n_out, hipStream_t s) {
  switch (form) {
    case 0: return launch_ring_t<KIND, 0>(a, n_out, s);
    case 1: return launch_ring_t<KIND, 1>(a, n_out, s);
    case 2: return launch_ring_t<KIND, 2>(a, n_out, s);
    case 3: return launch_ring_t<KIND, 3>(a, n_out, s);
    default: return launch_ring_t<KIND, 4>(a, n_out, s);
  }
}

// Rows the weight-streaming kernel takes.  Verify passes with it, and with the ring kernel in its place:
// FlanT5-xl of 40, 72 and 128 rows 2283, 2582 and 3059 us against 3095, 2984 and 3474, FlanT5-base of
// 128 rows 823 against 1135.  The line is drawn for such layers; with LLaVA-7B's (4096 wide) the two
// meet at 36 to 48 rows (6299 and 6534 against 6148 and 6515) and 96 and 128 rows would be faster on
// the ring kernel (8907 and 10237 against 8151 and 8530).
constexpr int ROWS_MAX = 128;

}  // namespace

hipError_t launch_rows_prep(const float* x, int ldx, int M, int K, const float* gain,
                            const float* shift, float eps, bf16_t* out, float* ssq,
                            hipStream_t s) {
  if (M < 1 || K % 32) return hipErrorInvalidValue;
  hipLaunchKernelGGL(rows_prep_kernel, dim3(M), dim3(256), 0, s, x, ldx, K, gain, shift, eps, out,
                     (M + 15) / 16, ssq);
  return hipGetLastError();
}

size_t rows_ssq_floats(int d_model, int rows) {
  const size_t tiles = (size_t)(d_model + 15) / 16;
  const size_t few = tiles * 2 * 16, mid = tiles * (size_t)((rows < ROWS_MAX ? rows : ROWS_MAX) + 15),
               big = (size_t)(d_model / 32 + 2) * (size_t)(rows + 15);
  const size_t m = few > mid ? few : mid;
  return m > big ? m : big;
}

hipError_t launch_linear_rows(const LinearArgs& args, hipStream_t s, int* n_parts, int* n_ssq) {
  LinearArgs a = args;
  a.row_groups = (a.M + 15) / 16;
  const bool gated = (a.epi == EPI_GATED_GELU || a.epi == EPI_GATED_SILU);
  if (!a.in_planes || a.wdtype != SSD_BF16 || a.K % 64 || a.M < 1 || a.norm == NORM_LN ||
      a.norm == NORM_SOFTMAX || a.n_per < 1)
    return hipErrorInvalidValue;
  if (a.norm == NORM_RMS && (!a.in_ssq || a.in_nssq < 1)) return hipErrorInvalidValue;
  if (gated && (!a.out_planes || a.n_per % 64)) return hipErrorInvalidValue;
  if (a.epi == EPI_QKV ? a.n_mats != 3 || (a.d_head != 64 && a.d_head != 128) : !gated && a.n_mats != 1)
    return hipErrorInvalidValue;
  const int n_out = gated ? a.n_per : a.n_per * a.n_mats;
  const bool cross = a.epi == EPI_CROSS;
  if (cross && (!a.wtab || a.n_tab < 1 || a.norm != NORM_NONE || a.n_visual < 1 || (a.d_head != 64 && a.d_head != 128) ||
                n_out != a.n_heads * a.d_head || !a.cross_k || !a.cross_v))
    return hipErrorInvalidValue;
  LinearArgs b = a;
  b.ksplit = 1;
  if (a.M <= ROWS_MAX) {
    const RowsShape sh = rows_shape(cross ? n_out * a.n_tab : n_out, a.M, a.epi);
    const int tf = gated || sh.mode == GR_HALF ? 8 : 16;
    const int blocks = ((n_out + tf - 1) / tf + sh.nt - 1) / sh.nt;
    if (b.epi == EPI_ARGMAX) b.n_parts = blocks;
    if (n_parts) *n_parts = b.n_parts;
    if (n_ssq) *n_ssq = blocks;
    const bool rms = b.norm == NORM_RMS;
    if (cross) return launch_rows_cross(b, sh, blocks, s);
    if (rms != (b.epi == EPI_STORE || gated || b.epi == EPI_QKV || b.epi == EPI_ARGMAX)) return hipErrorInvalidValue;
    if (b.epi == EPI_STORE) return launch_rows_store_rms(b, sh, blocks, s);
    if (b.epi == EPI_RESID) return launch_rows_resid(b, sh, blocks, s);
    if (b.epi == EPI_QKV) return launch_rows_qkv(b, sh, blocks, s);
    if (gated) return launch_rows_gated(b, sh, blocks, s);
    if (b.epi == EPI_ARGMAX) return launch_rows_argmax(b, sh, blocks, s);
    return launch_rows_bias(b, sh, blocks, s);
  }
  const bool vec = b.epi == EPI_ARGMAX || (n_out % 8 == 0 && b.n_per % 4 == 0);
  if (!vec) return hipErrorInvalidValue;
  const bool split = b.epi == EPI_RESID && b.kpart && n_out <= b.kpart_ld;
  const int width = gated ? 2 * n_out : n_out;
  const RingShape sh = ring_shape(cross ? n_out * a.n_tab : width, a.M, a.K, split, a.kpart_max);
  b.ksplit = sh.ksplit;
  const int nj = RING_FORMS[sh.form].nj, cols = (width + 32 * nj - 1) / (32 * nj);
  if (b.epi == EPI_ARGMAX) b.n_parts = 2 * cols;
  if (n_parts) *n_parts = b.n_parts;
  const int slices = (n_out + KSUM_COLS - 1) / KSUM_COLS;
  if (n_ssq) *n_ssq = sh.ksplit > 1 ? slices : 2 * cols;
  hipError_t e = gated ? launch_ring<RING_GATED>(b, sh.form, n_out, s)
                       : (cross ? launch_ring<RING_CROSS>(b, sh.form, n_out, s)
                       : b.epi == EPI_QKV ? launch_ring<RING_QKV>(b, sh.form, n_out, s)
                                           : launch_ring<RING_PLAIN>(b, sh.form, n_out, s));
  if (e != hipSuccess || sh.ksplit == 1) return e;
  hipLaunchKernelGGL(ksum_rows_kernel, dim3(a.row_groups, slices), dim3(256), 0, s, b, n_out);
  return hipGetLastError();
}

}  // namespace ssd
