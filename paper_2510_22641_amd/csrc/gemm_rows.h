// The weight-streaming kernel over row planes and its launchers; gemm.hip chooses the shape, and the
// gemm_rows_*.hip sources instantiate it one epilogue each (they compile side by side).
#pragma once

#include "device.h"
#include "gemv_common.h"
#include "kernels.h"

#include <climits>

namespace ssd {

// Launch shape of gemv_rows_kernel.
struct RowsShape {
  int mode, nt, rg;
};

hipError_t launch_rows_bias(const LinearArgs& a, RowsShape sh, int blocks, hipStream_t s);
hipError_t launch_rows_store_rms(const LinearArgs& a, RowsShape sh, int blocks, hipStream_t s);
hipError_t launch_rows_resid(const LinearArgs& a, RowsShape sh, int blocks, hipStream_t s);
hipError_t launch_rows_qkv(const LinearArgs& a, RowsShape sh, int blocks, hipStream_t s);
hipError_t launch_rows_gated(const LinearArgs& a, RowsShape sh, int blocks, hipStream_t s);
hipError_t launch_rows_cross(const LinearArgs& a, RowsShape sh, int blocks, hipStream_t s);
hipError_t launch_rows_argmax(const LinearArgs& a, RowsShape sh, int blocks, hipStream_t s);

namespace {

__device__ __forceinline__ const bf16_t* mat_ptr(const LinearArgs& a, int mat) {
  return reinterpret_cast<const bf16_t*>(pick_matrix(a, mat));
}

// Element of the cross-attention caches: row m = b Nv + n, feature f = h dh + e of layer l.
__device__ __forceinline__ size_t cross_at(const LinearArgs& a, int l, int m, int f) {
  const int b = m / a.n_visual, n = m - b * a.n_visual, sh = __builtin_ctz(a.d_head), h = f >> sh;
  return ((((size_t)l * a.cross_batch + b) * a.n_heads + h) * a.n_visual + n) * a.d_head + (f - (h << sh));
}

// ---------------------------------------------------------------------------------------------
// Weight streaming over RG row groups of 16: a block of eight waves owns NT tiles of 16 weight rows
// and 16 RG input rows; wave w takes an eighth of K.  Per 64-element step a wave reads a tile's rows
// as 128 contiguous bytes a row, eight lanes each (the vector memory path takes a quad of lanes with
// contiguous addresses as one access: with a row per lane, the order of the matrix operands, a load
// is 64 accesses instead of 8 and those bound the kernel), and passes them through its own LDS to
// the operand order; the plane fragments are operands as they lie.  U steps a batch, the next batch
// requested before the current one's products; the eight partial tiles are summed through LDS.  The
// blocks of a tile's row blocks run on one XCD (workgroups are dealt to the 8 XCDs round-robin), so
// that its weights cross the fabric once.
//
// A tile is 16 consecutive features; for QKV eight rotary pairs (rows r and r + 8: columns c + r and
// c + r + dh/2 of one head of one matrix), for the gated FFN eight features (rows r: gate, r + 8: up).
//
// MODE (at most 8 input rows, RG 1):
//  * GR_PACK: the B operand's columns carry the hi plane of rows 0..7 and, in columns 8..15, their
//    lo plane, so that one load and one product cover both; column t + 8 is added to column t.
//  * GR_HALF: a tile is 8 features (twice the blocks); the A operand holds them twice, over the two K
//    blocks of a step, and B's columns are the 8 rows over the same two: D[f][t] + D[f + 8][t + 8].
constexpr int GR_WAVES = 8;
enum GrMode { GR_FULL = 0, GR_PACK = 1, GR_HALF = 2 };

// 16-byte loads a lane and step of the weights and of the planes
constexpr int gr_wloads(int mode, int nt) { return mode == GR_HALF ? nt : 2 * nt; }
constexpr int gr_aloads(int mode, int rg) { return mode == GR_FULL ? 4 * rg : 2; }
// registers of two one-step batches and the accumulators within a wave's share (QKV's addresses and
// rotary factors come on top: of 4 tiles and 2 groups it spills three registers)
constexpr bool gr_fits(int nt, int rg) { return 16 * (nt + 2 * rg) + 4 * nt * rg <= 170; }
// steps a batch that two batches' registers hold, and that one's hold
constexpr int gr_batch(int mode, int nt, int rg) {
  const int u = (168 - 4 * nt * rg) / (8 * (gr_wloads(mode, nt) + gr_aloads(mode, rg)));
  return u < 1 ? 1 : (u > 6 ? 6 : u);
}
constexpr int gr_one(int mode, int nt, int rg) {
  return (192 - 4 * nt * rg) / (4 * (gr_wloads(mode, nt) + gr_aloads(mode, rg)));
}

// The epilogue is a template parameter: with no branch on it ahead of the first loads, every load
// of the prologue goes out in one burst instead of waiting for the branches' arguments in turn.
enum GrKind { GR_BIAS = 0, GR_STORE_RMS, GR_RESID, GR_QKV, GR_GATED, GR_ARGMAX, GR_CROSS };

// ONE: a wave's share of K fits one batch (everything it reads is in flight at once).  ONCE: one row
// block, so each weight is read by one block only and need not stay in the caches (at 12 rows of the
// LLaMA-7B shape gate/up 38.0 -> 35.0 us; with several row blocks it costs, 21.6 -> 25.6 us for the
// QKV of 72 rows at the FlanT5-xl shape).
template <int KIND, int MODE, int NT, int RG, int U, bool ONE, bool ONCE>
__global__ __launch_bounds__(64 * GR_WAVES) void gemv_rows_kernel(const LinearArgs a) {
  constexpr bool qkv = KIND == GR_QKV, gated = KIND == GR_GATED, resid = KIND == GR_RESID;
  constexpr bool rms = KIND == GR_STORE_RMS || qkv || gated || KIND == GR_ARGMAX;
  constexpr int ROWS = 16 * RG, TF = MODE == GR_HALF ? 8 : 16;
  constexpr int WL = MODE == GR_HALF ? 1 : 2;  // 1 KB pieces (8 rows x 64 elements) of a tile and step
  constexpr int SP = 64 * GR_WAVES / ROWS;     // threads that share a row's partial sums of squares
  constexpr int SV = RG >= 3 && NT >= 2 ? 8 : 16;  // of which each thread requests this many up front
  constexpr int RP = (ROWS + 31) / 32;         // rows per thread in the epilogue
  static_assert(MODE == GR_FULL || RG == 1, "8 rows");
  // staging of a step's weights [wave][NT][WL][1 KB], then the partial tiles [wave][NT][RG][16][17]
  extern __shared__ __attribute__((aligned(16))) float part[];
  __shared__ float ssq_red[SP][ROWS];
  __shared__ float rs[ROWS];

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, c = lane & 15;
  const int K = a.K, M = a.M, ng = a.row_groups, ssq_ld = 16 * ng;
  const int n_out = qkv ? 3 * a.n_per : a.n_per;
  constexpr int tf = gated ? 8 : TF;           // features a tile
  const int tiles = (n_out + tf - 1) / tf;
  // GR_CROSS: matrix mtx of the table
  const int mtx = KIND == GR_CROSS ? blockIdx.z / a.tab_z : 0;
  const int by = blockIdx.y, bx = (blockIdx.z - mtx * a.tab_z) * 8 + blockIdx.x;
  const int t0 = by * ROWS, j0 = bx * NT;
  if (j0 >= tiles) return;  // the whole block

  // QKV tile vt: matrix and first column (d_head is 64 or 128: d_head / 16 tiles a head)
  const int half = a.d_head >> 1, sh = qkv ? __builtin_ctz(a.d_head >> 4) : 0, per_mat = a.n_heads << sh;
  auto qkv_tile = [&](int vt, int& mat, int& c8) {
    mat = vt >= 2 * per_mat ? 2 : (vt >= per_mat ? 1 : 0);
    const int rem = vt - mat * per_mat, h = rem >> sh;
    c8 = h * a.d_head + 8 * (rem - (h << sh));
  };
  // this lane's weight row of each piece: row lane / 8, elements 8 (lane % 8) .. of a step
  const bf16_t* wrow[NT][WL];
  const bf16_t* w0 = reinterpret_cast<const bf16_t*>(KIND == GR_CROSS ? a.wtab[mtx] : a.w[0]);
#pragma unroll
  for (int j = 0; j < NT; ++j)
#pragma unroll
    for (int hf = 0; hf < WL; ++hf) {
      const int vt = min(j0 + j, tiles - 1), r = lane >> 3;
      const bf16_t* p;
      if (qkv) {
        int m, c8;
        qkv_tile(vt, m, c8);
        p = mat_ptr(a, m) + (size_t)(c8 + r + hf * half) * K;
      } else if (gated) {
        p = mat_ptr(a, hf) + (size_t)min(vt * 8 + r, a.n_per - 1) * K;
      } else {
        p = w0 + (size_t)min(vt * TF + 8 * hf + r, n_out - 1) * K;
      }
      wrow[j][hf] = p + (lane & 7) * 8;
    }
  // this lane's plane elements of K block 0 of step 0 (a row group past the last repeats it and is
  // never stored)
  constexpr int AL = MODE == GR_FULL ? RG : 1;
  const bf16_t* brow[AL];
#pragma unroll
  for (int i = 0; i < AL; ++i) {
    const bf16_t* p = a.in_planes + (size_t)min(RG * by + i, ng - 1) * PLANE_FRAG;
    if (MODE == GR_FULL) p += lane * 8;
    else p += (g * 16 + (c & 7)) * 8 + (MODE == GR_PACK && c >= 8 ? PLANE_LO : 0);
    if (MODE == GR_HALF && c >= 8) p += (size_t)ng * PLANE_FRAG;  // K block 1
    brow[i] = p;
  }
  const size_t kstep = (size_t)ng * PLANE_FRAG;

  // requested before the main batches (the wait counter retires loads in issue order): partial
  // sums of squares, the old residual values and the sequence lengths of this thread's outputs
  float sv[SV];
  const int srow = tid % ROWS, sp0 = tid / ROWS;
  if (rms) {
#pragma unroll
    for (int i = 0; i < SV; ++i)
      sv[i] = a.in_ssq[(size_t)min(sp0 + SP * i, a.in_nssq - 1) * ssq_ld + min(t0 + srow, M - 1)];
  }
  const int f = tid & 15, rr = tid >> 4;  // epilogue: feature f of a tile, rows rr + 32 i
  constexpr bool pre = resid && NT == 1;  // (with several tiles they are read in the epilogue)
  float y_old[RP], gain = 1.f;
  int qpos[RP];
#pragma unroll
  for (int i = 0; i < RP; ++i) {
    const int tg = min(t0 + rr + 32 * i, M - 1);
    qpos[i] = qkv ? a.kv.seq_len[tg / a.C] : 0;
    y_old[i] = pre ? a.y[(size_t)tg * a.ldy + min(j0 * TF + f, n_out - 1)] : 0.f;
  }
  if (pre) gain = (a.out_gain ? a.out_gain : a.y)[min(j0 * TF + f, n_out - 1)];

  f32x4_t acc[NT][RG];
#pragma unroll
  for (int j = 0; j < NT; ++j)
#pragma unroll
    for (int i = 0; i < RG; ++i) acc[j][i] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  const int steps = K / 64;
  const int s_beg = steps * wave / GR_WAVES, s_end = steps * (wave + 1) / GR_WAVES;
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  // Blocks that start together would ask the caches for the same plane fragments at the same time:
  // each wave starts its range at a step of its own and wraps around (W_o of 72 rows at the
  // FlanT5-xl shape 10.4 -> 9.7 us).
  const int rot = s_end > s_beg ? (bx + by + wave) % (s_end - s_beg) : 0;
  struct Batch {
    u32x4 w[U][NT][WL];
    bf16x8_t x[U][2][MODE == GR_FULL ? 2 * RG : 1];  // [K block or, GR_HALF, plane][group][hi, lo]
  };
  auto load = [&](Batch& q, int s0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      int st = min(s0 + u, s_end - 1) + rot;
      if (st >= s_end) st -= s_end - s_beg;
      st = max(st, 0);
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int hf = 0; hf < WL; ++hf) {
          const u32x4* p = reinterpret_cast<const u32x4*>(wrow[j][hf] + st * 64);
          q.w[u][j][hf] = ONCE ? __builtin_nontemporal_load(p) : *p;
        }
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int i = 0; i < AL; ++i) {
          if (MODE == GR_HALF) {
            q.x[u][kb][0] = *reinterpret_cast<const bf16x8_t*>(brow[0] + 2 * st * kstep + kb * PLANE_LO);
          } else {
            const bf16_t* p = brow[i] + (2 * st + kb) * kstep;
            if (MODE == GR_PACK) {
              q.x[u][kb][0] = *reinterpret_cast<const bf16x8_t*>(p);
            } else {
              q.x[u][kb][2 * i] = *reinterpret_cast<const bf16x8_t*>(p);
              q.x[u][kb][2 * i + 1] = *reinterpret_cast<const bf16x8_t*>(p + PLANE_LO);
            }
          }
        }
    }
    __builtin_amdgcn_sched_barrier(0);  // the whole batch in flight before the products
  };
  // the wave's staging: chunk (lane % 8) of a piece's row r = lane / 8 at position chunk ^ r, so that
  // the eight rows an operand read takes together lie in different banks
  unsigned char* stage = reinterpret_cast<unsigned char*>(part) + (size_t)wave * NT * WL * 1024;
  unsigned char* wr = stage + (lane >> 3) * 128 + (((lane & 7) ^ (lane >> 3)) << 4);
  const unsigned char* rd = stage + (MODE == GR_HALF ? 0 : (c >> 3) * 1024) + (c & 7) * 128;
  const int ch0 = MODE == GR_HALF ? 4 * (c >> 3) + g : g;  // this lane's chunk (K block 1: + 4)
  const int rpos[2] = {(ch0 ^ (c & 7)) << 4, ((ch0 ^ 4) ^ (c & 7)) << 4};
  auto mul = [&](const Batch& q, int s0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (s0 + u >= s_end) break;  // uniform over the wave
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int hf = 0; hf < WL; ++hf) *reinterpret_cast<u32x4*>(wr + (j * WL + hf) * 1024) = q.w[u][j][hf];
#pragma unroll
      for (int kb = 0; kb < (MODE == GR_HALF ? 1 : 2); ++kb)
#pragma unroll
        for (int j = 0; j < NT; ++j) {
          const bf16x8_t w = *reinterpret_cast<const bf16x8_t*>(rd + j * WL * 1024 + rpos[kb]);
          if (MODE == GR_HALF) {
            acc[j][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, q.x[u][0][0], acc[j][0], 0, 0, 0);
            acc[j][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, q.x[u][1][0], acc[j][0], 0, 0, 0);
          } else if (MODE == GR_PACK) {
            acc[j][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, q.x[u][kb][0], acc[j][0], 0, 0, 0);
          } else {
#pragma unroll
            for (int i = 0; i < RG; ++i)
              acc[j][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, q.x[u][kb][2 * i], acc[j][i], 0, 0, 0);
#pragma unroll
            for (int i = 0; i < RG; ++i)
              acc[j][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, q.x[u][kb][2 * i + 1], acc[j][i], 0, 0, 0);
          }
        }
    }
  };
  // the page entries and rotary factors of this thread's outputs go out behind the first batch
  // (lane f of 8: pair f of each tile)
  QkvPre pq[qkv ? RP : 1][qkv ? NT : 1];
  auto request_qkv = [&]() {
    if constexpr (qkv) {
#pragma unroll
      for (int i = 0; i < RP; ++i) {
        const int tg = min(t0 + rr + 32 * i, M - 1), b = tg / a.C, pos = qpos[i] + a.kv.pos_off + (tg - b * a.C);
        const int page = a.kv.page_table[(size_t)b * a.kv.max_pages + min(pos >= 0 ? pos / a.kv.page_size : 0, a.kv.max_pages - 1)];
        const int tp = pos < 0 ? 0 : (pos >= a.max_seq ? a.max_seq - 1 : pos);
#pragma unroll
        for (int j = 0; j < NT; ++j) {
          pq[i][j] = {pos, page, 1.f, 0.f};
          int m, c8;
          qkv_tile(min(j0 + j, tiles - 1), m, c8);
          if (a.rope_cos && m < 2) {
            const size_t o = (size_t)tp * half + (c8 & (a.d_head - 1)) + (f & 7);
            pq[i][j].cs = a.rope_cos[o];
            pq[i][j].sn = a.rope_sin[o];
          }
        }
      }
    }
  };
  if constexpr (ONE) {
    Batch q;
    load(q, s_beg);
    request_qkv();
    mul(q, s_beg);
  } else {
    Batch q0, q1;
    int s0 = s_beg;
    load(q0, s0);
    request_qkv();
    for (;;) {
      if (s0 + U >= s_end) { mul(q0, s0); break; }
      load(q1, s0 + U);
      mul(q0, s0);
      s0 += U;
      if (s0 + U >= s_end) { mul(q1, s0); break; }
      load(q0, s0 + U);
      mul(q1, s0);
      s0 += U;
    }
  }

  // D[feature 4 g + e][row c] of each tile and row group, over the staging (everyone is done with it)
  __syncthreads();
#pragma unroll
  for (int j = 0; j < NT; ++j)
#pragma unroll
    for (int i = 0; i < RG; ++i) {
      float* p = part + (((size_t)wave * NT + j) * RG + i) * (16 * 17) + c;
#pragma unroll
      for (int e = 0; e < 4; ++e) p[(4 * g + e) * 17] = acc[j][i][e];
    }
  if (rms && sp0 < SP) {
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < SV; ++i) s += sp0 + SP * i < a.in_nssq ? sv[i] : 0.f;
    for (int p = sp0 + SP * SV; p < a.in_nssq; p += SP) s += a.in_ssq[(size_t)p * ssq_ld + min(t0 + srow, M - 1)];
    ssq_red[sp0][srow] = s;
  }
  __syncthreads();
  if (rms) {
    if (tid < ROWS) {
      float s2 = 0.f;
#pragma unroll
      for (int i = 0; i < SP; ++i) s2 += ssq_red[i][tid];
      rs[tid] = 1.0f / sqrtf(s2 / (float)K + a.eps);
    }
    __syncthreads();
  }

#pragma unroll
  for (int i = 0; i < RP; ++i) {
    const int row = rr + 32 * i, tg = t0 + row;
    if (ROWS % 32 && row >= ROWS) break;  // whole waves: ROWS is a multiple of 16
    const bool rok = tg < M;
    if (MODE != GR_FULL && row >= 8) break;  // whole waves
    const float rscale = rms ? rs[row] : 1.f;
    auto out = [&](int j) {
      const float* p = part + ((size_t)j * RG + (row >> 4)) * (16 * 17) + f * 17 + (row & 15);
      const float* p2 = MODE == GR_PACK ? p + 8 : p + 8 * 17 + 8;
      float v = 0.f;
#pragma unroll
      for (int w = 0; w < GR_WAVES; ++w) {
        v += p[(size_t)w * NT * RG * (16 * 17)];
        if (MODE == GR_PACK || (MODE == GR_HALF && f < 8)) v += p2[(size_t)w * NT * RG * (16 * 17)];
      }
      return v * rscale;
    };
    float best = -INFINITY, y2 = 0.f;
    int besti = INT_MAX;
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      const int vt = j0 + j, n = vt * tf + f;
      const bool ok = rok && vt < tiles && f < tf && n < n_out;
      const float v = out(j);
      if (qkv || gated) {
        const float v1 = __shfl_xor(v, 8, SSD_WAVE);
        if (!rok || vt >= tiles || f >= 8) continue;
        if constexpr (qkv) {
          int m, c8;
          qkv_tile(vt, m, c8);
          qkv_store_pre(a, m, c8 + f, tg, pq[i][j], v, v1);
        } else if (ok) {
          store_planes1(a.out_planes + plane_at(tg, n, ng), apply_epi_act(a.epi, v, v1));
        }
        continue;
      }
      if (!ok) continue;
      if (KIND == GR_ARGMAX) {
        argmax_merge(best, besti, v, n);
        if (a.logits) a.logits[(size_t)tg * a.ldl + n] = v;
        continue;
      }
      if constexpr (KIND == GR_CROSS) {
        const size_t o = cross_at(a, mtx >> 1, tg, n);
        void* dst = mtx & 1 ? a.cross_v : a.cross_k;
        if (a.kvdtype == 1) store_elem(reinterpret_cast<bf16_t*>(dst) + o, v);
        else store_elem(reinterpret_cast<float*>(dst) + o, v);
        continue;
      }
      float* yp = a.y + (size_t)tg * a.ldy + n;
      if (resid) {
        const float t = (pre ? y_old[i] : *yp) + v;
        *yp = t;
        if (a.stash) a.stash[(size_t)tg * a.lds + n] = t;
        if (a.out_planes)
          store_planes1(a.out_planes + plane_at(tg, n, ng), a.out_gain ? (pre ? gain : a.out_gain[n]) * t : t);
        y2 = fmaf(t, t, y2);
      } else if (KIND == GR_BIAS && a.epi == EPI_BIAS_GELU) {
        const float t = gelu_tanh(v + a.bias[n]);
        *yp = t;
        if (a.out_planes) store_planes1(a.out_planes + plane_at(tg, n, ng), t);
      } else if (KIND == GR_BIAS) {
        *yp = (a.resid ? a.resid[(size_t)tg * a.ldr + n] : 0.f) + (v + a.bias[n]);
      } else {
        *yp = v;
      }
    }
    // the row's 16 lanes: the block's argmax partial, or its partial sum of squares
    if (KIND == GR_ARGMAX) {
#pragma unroll
      for (int o = 8; o > 0; o >>= 1) {
        const float v2 = __shfl_xor(best, o, SSD_WAVE);
        const int i2 = __shfl_xor(besti, o, SSD_WAVE);
        argmax_merge(best, besti, v2, i2);
      }
      if (f == 0 && rok) {
        a.part_val[(size_t)tg * a.n_parts + bx] = best;
        a.part_idx[(size_t)tg * a.n_parts + bx] = besti;
      }
    } else if (resid && a.out_ssq) {
#pragma unroll
      for (int o = 8; o > 0; o >>= 1) y2 += __shfl_xor(y2, o, SSD_WAVE);
      if (f == 0 && rok) a.out_ssq[(size_t)bx * ssq_ld + tg] = y2;
    }
  }
}

template <int KIND, int MODE, int NT, int RG, int U, bool ONE, bool ONCE>
hipError_t launch_rows_u(const LinearArgs& a, int blocks, hipStream_t s) {
  constexpr int st = GR_WAVES * NT * (MODE == GR_HALF ? 1 : 2) * 1024, pt = GR_WAVES * NT * RG * 16 * 17 * 4;
  constexpr int shm = st > pt ? st : pt;
  if constexpr (shm > 56 * 1024) {
    static bool attr = false;
    if (!attr) {
      (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&gemv_rows_kernel<KIND, MODE, NT, RG, U, ONE, ONCE>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, shm);
      attr = true;
    }
  }
  // workgroups go to the 8 XCDs by linear id: x is the XCD
  LinearArgs b = a;
  b.tab_z = (blocks + 7) / 8;
  const dim3 grid(8, (a.M + 16 * RG - 1) / (16 * RG), b.tab_z * (KIND == GR_CROSS ? a.n_tab : 1));
  hipLaunchKernelGGL((gemv_rows_kernel<KIND, MODE, NT, RG, U, ONE, ONCE>), grid, dim3(64 * GR_WAVES), shm, s, b);
  return hipGetLastError();
}

// Steps a batch: a wave's whole share of K when the registers hold it and the blocks are one round
// (with more the extra registers would cost the blocks that run beside each other: the LM head of 6
// rows 32 us against 36), else double-buffered batches of as many as they hold.  One-batch depths are 2,
// 4 and 10, to keep the instances few: a wave of 5 to 9 steps reads its last one again, from cache.
// (Verify of 5 rows of four T5 layers 2560 wide, 5 steps a wave, 353 us; 445 with the kernel before,
// whose depths were balanced.)
template <int KIND, int MODE, int NT, int RG>
hipError_t launch_rows_t(const LinearArgs& a, int blocks, hipStream_t s) {
  constexpr int one = gr_one(MODE, NT, RG), u = gr_batch(MODE, NT, RG);
  const int row_blocks = (a.M + 16 * RG - 1) / (16 * RG);
  if (KIND != GR_CROSS && (long long)blocks * row_blocks <= cu_count()) {
    const int per_wave = (a.K / 64 + GR_WAVES - 1) / GR_WAVES;
    if constexpr (one >= 2) if (per_wave <= 2) return launch_rows_u<KIND, MODE, NT, RG, 2, true, MODE != GR_FULL>(a, blocks, s);
    if constexpr (one >= 4) if (per_wave <= 4) return launch_rows_u<KIND, MODE, NT, RG, 4, true, MODE != GR_FULL>(a, blocks, s);
    if constexpr (one >= 10) if (per_wave <= 10) return launch_rows_u<KIND, MODE, NT, RG, 10, true, MODE != GR_FULL>(a, blocks, s);
  }
  if constexpr (MODE == GR_FULL) if (row_blocks > 1) return launch_rows_u<KIND, MODE, NT, RG, u, false, false>(a, blocks, s);
  return launch_rows_u<KIND, MODE, NT, RG, u, false, true>(a, blocks, s);
}

template <int KIND, int NT>
hipError_t launch_rows_nt(const LinearArgs& a, RowsShape sh, int blocks, hipStream_t s) {
  if constexpr (KIND == GR_BIAS) {  // the imitation network past 8 rows
    if (sh.mode != GR_FULL) return hipErrorInvalidValue;
  } else {
    if (sh.mode == GR_PACK) return launch_rows_t<KIND, GR_PACK, NT, 1>(a, blocks, s);
    if constexpr (NT == 1 && (KIND == GR_STORE_RMS || KIND == GR_RESID))
      if (sh.mode == GR_HALF) return launch_rows_t<KIND, GR_HALF, 1, 1>(a, blocks, s);
  }
  if (sh.rg == 1) return launch_rows_t<KIND, GR_FULL, NT, 1>(a, blocks, s);
  if constexpr (gr_fits(NT, 2)) if (sh.rg == 2) return launch_rows_t<KIND, GR_FULL, NT, 2>(a, blocks, s);
  if constexpr (gr_fits(NT, 3)) if (sh.rg == 3) return launch_rows_t<KIND, GR_FULL, NT, 3>(a, blocks, s);
  if constexpr (gr_fits(NT, 4)) if (sh.rg == 4) return launch_rows_t<KIND, GR_FULL, NT, 4>(a, blocks, s);
  return hipErrorInvalidValue;
}

template <int KIND>
hipError_t launch_rows_kind(const LinearArgs& a, RowsShape sh, int blocks, hipStream_t s) {
  switch (sh.nt) {
    case 1: return launch_rows_nt<KIND, 1>(a, sh, blocks, s);
    case 2: return launch_rows_nt<KIND, 2>(a, sh, blocks, s);
    case 3: return launch_rows_nt<KIND, 3>(a, sh, blocks, s);
    default: return launch_rows_nt<KIND, 4>(a, sh, blocks, s);
  }
}

}  // namespace

}  // namespace ssd
