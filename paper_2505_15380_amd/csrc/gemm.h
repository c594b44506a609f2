// Skinny GEMMs of the decoder: Y[M,N] = X[M,Kd] . W[N,Kd]^T with M = rows of one forward (<= 512).
// Up to a few tens of rows the work is weight streaming: every weight byte is read once, coalesced, and the
// contraction runs on MFMA 16x16x32 bf16 tiles (rows padded to 16; padded rows cost nothing that matters).
//
// Work decomposition, identical for both storage types:
//   a workgroup (4 waves) owns two 16-column tiles (t0 from W0, t1 from W1) and one global k-split;
//   its waves split the k range between them, partial tiles are summed through LDS in a fixed order,
//   and one thread per (row, col) applies the epilogue.  Nothing is accumulated with atomics, so every output
//   element has one summation order that does not depend on M: a row computed alone (autoregressive step)
//   and the same row computed among K+1 (verification) give the same bits.
//
// bf16 weights are pre-packed so that a wave reads one tile (16 out-features x 32 in-features) as 64
// consecutive 16-byte pieces: piece l of tile (nt, kt) = W[nt*16 + l%16][kt*32 + 8*(l/16) .. +7], tiles ordered
// [nt][kt].  That is exactly the B-operand fragment of the MFMA, so a weight goes from HBM to the matrix
// core through one dwordx4 load and nothing else.
#pragma once
#include "common.h"

namespace ssd {

enum { EPI_PARTIAL = 0, EPI_QKV = 1, EPI_SWIGLU = 2, EPI_RESID = 3 };

struct GemmArgs {
  const void* A;     // activations [M][lda]
  int lda;
  const void* W0;    // weight matrix of tile slot 0 (packed bf16, or canonical fp32 [N][K])
  const void* W1;    // weight matrix of tile slot 1
  int M, N, K;       // N = out features of one matrix (unpadded)
  int gs;            // global k-splits
  // EPI_PARTIAL: out[s][m][n]
  float* out;
  size_t out_split_stride;
  int ldo;
  // EPI_QKV: bias, rotary table, destination of q and of the cache rows
  const float* bias;
  const float2* rope;   // [pos][hd/2] (cos, sin)
  Rows rows;
  float* q;             // [M][nq*hd]
  KvView kv;
  int layer, nq;
  // EPI_SWIGLU
  void* act;            // [M][N]
  int act_split_kt;     // > 0: act is written as split rows (common.h) with this many k-tiles per row (N / 32)
  // the norm between two GEMMs without a pass of its own (bf16).  EPI_RESID adds the residual and leaves what the next GEMM
  // needs: its operand h * gain, and each row's sum of squares over every 16 columns.  EPI_SWIGLU with rms_d > 0 divides
  // its results by the row's r.m.s. computed from these.
  float* h;             // EPI_RESID: residual stream [M][N], updated
  const float* gain;    // EPI_RESID: gain of the norm that follows
  void* hg;             // EPI_RESID: h * gain as split rows
  float* sumsq;         // [M][rms_d / 16] written by EPI_RESID, read by EPI_SWIGLU
  int rms_d;            // columns of the normalised row; 0: the operand is normalised already
  float rms_eps;
};

// ------------------------------------------------------------------------------------------ epilogues
template <int EPI, typename AT, typename KVT>
__device__ __forceinline__ void gemm_epilogue(const GemmArgs& g, int t0, int t1, int split, int row, int col,
                                              float v0, float v1) {
  if (row >= g.M) return;
  if (EPI == EPI_PARTIAL) {
    float* o = g.out + (size_t)split * g.out_split_stride + (size_t)row * g.ldo;
    const int n0 = t0 * 16 + col, n1 = t1 * 16 + col;
    if (n0 < g.N) o[n0] = v0;
    if (n1 < g.N) o[n1] = v1;
  } else if (EPI == EPI_SWIGLU) {
    const int n = t0 * 16 + col;
    if (n < g.N) {
      const float s = v0 / (1.0f + expf(-v0));
      if (g.act_split_kt > 0) st_split_value((bf16_t*)g.act, g.act_split_kt, row, n, s * v1);
      else AT::st((typename AT::T*)g.act + (size_t)row * g.N + n, s * v1);
    }
  } else {  // EPI_QKV: the two tiles hold dims d and d + hd/2 of one head
    const int hd = g.kv.hd, half = hd >> 1;
    const int n0 = t0 * 16 + col;
    const int head = n0 / hd, d = n0 - head * hd;
    if (g.bias) { v0 += g.bias[n0]; v1 += g.bias[n0 + half]; }
    const int nq = g.nq, nkv = g.kv.nkv;
    const int pos = g.rows.pos[row];
    if (head < nq + nkv) {
      const float2 cs = g.rope[(size_t)pos * half + d];
      const float r0 = v0 * cs.x - v1 * cs.y;
      const float r1 = v1 * cs.x + v0 * cs.y;
      v0 = r0; v1 = r1;
    }
    if (head < nq) {
      float* qo = g.q + (size_t)row * nq * hd + head * hd + d;
      qo[0] = v0; qo[half] = v1;
    } else if (g.rows.active[row]) {
      const int which = head < nq + nkv ? 0 : 1;
      const int kvh = head - nq - which * nkv;
      const int seq = g.rows.seq0 + row / g.rows.R;
      const int blk = g.kv.table[seq * g.kv.mbps + pos / g.kv.bt];
      if (blk >= 0) {
        typename KVT::T* base = (typename KVT::T*)g.kv.pool + kv_offset(g.kv, g.layer, which, blk, kvh, 0);
        const int tok = pos % g.kv.bt;
        if (which == 0) {                                   // keys: [token][dim]
          KVT::st(base + tok * hd + d, v0);
          KVT::st(base + tok * hd + d + half, v1);
        } else {                                            // values: [dim][token] (token-minor)
          KVT::st(base + d * g.kv.bt + tok, v0);
          KVT::st(base + (d + half) * g.kv.bt + tok, v1);
        }
      }
    }
  }
}

template <int EPI>
__device__ __forceinline__ bool gemm_tiles(const GemmArgs& g, int item, int hd, int& t0, int& t1, int& split) {
  const int ntiles = (g.N + 15) >> 4;
  if (EPI == EPI_PARTIAL) {
    const int npairs = (ntiles + 1) >> 1;
    split = item / npairs;
    const int p = item - split * npairs;
    t0 = 2 * p; t1 = 2 * p + 1;
  } else if (EPI == EPI_SWIGLU) {
    split = 0; t0 = item; t1 = item;
  } else {
    const int per_head = hd >> 5;              // pairs of tiles per head
    const int head = item / per_head, i = item - head * per_head;
    split = 0; t0 = head * (hd >> 4) + i; t1 = t0 + per_head;
  }
  return t0 < ntiles;
}

// Sum the four waves' partial tiles (fixed order) and run the epilogue: thread tid owns (row tid/16, col tid%16).
template <int EPI, typename AT, typename KVT>
__device__ __forceinline__ void gemm_reduce_tile(const GemmArgs& g, float (*red)[2][256], int t0, int t1, int split,
                                                 int mt) {
  const int tid = threadIdx.x;
  const float v0 = (red[0][0][tid] + red[1][0][tid]) + (red[2][0][tid] + red[3][0][tid]);
  const float v1 = (red[0][1][tid] + red[1][1][tid]) + (red[2][1][tid] + red[3][1][tid]);
  gemm_epilogue<EPI, AT, KVT>(g, t0, t1, split, mt * 16 + (tid >> 4), tid & 15, v0, v1);
}

// -------------------------------------------------------------------------------------- fp32 / VALU
// Same decomposition for the fp32 parity configuration; weights canonical [N][K] fp32, K % 32 == 0.
template <int EPI, typename KVT>
__global__ void __launch_bounds__(BLOCK) k_gemm_f32(GemmArgs g) {
  __shared__ float red[4][2][256];
  int t0, t1, split;
  if (!gemm_tiles<EPI>(g, blockIdx.x, g.kv.hd, t0, t1, split)) return;
  const int ntiles = (g.N + 15) >> 4;
  const bool has1 = (EPI != EPI_PARTIAL) || (t1 < ntiles);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int KT = g.K >> 5;
  const int per_s = KT / g.gs, rem_s = KT - per_s * g.gs;
  const int wg_b = split * per_s + min(split, rem_s), wg_n = per_s + (split < rem_s ? 1 : 0);
  const int per_w = wg_n >> 2, rem_w = wg_n & 3;
  const int kb = wg_b + wave * per_w + min(wave, rem_w), ke = kb + per_w + (wave < rem_w ? 1 : 0);
  const int col = lane & 15, kg = lane >> 4;
  const int n0 = min(t0 * 16 + col, g.N - 1), n1 = min((has1 ? t1 : t0) * 16 + col, g.N - 1);
  const float* w0 = (const float*)g.W0 + (size_t)n0 * g.K;
  const float* w1 = (const float*)g.W1 + (size_t)n1 * g.K;
  const float* A = (const float*)g.A;
  const int MTn = (g.M + 15) >> 4;
  for (int mt = 0; mt < MTn; ++mt) {
    float a0[16], a1[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) { a0[r] = 0.f; a1[r] = 0.f; }
    const int rows = min(16, g.M - mt * 16);
    for (int k = kb * 32 + kg; k < ke * 32; k += 4) {
      const float x0 = w0[k], x1 = w1[k];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        if (r < rows) {
          const float a = A[(size_t)(mt * 16 + r) * g.lda + k];
          a0[r] = fmaf(a, x0, a0[r]);
          a1[r] = fmaf(a, x1, a1[r]);
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      float s0 = a0[r], s1 = a1[r];
      s0 += __shfl_xor(s0, 16, WAVE); s0 += __shfl_xor(s0, 32, WAVE);
      s1 += __shfl_xor(s1, 16, WAVE); s1 += __shfl_xor(s1, 32, WAVE);
      if (kg == 0) { red[wave][0][r * 16 + col] = s0; red[wave][1][r * 16 + col] = s1; }
    }
    __syncthreads();
    gemm_reduce_tile<EPI, F32, KVT>(g, red, t0, has1 ? t1 : ntiles, split, mt);
  }
}

// Repack a canonical bf16 matrix [N][K] into MFMA B-fragment tiles (see the top of this file).
// One thread per 16-byte piece; rows >= N are zero.
__global__ void k_pack_bf16(const bf16_t* __restrict__ w, uint4* __restrict__ out, int N, int K, int ntiles) {
  const int KT = K >> 5;
  const size_t total = (size_t)ntiles * KT * 64;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (size_t)gridDim.x * blockDim.x) {
    const int l = (int)(i & 63);
    const size_t tile = i >> 6;
    const int kt = (int)(tile % KT), nt = (int)(tile / KT);
    const int n = nt * 16 + (l & 15), k = kt * 32 + (l >> 4) * 8;
    uint4 v = uint4{0, 0, 0, 0};
    if (n < N) v = *(const uint4*)(w + (size_t)n * K + k);
    out[i] = v;
  }
}

}  // namespace ssd
