// GEMMs of the decoder, Y[M,N] = X[M,K] . W[N,K]^T with M = rows of one forward: what both storage types share (arguments,
// epilogues) and the fp32 kernel.  The bf16 kernels are in gemm_tile.h.
//
// No output element is accumulated with atomics, so a launch gives the same bits every time.  fp32: an element's order of sums
// follows from K alone, and a row has the same bits alone (autoregressive step) and among K + 1 (verification).  bf16: the
// kernel, its tile and the k-slices are chosen from the launch's sizes, and the order of sums with them.
//
// bf16 weights are pre-packed so that a wave reads one tile (16 out-features x 32 in-features) as 64
// consecutive 16-byte pieces: piece l of tile (nt, kt) = W[nt*16 + l%16][kt*32 + 8*(l/16) .. +7], tiles ordered
// [nt][kt].  That is exactly an operand fragment of the MFMA, so a weight goes from HBM to the matrix
// core through one dwordx4 load and nothing else.
#pragma once
#include "common.h"

namespace ssd {

enum { EPI_PARTIAL = 0, EPI_QKV = 1, EPI_SWIGLU = 2, EPI_RESID = 3 };

struct GemmArgs {
  const void* A;     // activations: fp32 [M][K], or split rows (common.h)
  const void* W0;    // weight matrix of tile slot 0 (packed bf16, or canonical fp32 [N][K])
  const void* W1;    // weight matrix of tile slot 1
  int M, N, K;       // N = out features of one matrix (unpadded)
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
  // the norm before a GEMM without a pass of its own.  fp32: A is the residual stream, and a kernel given a `gain` normalises
  // its rows itself (and EPI_RESID only adds to the residual stream).  bf16: EPI_RESID adds the residual and leaves what the next GEMM
  // needs: its operand h * gain, and each row's sum of squares, over every 16 columns (launches of up to 64 rows) or in sum_pieces
  // pieces.  EPI_SWIGLU with rms_d > 0 divides its results by the row's r.m.s. computed from these.
  float* h;             // EPI_RESID: residual stream [M][N], updated
  const float* gain;    // fp32: gain of the norm before; bf16, EPI_RESID: gain of the norm that follows
  void* hg;             // EPI_RESID: h * gain as split rows
  float* sumsq;         // written by EPI_RESID, read by EPI_SWIGLU: [M][rms_d / 16], or [M][sum_pieces rounded up to 16]
  int sum_pieces;       // bf16: > 0: pieces that a row's sum of squares is in; 0: one per 16 columns (EPI_RESID: any other value asks for pieces)
  int rms_d;            // columns of the normalised row; 0: the operand is normalised already
  float rms_eps;
};

// ------------------------------------------------------------------------------------------ epilogues
// One output row's columns `col` of the tiles t0 and t1 (t1 beyond the last tile: nothing there).
template <int EPI>
__device__ __forceinline__ void gemm_epilogue_f32(const GemmArgs& g, int t0, int t1, int row, int col, float v0, float v1, int pos, int blk,
                                                  float2 cs) {
  const int n0 = t0 * 16 + col, n1 = t1 * 16 + col;
  if (EPI == EPI_PARTIAL) {
    float* o = g.out + (size_t)row * g.ldo;
    if (n0 < g.N) o[n0] = v0;
    if (n1 < g.N) o[n1] = v1;
  } else if (EPI == EPI_RESID) {
    float* o = g.h + (size_t)row * g.N;
    if (n0 < g.N) o[n0] += v0;
    if (n1 < g.N) o[n1] += v1;
  } else if (EPI == EPI_SWIGLU) {
    if (n0 < g.N) ((float*)g.act)[(size_t)row * g.N + n0] = v0 / (1.0f + expf(-v0)) * v1;
  } else {  // EPI_QKV: the two tiles hold dims d and d + hd/2 of one head
    const int hd = g.kv.hd, half = hd >> 1;
    const int head = n0 / hd, d = n0 - head * hd;
    if (g.bias) { v0 += g.bias[n0]; v1 += g.bias[n0 + half]; }
    const int nq = g.nq, nkv = g.kv.nkv;
    if (head < nq + nkv) {
      const float r0 = v0 * cs.x - v1 * cs.y;
      const float r1 = v1 * cs.x + v0 * cs.y;
      v0 = r0; v1 = r1;
    }
    if (head < nq) {
      float* qo = g.q + (size_t)row * nq * hd + head * hd + d;
      qo[0] = v0; qo[half] = v1;
    } else if (blk >= 0) {
      const int which = head < nq + nkv ? 0 : 1;
      const int kvh = head - nq - which * nkv;
      float* base = (float*)g.kv.pool + kv_offset(g.kv, g.layer, which, blk, kvh, 0);
      const int tok = pos % g.kv.bt;
      if (which == 0) {                                     // keys: [token][dim]
        base[tok * hd + d] = v0;
        base[tok * hd + d + half] = v1;
      } else {                                              // values: [dim][token] (token-minor)
        base[d * g.kv.bt + tok] = v0;
        base[(d + half) * g.kv.bt + tok] = v1;
      }
    }
  }
}

// ------------------------------------------------------------------------------------------------------------ fp32
// Weights canonical fp32 [N][K], K % 32 == 0, on v_mfma_f32_16x16x4_f32: full fp32 products and sums.  A workgroup owns 16
// rows x two column tiles (t0 from W0, t1 from W1; EPI_QKV: the tiles that hold dims d and d + hd/2 of one head) and its 4 to
// 16 waves share the k range in steps of 16: a lane loads 16 bytes of each operand, four consecutive k, and the step's four
// instructions take one of them each from every lane.  The waves' sums meet in LDS in wave order.
//
// With a gain, A is the residual stream and the kernel normalises it: it multiplies by the gain as it loads, sums the
// squares beside the products and divides the results by the r.m.s. at the end, so no kernel runs between two GEMMs.
//
// What bounds it at the sizes that fp32 is used at (a few rows, widths of 64 to 512) is the length of one workgroup's chain -
// launch, operands, reduction, epilogue - so a wave has at most four steps, all requested at once, before more waves run
// out.  Five rows of width 128: 3.5 to 4.8 us, where a kernel on vector units with a scalar load per k took 9.6.
constexpr int GF_MAX_WAVES = 16;

template <int EPI>
__global__ void __launch_bounds__(GF_MAX_WAVES * 64) k_gemm_f32(GemmArgs g) {
  __shared__ float red[GF_MAX_WAVES][2][256];
  __shared__ float red_ss[GF_MAX_WAVES][16];
  const int ntiles = (g.N + 15) >> 4;
  int t0, t1;
  if (EPI == EPI_QKV) {
    const int per_head = g.kv.hd >> 5, head = blockIdx.x / per_head, i = blockIdx.x - head * per_head;
    t0 = head * (g.kv.hd >> 4) + i; t1 = t0 + per_head;
  } else if (EPI == EPI_SWIGLU) {
    t0 = t1 = blockIdx.x;
  } else {
    t0 = 2 * blockIdx.x; t1 = t0 + 1;
  }
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), nw = blockDim.x >> 6;
  const int steps = g.K >> 4, per = steps / nw, rem = steps - per * nw;
  const int kb = wave * per + min(wave, rem), ke = kb + per + (wave < rem ? 1 : 0);
  const int li = lane & 15, kg = lane >> 4, m0 = blockIdx.y * 16;
  const f32x4* w0 = (const f32x4*)((const float*)g.W0 + (size_t)min(t0 * 16 + li, g.N - 1) * g.K) + kg;
  const f32x4* w1 = (const f32x4*)((const float*)g.W1 + (size_t)min(t1 * 16 + li, g.N - 1) * g.K) + kg;
  const f32x4* ap = (const f32x4*)((const float*)g.A + (size_t)min(m0 + li, g.M - 1) * g.K) + kg;
  const f32x4* gp = (const f32x4*)g.gain + kg;
  constexpr int U = 4;
  f32x4 acc0 = {0, 0, 0, 0}, acc1 = {0, 0, 0, 0};
  float ss = 0.f;
  // EPI_QKV: where the row's key and value go and its rotation, requested behind the operands
  const int row = m0 + (tid >> 4);
  const bool mine = tid < 256 && row < g.M;
  int pos = 0, active = 0, blk = -1;
  float2 cs = {0.f, 0.f};
  if (EPI == EPI_QKV && mine) { pos = g.rows.pos[row]; active = g.rows.active[row]; }
  int k = kb;
  do {                                                     // (also by a wave without steps, K / 16 < nw: its threads have rows to request)
    f32x4 a[U], x0[U], x1[U], gn[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int kk = min(k + u, ke - 1) * 4;
      a[u] = ap[kk]; x0[u] = w0[kk]; x1[u] = w1[kk];
      if (g.gain) gn[u] = gp[kk];
    }
    if (EPI == EPI_QKV && mine && k == kb) {
      cs = g.rope[(size_t)pos * (g.kv.hd >> 1) + (t0 * 16 + (tid & 15)) % g.kv.hd];
      blk = g.kv.table[(g.rows.seq0 + row / g.rows.R) * g.kv.mbps + pos / g.kv.bt];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (k + u >= ke) break;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        float x = a[u][j];
        if (g.gain) { ss = fmaf(x, x, ss); x *= gn[u][j]; }
        acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(x, x0[u][j], acc0, 0, 0, 0);
        acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(x, x1[u][j], acc1, 0, 0, 0);
      }
    }
    k += U;
  } while (k < ke);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    red[wave][0][(4 * kg + r) * 16 + li] = acc0[r];
    red[wave][1][(4 * kg + r) * 16 + li] = acc1[r];
  }
  if (g.gain) {
    ss += __shfl_xor(ss, 16, WAVE); ss += __shfl_xor(ss, 32, WAVE);
    if (kg == 0) red_ss[wave][li] = ss;
  }
  __syncthreads();
  if (!mine) return;
  float v0 = 0.f, v1 = 0.f, tot = 0.f;
  for (int w = 0; w < nw; ++w) {
    v0 += red[w][0][tid];
    v1 += red[w][1][tid];
    tot += g.gain ? red_ss[w][tid >> 4] : 0.f;
  }
  if (g.gain) {
    const float inv = 1.0f / sqrtf(tot / (float)g.K + g.rms_eps);
    v0 *= inv; v1 *= inv;
  }
  gemm_epilogue_f32<EPI>(g, t0, t1, row, tid & 15, v0, v1, pos, active ? blk : -1, cs);
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
