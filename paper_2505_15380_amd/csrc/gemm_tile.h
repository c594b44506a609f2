// GEMMs of the decoder with bf16 storage where it runs one launch per operator (more than 16 rows, or head size
// 32), Y[M,N] = X[M,Kd] . W[N,Kd]^T on MFMA 16x16x32 bf16 tiles, on operands that are already in fragment order: weights as packed tiles (gemm.h), activations as split rows (common.h: hi and lo bf16
// halves, 1 KB per fragment).  The weight fragment is the matrix core's first operand, so that an accumulator register
// group holds four consecutive output features of one row: lane l has row l % 16, features 4 (l / 16) .. + 3 of a tile.
#pragma once
#include "gemm.h"

namespace ssd {

// How the output is cut up: blocks of row tiles x blocks of column tiles (x k-slices where the output is k-split
// partials).  Consecutive workgroup indices go to the eight XCDs in turn, and each XCD's L2 fetches what its workgroups read: either the XCDs of a
// slice form a grid of row groups x column groups, each XCD a contiguous rectangle of blocks, so that activations are fetched by as many XCDs as
// there are column groups, and weights by as many as there are row groups; or each XCD takes a contiguous run of the order (slice, column
// block, row block).  The host takes the placement of the least bytes (place_tiles).
struct TilePlan {
  int n_colb, n_rowb, n_slices, slice_kt;     // slice_kt: k-tiles per workgroup
  int per_xcd;                                // workgroups of an XCD
  int rows_xcd, cols_xcd;                     // blocks of an XCD's rectangle; rows_xcd = 0: runs
  int lg_per, lg_colg;                        // logarithms of a slice's XCDs and of its column groups
  uint32_t rows_inv;                          // 2^20 / rows_xcd + 1: i / rows_xcd = i * rows_inv >> 20 for i < 4096 and rows_xcd <= 256
};
// The block of a workgroup; false where it has none.  (Three integer divisions here took 0.1 us of every launch.)
__host__ __device__ __forceinline__ bool tile_block(const TilePlan& p, int workgroup, int& colb, int& rowb, int& slice) {
  const int x = workgroup & 7, i = workgroup >> 3;
  if (p.rows_xcd) {
    const int y = x & ((1 << p.lg_per) - 1), c = (int)(((uint32_t)i * p.rows_inv) >> 20);
    slice = x >> p.lg_per;
    rowb = (y >> p.lg_colg) * p.rows_xcd + i - c * p.rows_xcd;
    colb = (y & ((1 << p.lg_colg) - 1)) * p.cols_xcd + c;
    return i < p.per_xcd && rowb < p.n_rowb && c < p.cols_xcd && colb < p.n_colb;
  }
  const int o = x * p.per_xcd + i;
  const int per_slice = p.n_colb * p.n_rowb;
  slice = o / per_slice;
  const int rem = o - slice * per_slice;
  colb = rem / p.n_rowb;
  rowb = rem - colb * p.n_rowb;
  return slice < p.n_slices && i < p.per_xcd;
}

// Column tile of slot j of column group cb (a group has TN slots).  SwiGLU: the first half of the slots from the gate matrix,
// the second half the same tiles of the up matrix.  QKV: slots j and j + TN/2 hold dims d and d + head_dim/2 of a head, the
// pairs that the rotary embedding turns.
template <int EPI, int TN>
__device__ __forceinline__ int slot_tile(int cb, int j, int hd) {
  if (EPI == EPI_PARTIAL || EPI == EPI_RESID) return cb * TN + j;
  const int p = cb * (TN / 2) + (j % (TN / 2));
  if (EPI == EPI_SWIGLU) return p;
  const int lg = __builtin_ctz(hd) - 5, head = p >> lg, i = p - (head << lg);      // (head sizes are powers of two)
  return (head << (lg + 1)) + i + (j >= TN / 2 ? 1 << lg : 0);
}

// What the QKV epilogue needs of a row, requested ahead of the contraction.
struct RowDest {
  int pos, blk;          // blk < 0: the row's key and value are not stored
};
__device__ __forceinline__ RowDest row_dest(const GemmArgs& g, int row) {
  RowDest d{0, -1};
  if (row < g.M) {
    d.pos = g.rows.pos[row];
    if (g.rows.active[row]) d.blk = g.kv.table[(g.rows.seq0 + row / g.rows.R) * g.kv.mbps + d.pos / g.kv.bt];
  }
  return d;
}

// 1 / r.m.s. of the rows of row tile mt for the epilogue's lanes (row = lane % 16), from the sums of squares that EPI_RESID left:
// each lane group sums a quarter of a row's.  In two steps: the loads go out ahead of the operands', the sum is taken while
// those travel.  Two forms: a sum per 16 columns (up to 64 rows, where a few workgroups read them), or one per workgroup or pair of
// tiles that made them, 16 bytes a lane: 56 scattered loads per row and workgroup cost gate / up of 1024 rows of width 896 2 us, of
// width 1536 9 us.
struct RowSums {
  const float* p;
  float x[16];
};
template <bool FINE>
__device__ __forceinline__ RowSums row_sums_load(const GemmArgs& g, int mt) {
  const int lane = threadIdx.x & 63, lg = lane >> 4, row = min(mt * 16 + (lane & 15), g.M - 1);
  RowSums r;
  if (FINE) {
    const int nt = g.rms_d >> 4;
    r.p = g.sumsq + (size_t)row * nt + lg;
#pragma unroll
    for (int u = 0; u < 16; ++u) r.x[u] = 4 * u + lg < nt ? r.p[4 * u] : 0.f;
  } else {
    r.p = g.sumsq + (size_t)row * ((g.sum_pieces + 15) & ~15) + 4 * lg;
#pragma unroll
    for (int u = 0; u < 4; ++u) {                          // (what lies between the last piece and the next multiple of 16 was never written)
      const f32x4 v = 16 * u < g.sum_pieces ? *(const f32x4*)(r.p + 16 * u) : f32x4{0, 0, 0, 0};
#pragma unroll
      for (int i = 0; i < 4; ++i) r.x[4 * u + i] = 16 * u + 4 * lg + i < g.sum_pieces ? v[i] : 0.f;
    }
  }
  return r;
}
template <bool FINE>
__device__ __forceinline__ float row_inv_rms(const GemmArgs& g, const RowSums& r) {
  const int lg = (threadIdx.x & 63) >> 4;
  float s = 0.f;
#pragma unroll
  for (int u = 0; u < 16; ++u) s += r.x[u];
  if (FINE) {
    const int nt = g.rms_d >> 4;
    for (int u0 = 16; 4 * u0 < nt; u0 += 8) {              // (d_model > 1024)
      float y[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) y[u] = 4 * (u0 + u) + lg < nt ? r.p[4 * (u0 + u)] : 0.f;
#pragma unroll
      for (int u = 0; u < 8; ++u) s += y[u];
    }
  } else {
    for (int u = 64; u < g.sum_pieces; u += 16)            // (more than 64 pieces: d_model > 2048)
#pragma unroll
      for (int i = 0; i < 4; ++i) s += u + 4 * lg + i < g.sum_pieces ? r.p[u + i] : 0.f;
  }
  return 1.0f / sqrtf(sum_over_groups(s) / (float)g.rms_d + g.rms_eps);
}

// What EPI_RESID's epilogue of a pair of tiles needs from memory besides the sums: the residual stream and the gain of the lane's
// features.  Requested ahead of the contraction, so that its latency is not one more link of the chain at the kernel's end (1024 rows
// of width 896 in tiles of 4 x 4 11.0 -> 10.7 us, 97 rows 5.5 -> 5.3).
struct ResidOperands {
  f32x4 h[2], gain[2];
};
template <int EPI>
__device__ __forceinline__ ResidOperands resid_operands(const GemmArgs& g, int t0, int t1, int row, int col) {
  ResidOperands e;
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int t = q ? t1 : t0, n = t * 16 + col;
    const bool ok = EPI == EPI_RESID && row < g.M && t < (g.N + 15) >> 4;
    e.h[q] = ok ? *(const f32x4*)(g.h + (size_t)row * g.N + n) : f32x4{0, 0, 0, 0};
    e.gain[q] = ok ? *(const f32x4*)(g.gain + n) : f32x4{0, 0, 0, 0};
  }
  return e;
}

// Epilogue of four consecutive features of one row: tile slot j < TN/2 (v0) and its partner j + TN/2 (v1); for partial
// outputs two independent tiles.  `col` = 4 (lane / 16).  EPI_RESID returns the lane's share of the row's sum of squares over them
// (where the pieces are not 16 columns: else they are written here).
template <int EPI>
__device__ __forceinline__ float tile_epilogue(const GemmArgs& g, int t0, int t1, int slice, int row, int col, f32x4 v0, f32x4 v1,
                                              const RowDest rd, const ResidOperands& e, float inv) {
  const int ntiles = (g.N + 15) >> 4;
  if (EPI == EPI_RESID) {                                  // (all lanes stay: the sums cross them)
    float sum = 0.f;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int t = q ? t1 : t0, n = t * 16 + col;
      const bool ok = row < g.M && t < ntiles;
      f32x4 v = q ? v1 : v0;
      float ss = 0.f;
      if (ok) {
        float* hp = g.h + (size_t)row * g.N + n;
        v += e.h[q];
        *(f32x4*)hp = v;
#pragma unroll
        for (int r = 0; r < 4; ++r) ss = fmaf(v[r], v[r], ss);
        const f32x4 y = v * e.gain[q];
        bf16_t* o = (bf16_t*)g.hg + split_index(row, n, g.N >> 5);
        *(uint2*)o = hi_pairs(y);
        *(uint2*)(o + 512) = lo_pairs(y);
      }
      if (g.sum_pieces) sum += ss;
      else {
        ss = sum_over_groups(ss);
        if (ok && col == 0) g.sumsq[(size_t)row * ntiles + t] = ss;
      }
    }
    return sum;
  }
  if (row >= g.M || t0 >= ntiles) return 0.f;
  if (EPI == EPI_PARTIAL) {
    float* o = g.out + (size_t)slice * g.out_split_stride + (size_t)row * g.ldo;
    const int n0 = t0 * 16 + col, n1 = t1 * 16 + col;
    if ((g.N & 3) == 0) {
      if (n0 < g.N) *(f32x4*)(o + n0) = v0;
      if (n1 < g.N) *(f32x4*)(o + n1) = v1;
    } else {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        if (n0 + r < g.N) o[n0 + r] = v0[r];
        if (n1 + r < g.N) o[n1 + r] = v1[r];
      }
    }
  } else if (EPI == EPI_SWIGLU) {
    f32x4 y;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float a = v0[r] * inv;
      y[r] = a / (1.0f + expf(-a)) * (v1[r] * inv);
    }
    bf16_t* o = (bf16_t*)g.act + split_index(row, t0 * 16 + col, g.act_split_kt);
    *(uint2*)o = hi_pairs(y);
    *(uint2*)(o + 512) = lo_pairs(y);
  } else {
    const int hd = g.kv.hd, half = hd >> 1, nq = g.nq, nkv = g.kv.nkv;
    const int n0 = t0 * 16 + col, head = n0 >> __builtin_ctz(hd), d = n0 & (hd - 1);
    v0 *= inv; v1 *= inv;                                  // (1 unless the operand is still to be normalised)
    if (g.bias) {
      const f32x4 b0 = *(const f32x4*)(g.bias + n0), b1 = *(const f32x4*)(g.bias + n0 + half);
#pragma unroll
      for (int r = 0; r < 4; ++r) { v0[r] += b0[r]; v1[r] += b1[r]; }
    }
    if (head < nq + nkv) {
      const f32x4* cs = (const f32x4*)(g.rope + (size_t)rd.pos * half + d);
      const f32x4 c0 = cs[0], c1 = cs[1];
      const float c[4] = {c0[0], c0[2], c1[0], c1[2]}, s[4] = {c0[1], c0[3], c1[1], c1[3]};
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float r0 = v0[r] * c[r] - v1[r] * s[r], r1 = v1[r] * c[r] + v0[r] * s[r];
        v0[r] = r0; v1[r] = r1;
      }
    }
    if (head < nq) {
      float* qo = g.q + (size_t)row * nq * hd + head * hd + d;
      *(f32x4*)qo = v0;
      *(f32x4*)(qo + half) = v1;
    } else if (rd.blk >= 0) {
      const int which = head < nq + nkv ? 0 : 1, kvh = head - nq - which * nkv;
      bf16_t* base = (bf16_t*)g.kv.pool + kv_offset(g.kv, g.layer, which, rd.blk, kvh, 0);
      const int tok = rd.pos % g.kv.bt;
      if (which == 0) {
        *(uint2*)(base + tok * hd + d) = make_uint2(f2_to_bf16x2(v0[0], v0[1]), f2_to_bf16x2(v0[2], v0[3]));
        *(uint2*)(base + tok * hd + d + half) = make_uint2(f2_to_bf16x2(v1[0], v1[1]), f2_to_bf16x2(v1[2], v1[3]));
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          base[(d + r) * g.kv.bt + tok] = f_to_bf16(v0[r]);
          base[(d + r + half) * g.kv.bt + tok] = f_to_bf16(v1[r]);
        }
      }
    }
  }
  return 0.f;
}
// The piece of a row's sum of squares that this wave has made (all lanes call it).
__device__ __forceinline__ void store_row_sum(const GemmArgs& g, int row, int piece, int pieces, float sum) {
  sum = sum_over_groups(sum);
  if (row < g.M && (threadIdx.x & 63) < 16) g.sumsq[(size_t)row * ((pieces + 15) & ~15) + piece] = sum;
}

// The order of a k-tile's instructions: a matrix instruction or two, then a request to memory or a read of the next k-tile's fragments, and so
// on.  (Left alone, the compiler puts the reads behind nearly all of the matrix instructions, right ahead of the wait for them.)
template <int MFMA, int VMEM, int READS>
__device__ __forceinline__ void sched_interleave() {
  constexpr int N = VMEM + READS;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    if (MFMA > i) __builtin_amdgcn_sched_group_barrier(0x008, MFMA >= 2 * N ? 2 : 1, 0);
    if (i < VMEM) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
    else __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
  }
  __builtin_amdgcn_sched_group_barrier(0x008, MFMA, 0);
}

// ------------------------------------------------------------------------------------------ large tiles
// A workgroup of W waves owns W * TM row tiles x TN column-tile slots over a k range; wave w owns row tiles w TM .. and
// all the column tiles.  It loads its own activation fragments into registers, UA k-tiles ahead; the weight fragments
// that all waves need go from memory to LDS with direct loads (16 bytes per lane, a fragment per instruction, no
// registers), NBUF k-tiles ahead, and from there into registers one k-tile ahead, beside the matrix instructions.  One barrier per k-tile: it is
// passed when every wave has read k-tile k, whose buffer the next request then overwrites, and every wave's share of k-tile k + 1 has arrived.
// What bounds it with many rows, by clock stamps: gate / up of 1024 rows of the 0.5B shape (16 x 10) 33.6 us, of which the loop is 20.8.  A k-tile takes 1460 cycles
// where its matrix instructions need 1280, at 1.96 GHz; the same instructions from registers alone settle at 2.06 GHz, with the reads from LDS at
// 1.94 (28 k-tiles of them by themselves run at 2.27).  3.5 us are first operands, 3.3 the epilogue, 5 the launch and the drain.  With few rows it is latency.  Ahead of the waits, the order
// and the reads above, in a forward: 35.8 -> 34.5 us; 8 x 7 of down 21.7 (k_gemm_block) -> 20.8; output projection 10.6 (k_gemm_kwave) -> 10.0.
template <int EPI, int TM, int TN, int W, int NBUF, int UA, int MINB>
__global__ void __launch_bounds__(W * 64, MINB) k_gemm_tile(GemmArgs g, TilePlan p) {
  constexpr int LW = (TN + W - 1) / W;                     // weight fragments a wave requests per k-tile
  static_assert(UA >= NBUF - 1 && UA % 2 == 0 && (EPI == EPI_PARTIAL || EPI == EPI_RESID || TN % 2 == 0), "the first waits rely on it");
  __shared__ u32x4 stage[NBUF][TN][64];
  int colb, rowb, slice;
  if (!tile_block(p, (int)blockIdx.x, colb, rowb, slice)) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int KT = g.K >> 5, ntiles = (g.N + 15) >> 4, last_mt = (g.M - 1) >> 4;
  const int kb = slice * p.slice_kt, nk = min(KT, kb + p.slice_kt) - kb;
  const int hd = g.kv.hd;
  rsrc_t ws[LW];
  int wdst[LW];
#pragma unroll
  for (int q = 0; q < LW; ++q) {                           // (the last ones repeat an earlier slot where TN is not a multiple of W)
    const int j = (q * W + wave) % TN;
    const int t = slot_tile<EPI, TN>(colb, j, hd);
    const void* w = (EPI == EPI_SWIGLU && j >= TN / 2) ? g.W1 : g.W0;
    ws[q] = load_rsrc((const char*)w + ((size_t)(t < ntiles ? t : 0) * KT + kb) * 1024);
    wdst[q] = j;
  }
  auto request_w = [&](int k, int buf) {
#pragma unroll
    for (int q = 0; q < LW; ++q)
      load_to_lds(ws[q], &stage[buf][wdst[q]][0], lane * 16, k * 1024);
  };
  const u32x4* ap[TM];
#pragma unroll
  for (int i = 0; i < TM; ++i) ap[i] = (const u32x4*)g.A + ((size_t)min((rowb * W + wave) * TM + i, last_mt) * KT + kb) * 128 + lane;
  u32x4 a[UA][TM][2];
  auto request_a = [&](int u, int k) {
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      a[u][i][0] = ap[i][(size_t)k * 128];
      a[u][i][1] = ap[i][(size_t)k * 128 + 64];
    }
  };
  constexpr int PAIRS = (TN + 1) / 2;                      // (an odd last slot is alone)
  ResidOperands ro[TM][PAIRS];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < PAIRS; ++j)
      ro[i][j] = resid_operands<EPI>(g, slot_tile<EPI, TN>(colb, j < TN / 2 ? j : TN - 1, hd), j < TN / 2 ? slot_tile<EPI, TN>(colb, j + TN / 2, hd) : 0x7FFFFF,
                                     ((rowb * W + wave) * TM + i) * 16 + (lane & 15), 4 * (lane >> 4));
  RowDest rd[TM];
#pragma unroll
  for (int i = 0; i < TM; ++i) rd[i] = EPI == EPI_QKV ? row_dest(g, ((rowb * W + wave) * TM + i) * 16 + (lane & 15)) : RowDest{0, -1};
  const bool scaled = (EPI == EPI_SWIGLU || EPI == EPI_QKV) && g.rms_d > 0;
  RowSums rs[TM];
  if (scaled)
#pragma unroll
    for (int i = 0; i < TM; ++i) rs[i] = row_sums_load<false>(g, (rowb * W + wave) * TM + i);
#pragma unroll
  for (int b = 0; b < NBUF; ++b) request_w(min(b, nk - 1), b);
  asm volatile("" ::: "memory");                           // the first waits count the activations' requests as the later ones
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int u = 0; u < UA; ++u) {
    request_a(u, min(u, nk - 1));
    __builtin_amdgcn_sched_barrier(0);                     // (in this order: else the loop's first wait for a[0], which the compiler places, waits for all of them)
  }
  float inv[TM];
#pragma unroll
  for (int i = 0; i < TM; ++i) inv[i] = scaled ? row_inv_rms<false>(g, rs[i]) : 1.0f;
  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0, 0, 0, 0};
  u32x4 w[2][TN];
  auto fetch = [&](int s, int b) {
#pragma unroll
    for (int j = 0; j < TN; ++j) w[s][j] = stage[b][j][lane];
  };
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NBUF - 1) * LW + UA * 2 * TM) : "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  fetch(0, 0);
  int buf = 0;                                             // buffer of k-tile k
  auto one = [&](auto tail, int u, int k) {
    // k-tile k + 1's weights have arrived when at most this wave's later requests are outstanding.  (`tail`: bodies behind the main loop so far.
    // What those load of the activations is not used, and the compiler leaves it out.)
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((NBUF - 2) * LW + (NBUF - 1 > decltype(tail)::value ? NBUF - 1 - decltype(tail)::value : 0) * 2 * TM) : "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    request_w(min(k + NBUF, nk - 1), buf);
    buf = buf + 1 == NBUF ? 0 : buf + 1;
    fetch((u & 1) ^ 1, buf);
    asm volatile("" ::: "memory");
    const u32x4* const wk = w[u & 1];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const bf16x8 hi = __builtin_bit_cast(bf16x8, a[u][i][0]), lo = __builtin_bit_cast(bf16x8, a[u][i][1]);
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wk[j]), lo, acc[i][j], 0, 0, 0);
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wk[j]), hi, acc[i][j], 0, 0, 0);
    }
    sched_interleave<2 * TM * TN, LW, TN>();
    __builtin_amdgcn_sched_barrier(0);
    request_a(u, min(k + UA, nk - 1));
    __builtin_amdgcn_sched_barrier(0);
  };
  const int kfull = (nk / UA) * UA;
  for (int k0 = 0; k0 < kfull; k0 += UA) {
#pragma unroll
    for (int u = 0; u < UA; ++u) one(std::integral_constant<int, 0>(), u, k0 + u);
  }
  for_each_index([&](auto u) { if (kfull + u < nk) one(u, u, kfull + u); }, std::make_integer_sequence<int, UA - 1>());      // (uniform over the workgroup)
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");         // the requests past the end
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int row = ((rowb * W + wave) * TM + i) * 16 + (lane & 15);
    float sum = 0.f;
#pragma unroll
    for (int j = 0; j < TN / 2; ++j)
      sum += tile_epilogue<EPI>(g, slot_tile<EPI, TN>(colb, j, hd), slot_tile<EPI, TN>(colb, j + TN / 2, hd), slice, row, 4 * (lane >> 4), acc[i][j],
                         acc[i][j + TN / 2], rd[i], ro[i][j], inv[i]);
    if (TN % 2)
      sum += tile_epilogue<EPI>(g, slot_tile<EPI, TN>(colb, TN - 1, hd), 0x7FFFFF, slice, row, 4 * (lane >> 4), acc[i][TN - 1], acc[i][TN - 1],
                              rd[i], ro[i][PAIRS - 1], inv[i]);
    if (EPI == EPI_RESID && g.sum_pieces) store_row_sum(g, row, colb, p.n_colb, sum);
  }
}

// ------------------------------------------------------------------------------------------ some rows
// The same where a workgroup's tile is the whole work of its compute unit, or nearly, and the latency of a k-tile counts (65 to 500 rows): both
// operands go from memory to LDS with direct loads, NBUF k-tiles ahead, and a wave (WR x WC of them, each TM row tiles x TN
// slots) reads the fragments of k-tile k + 1 into registers beside the matrix instructions of k-tile k.  No load in flight has a register,
// so the only waits are the counted ones.  One barrier per k-tile: it is passed when every wave has read k-tile k, whose buffer the next
// request then overwrites, and every wave's share of k-tile k + 1 has arrived.  Order of an element's sum as in k_gemm_tile.
// What bounds it up to about 250 rows is the intake of a compute unit, 60 bytes a nanosecond of activations that every column block
// reads again and of weights from HBM, whatever the depth (3 to 11 k-tiles in flight: the same): gate / up of 97 rows in 4 x 6 11.8 us.  With more rows
// its reads of LDS weigh: (2 TM + TN) KB per wave and k-tile against 8 TM TN cycles of matrix instructions, at 128 bytes a cycle, so its
// large tiles have waves of 2 x 6 and 2 x 8.
template <int EPI, int RT, int CT, int WR, int WC, int NBUF>
__global__ void __launch_bounds__(WR * WC * 64) k_gemm_block(GemmArgs g, TilePlan p) {
  constexpr int W = WR * WC, TM = RT / WR, TN = CT / WC;
  constexpr int F = 2 * RT + CT, LPW = (F + W - 1) / W;    // fragments of a k-tile (hi and lo of the rows, then the weights); of them, a wave requests
  static_assert(EPI != EPI_RESID && RT % WR == 0 && CT % WC == 0 && (EPI == EPI_PARTIAL || TN % 2 == 0), "");
  extern __shared__ u32x4 lds[];                           // [NBUF][F][64]
  int colb, rowb, slice;
  if (!tile_block(p, (int)blockIdx.x, colb, rowb, slice)) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), wr = wave / WC, wc = wave - wr * WC;
  const int KT = g.K >> 5, ntiles = (g.N + 15) >> 4, last_mt = (g.M - 1) >> 4;
  const int kb = slice * p.slice_kt, nk = min(KT, kb + p.slice_kt) - kb, hd = g.kv.hd;
  rsrc_t src[LPW];
  int step[LPW], dst[LPW];
#pragma unroll
  for (int q = 0; q < LPW; ++q) {                          // (the last ones repeat earlier fragments where F is not a multiple of W)
    const int f = (q * W + wave) % F;
    dst[q] = f;
    if (f < 2 * RT) {
      src[q] = load_rsrc((const char*)g.A + ((size_t)min(rowb * RT + f / 2, last_mt) * KT + kb) * 2048 + (f & 1) * 1024);
      step[q] = 2048;
    } else {
      const int j = f - 2 * RT, t = slot_tile<EPI, CT>(colb, j, hd);
      src[q] = load_rsrc((const char*)(EPI == EPI_SWIGLU && j >= CT / 2 ? g.W1 : g.W0) + ((size_t)(t < ntiles ? t : 0) * KT + kb) * 1024);
      step[q] = 1024;
    }
  }
  auto request = [&](int k, int buf) {
#pragma unroll
    for (int q = 0; q < LPW; ++q)
      load_to_lds(src[q], &lds[(buf * F + dst[q]) * 64], lane * 16, k * step[q]);
  };
  // slot of the workgroup's CT that is this wave's j-th (paired tiles: the pairs of the same columns)
  auto slot = [&](int j) {
    return EPI == EPI_PARTIAL ? wc * TN + j : j < TN / 2 ? wc * (TN / 2) + j : CT / 2 + wc * (TN / 2) + j - TN / 2;
  };
  auto tile = [&](int j) { return j < TN ? slot_tile<EPI, CT>(colb, slot(j), hd) : 0x7FFFFF; };
  auto row_of = [&](int i) { return ((rowb * WR + wr) * TM + i) * 16 + (lane & 15); };
  constexpr int PAIRS = (TN + 1) / 2, HALF = TN / 2 + TN % 2;       // (an odd slot is alone)
  RowDest rd[TM];
#pragma unroll
  for (int i = 0; i < TM; ++i) rd[i] = EPI == EPI_QKV ? row_dest(g, row_of(i)) : RowDest{0, -1};
  const bool scaled = (EPI == EPI_SWIGLU || EPI == EPI_QKV) && g.rms_d > 0;
  RowSums rs[TM];
  if (scaled)
#pragma unroll
    for (int i = 0; i < TM; ++i) rs[i] = row_sums_load<false>(g, (rowb * WR + wr) * TM + i);
#pragma unroll
  for (int b = 0; b < NBUF; ++b) request(min(b, nk - 1), b);
  float inv[TM];
#pragma unroll
  for (int i = 0; i < TM; ++i) inv[i] = scaled ? row_inv_rms<false>(g, rs[i]) : 1.0f;
  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0, 0, 0, 0};
  u32x4 a[2][TM][2], w[2][TN];
  auto fetch = [&](int s, int buf) {
    const u32x4* b = lds + buf * F * 64 + lane;
#pragma unroll
    for (int j = 0; j < TN; ++j) w[s][j] = b[(2 * RT + slot(j)) * 64];
#pragma unroll
    for (int i = 0; i < TM; ++i) { a[s][i][1] = b[(2 * (wr * TM + i) + 1) * 64]; a[s][i][0] = b[2 * (wr * TM + i) * 64]; }
  };
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NBUF - 1) * LPW) : "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  fetch(0, 0);
  int buf = 0;                                             // of k-tile k
  auto one = [&](int s, int k) {
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((NBUF - 2) * LPW) : "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    request(min(k + NBUF, nk - 1), buf);
    buf = buf + 1 == NBUF ? 0 : buf + 1;
    fetch(s ^ 1, buf);                                     // (behind the last k-tile: a repeated one, not used)
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const bf16x8 hi = __builtin_bit_cast(bf16x8, a[s][i][0]), lo = __builtin_bit_cast(bf16x8, a[s][i][1]);
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w[s][j]), lo, acc[i][j], 0, 0, 0);
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w[s][j]), hi, acc[i][j], 0, 0, 0);
    }
    sched_interleave<2 * TM * TN, LPW, 2 * TM + TN>();
    __builtin_amdgcn_sched_barrier(0);
  };
  int k = 0;
  for (; k + 2 <= nk; k += 2) { one(0, k); one(1, k + 1); }
  if (k < nk) one(0, k);                                   // (uniform over the workgroup)
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");       // the requests past the end
  const ResidOperands none{};
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < PAIRS; ++j)
      tile_epilogue<EPI>(g, tile(j), tile(j + HALF), slice, row_of(i), 4 * (lane >> 4), acc[i][j], acc[i][j + HALF < TN ? j + HALF : j], rd[i], none, inv[i]);
}

// ------------------------------------------------------------------------------------------ few rows
// A workgroup of W waves owns TM row tiles x TN column-tile slots over a k range; its waves take the k-tiles in turn
// (wave w: k-tiles w, w + W, ..) straight from memory into registers, U of them in flight, and meet once in LDS.  No
// barrier before that.  Order of an element's sum: a wave's k-tiles ascending, lo before hi, then the waves ascending.
template <int EPI, int TM, int TN, int W, int U>
__global__ void __launch_bounds__(W * 64, 1) k_gemm_kwave(GemmArgs g, TilePlan p) {
  constexpr int RPR = (128 / (W * TN)) < 1 ? 1 : (128 / (W * TN)) > TM ? TM : 128 / (W * TN);     // row tiles per round of the reduction
  __shared__ f32x4 red[W][RPR * TN][64];
  __shared__ float inv_rms[TM][16];
  int colb, rowb, slice;
  if (!tile_block(p, (int)blockIdx.x, colb, rowb, slice)) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int KT = g.K >> 5, ntiles = (g.N + 15) >> 4, last_mt = (g.M - 1) >> 4;
  const int kb = slice * p.slice_kt, ke = min(KT, kb + p.slice_kt);
  const int hd = g.kv.hd, nw = (ke - kb - wave + W - 1) / W;                                       // k-tiles of this wave
  const u32x4 *ap[TM], *wp[TN];
#pragma unroll
  for (int i = 0; i < TM; ++i) ap[i] = (const u32x4*)g.A + (size_t)min(rowb * TM + i, last_mt) * KT * 128 + lane;
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int t = slot_tile<EPI, TN>(colb, j, hd);
    wp[j] = (const u32x4*)((EPI == EPI_SWIGLU && j >= TN / 2) ? g.W1 : g.W0) + (size_t)(t < ntiles ? t : 0) * KT * 64 + lane;
  }
  u32x4 w[U][TN], a[U][TM][2];
  auto request = [&](int u, int i) {                       // slot u <- the wave's i-th k-tile
    const int kt = min(kb + wave + i * W, KT - 1);
#pragma unroll
    for (int j = 0; j < TN; ++j) w[u][j] = __builtin_nontemporal_load(wp[j] + (size_t)kt * 64);
#pragma unroll
    for (int m = 0; m < TM; ++m) {
      a[u][m][0] = ap[m][(size_t)kt * 128];
      a[u][m][1] = ap[m][(size_t)kt * 128 + 64];
    }
  };
  // the waves' tiles meet in LDS, RPR row tiles at a time; unit (row tile, slot pair) u is summed and written by wave u mod W
  constexpr int PAIRS = (TN + 1) / 2;
  static_assert(EPI != EPI_RESID || (RPR == TM && TM * PAIRS <= W), "one unit per wave: its operands are requested here");
  const int my_i = wave / PAIRS, my_j = wave - my_i * PAIRS, my_j1 = min(my_j + TN / 2 + TN % 2, TN - 1);
  ResidOperands ro;
  if (EPI == EPI_RESID && my_i < TM)
    ro = resid_operands<EPI>(g, slot_tile<EPI, TN>(colb, my_j, hd), my_j1 == my_j ? 0x7FFFFF : slot_tile<EPI, TN>(colb, my_j1, hd),
                             (rowb * TM + my_i) * 16 + (lane & 15), 4 * (lane >> 4));
  const bool scaled = EPI == EPI_SWIGLU && g.rms_d > 0 && wave < TM;
  RowSums rs;
  if (scaled) rs = row_sums_load<true>(g, rowb * TM + wave);
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (u < nw) request(u, u);
  if (scaled) {                                            // (read in the epilogue, after a barrier)
    const float v = row_inv_rms<true>(g, rs);
    if (lane < 16) inv_rms[wave][lane] = v;
  }
  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0, 0, 0, 0};
  auto contract = [&](int u) {
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const bf16x8 hi = __builtin_bit_cast(bf16x8, a[u][i][0]), lo = __builtin_bit_cast(bf16x8, a[u][i][1]);
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w[u][j]), lo, acc[i][j], 0, 0, 0);
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w[u][j]), hi, acc[i][j], 0, 0, 0);
    }
  };
  const int kfull = (nw / U) * U;
  for (int k0 = 0; k0 < kfull; k0 += U) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      contract(u);
      __builtin_amdgcn_sched_barrier(0);
      if (k0 + u + U < nw) request(u, k0 + u + U);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int u = 0; u < U - 1; ++u)
    if (kfull + u < nw) contract(u);
#pragma unroll
  for (int i0 = 0; i0 < TM; i0 += RPR) {
    RowDest rd[(RPR * PAIRS + W - 1) / W];
#pragma unroll
    for (int q = 0; q < (RPR * PAIRS + W - 1) / W; ++q) {
      const int u = q * W + wave;
      rd[q] = EPI == EPI_QKV ? row_dest(g, (rowb * TM + i0 + u / PAIRS) * 16 + (lane & 15)) : RowDest{0, -1};
    }
    if (i0) __syncthreads();
#pragma unroll
    for (int i = 0; i < RPR; ++i)
      if (i0 + i < TM)
#pragma unroll
        for (int j = 0; j < TN; ++j) red[wave][i * TN + j][lane] = acc[i0 + i][j];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < (RPR * PAIRS + W - 1) / W; ++q) {
      const int u = q * W + wave, i = u / PAIRS, j = u - i * PAIRS, j1 = min(j + TN / 2 + TN % 2, TN - 1);
      if (i < RPR && i0 + i < TM) {
        f32x4 v0 = red[0][i * TN + j][lane], v1 = red[0][i * TN + j1][lane];
#pragma unroll
        for (int x = 1; x < W; ++x) { v0 += red[x][i * TN + j][lane]; v1 += red[x][i * TN + j1][lane]; }
        const float sum = tile_epilogue<EPI>(g, slot_tile<EPI, TN>(colb, j, hd), j1 == j ? 0x7FFFFF : slot_tile<EPI, TN>(colb, j1, hd), slice,
                           (rowb * TM + i0 + i) * 16 + (lane & 15), 4 * (lane >> 4), v0, v1, rd[q], ro,
                           EPI == EPI_SWIGLU && g.rms_d > 0 ? inv_rms[i0 + i][lane & 15] : 1.0f);
        if (EPI == EPI_RESID && g.sum_pieces) store_row_sum(g, (rowb * TM + i) * 16 + (lane & 15), colb * PAIRS + j, p.n_colb * PAIRS, sum);
      }
    }
  }
}

}  // namespace ssd
