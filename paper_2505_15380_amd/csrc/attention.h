// Multi-query decode attention over the paged cache (Eq. 4: the K+1 rows of a verification attend to the
// whole prefix and causally to each other), as launches of its own:
//   k_attn_mfma   bf16, 16-token blocks, head size 64 or 128: the matrix cores on hi + lo halves (k_attn_combine_parts merges)
//   k_attn_f32    fp32, 16-token blocks: the fp32 matrix instructions (k_attn_combine merges)
//   k_attn_chunk  every other block size, head size 32 in bf16, and SSD_ATTN=valu: vector units (k_attn_combine merges)
// Parts and chunks are cut at absolute positions and merged in ascending order.  Those of the fp32 and of the chunk kernels
// have one size, so what a row combines - and therefore its bits - does not depend on how many rows are verified
// together; the size of k_attn_mfma's parts follows from the launch's shape.
#pragma once
#include <type_traits>

#include "common.h"

namespace ssd {

struct AttnArgs {
  const float* q;       // [M][nq*hd] rotated queries
  KvView kv;
  Rows rows;
  int layer, nq;
  float scale;
  float* o_part;        // [M][nq][NC][hd]
  float* ml_part;       // [M][nq][NC][2]
  int NC;               // chunk capacity of the partial buffers
  void* out;            // [M][nq*hd] (combine)
  int split_kt;         // > 0: `out` is written as split rows (common.h) with this many k-tiles per row (nq*hd / 32)
  int nparts, part_keys;      // k_attn_mfma, k_attn_f32: grid.x = nparts x (groups of) row tiles; keys per part, a multiple of 64
  int n_tg;                   // k_attn_mfma: groups of row tiles
  int nchunks;                // k_attn_f32: chunks of the longest sequence
};

// Work item = (chunk of 64 key positions, kv head, sequence).  The workgroup stages the chunk's keys and values in LDS once
// and serves every query row that shares them: R rows of the sequence x the G query heads of the group.  Each query row gets a
// partial (max, sum, weighted values) per chunk.
template <int HD, typename KVT>
__global__ void __launch_bounds__(BLOCK) k_attn_chunk(AttnArgs a) {
  __shared__ float Ks[ATT_CHUNK][HD + 1];
  __shared__ float Vs[ATT_CHUNK][HD];
  __shared__ float Qs[4][HD];
  __shared__ float Ps[4][ATT_CHUNK];
  const int chunk = blockIdx.x, kvh = blockIdx.y, brel = blockIdx.z;
  const int seq = a.rows.seq0 + brel;
  const int R = a.rows.R, G = a.nq / a.kv.nkv;
  const int m_first = brel * R, m_last = m_first + R - 1;
  const int cstart = chunk * ATT_CHUNK;
  const int pos_max = a.rows.pos[m_last];
  if (cstart > pos_max) return;                          // no row of this sequence reaches the chunk
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;

  // stage keys / values of positions cstart .. cstart+63 (zero where beyond pos_max or unmapped)
  typedef typename KVT::T kv_t;
  const kv_t* pool = (const kv_t*)a.kv.pool;
  for (int i = tid; i < ATT_CHUNK * HD; i += BLOCK) {
    const int c = i / HD, d = i - c * HD;
    const int p = cstart + c;
    float kx = 0.f, vx = 0.f;
    if (p <= pos_max) {
      const int blk = a.kv.table[seq * a.kv.mbps + p / a.kv.bt];
      if (blk >= 0) {
        kx = KVT::ld(pool + kv_offset(a.kv, a.layer, 0, blk, kvh, p % a.kv.bt) + d);
        vx = KVT::ld(pool + kv_offset(a.kv, a.layer, 1, blk, kvh, 0) + d * a.kv.bt + p % a.kv.bt);
      }
    }
    Ks[c][d] = kx;
    Vs[c][d] = vx;
  }
  __syncthreads();

  const int nrows = R * G;
  for (int r = wave; r < nrows; r += 4) {
    const int j = r / G, gq = r - j * G;
    const int m = m_first + j, hq = kvh * G + gq;
    const int pos = a.rows.pos[m];
    const float* qrow = a.q + (size_t)m * a.nq * HD + hq * HD;
    for (int d = lane; d < HD; d += WAVE) Qs[wave][d] = qrow[d];
    __builtin_amdgcn_wave_barrier();
    // score of key `lane`
    float s = 0.f;
#pragma unroll 8
    for (int d = 0; d < HD; ++d) s = fmaf(Qs[wave][d], Ks[lane][d], s);
    const bool valid = (cstart + lane) <= pos;
    s = valid ? s * a.scale : -INFINITY;
    const float mx = wave_max(s);
    const size_t pidx = ((size_t)m * a.nq + hq) * a.NC + chunk;
    float* op = a.o_part + pidx * HD;
    if (mx == -INFINITY) {                               // the row sees nothing of this chunk
      if (lane == 0) { a.ml_part[pidx * 2] = -INFINITY; a.ml_part[pidx * 2 + 1] = 0.f; }
      for (int d = lane; d < HD; d += WAVE) op[d] = 0.f;
      __builtin_amdgcn_wave_barrier();
      continue;
    }
    const float p = valid ? expf(s - mx) : 0.f;
    const float l = wave_sum(p);
    Ps[wave][lane] = p;
    __builtin_amdgcn_wave_barrier();
    for (int d = lane; d < HD; d += WAVE) {
      float o = 0.f;
#pragma unroll 8
      for (int c = 0; c < ATT_CHUNK; ++c) o = fmaf(Ps[wave][c], Vs[c][d], o);
      op[d] = o;
    }
    if (lane == 0) { a.ml_part[pidx * 2] = mx; a.ml_part[pidx * 2 + 1] = l; }
    __builtin_amdgcn_wave_barrier();
  }
}

// One wave per (row, query head): merge the row's partials - of chunks, or of k_attn_f32's parts, which leaves nothing to do
// for a row of one part - in ascending order.
template <int HD, typename AT>
__global__ void __launch_bounds__(WAVE) k_attn_combine(AttnArgs a) {
  const int m = blockIdx.x / a.nq, hq = blockIdx.x - m * a.nq;
  const int lane = threadIdx.x;
  const int nc = a.rows.pos[m] / a.part_keys + 1;
  if (a.part_keys > ATT_CHUNK && nc == 1) return;
  const size_t base = ((size_t)m * a.nq + hq) * a.NC;
  float mx = -INFINITY;
  for (int c = 0; c < nc; ++c) mx = fmaxf(mx, a.ml_part[(base + c) * 2]);
  float l = 0.f;
  float o[(HD + WAVE - 1) / WAVE];
#pragma unroll
  for (int i = 0; i < (HD + WAVE - 1) / WAVE; ++i) o[i] = 0.f;
  for (int c = 0; c < nc; ++c) {
    const float mc = a.ml_part[(base + c) * 2];
    if (mc == -INFINITY) continue;
    const float w = expf(mc - mx);
    l = fmaf(a.ml_part[(base + c) * 2 + 1], w, l);
#pragma unroll
    for (int i = 0; i < (HD + WAVE - 1) / WAVE; ++i) {
      const int d = lane + i * WAVE;
      if (d < HD) o[i] = fmaf(a.o_part[(base + c) * HD + d], w, o[i]);
    }
  }
  typename AT::T* out = (typename AT::T*)a.out + (size_t)m * a.nq * HD + hq * HD;
#pragma unroll
  for (int i = 0; i < (HD + WAVE - 1) / WAVE; ++i) {
    const int d = lane + i * WAVE;
    if (d < HD) {
      if (a.split_kt > 0) st_split_value((bf16_t*)a.out, a.split_kt, m, hq * HD + d, o[i] / l);
      else AT::st(out + d, o[i] / l);
    }
  }
}

// The same for fp32 caches with 16-token blocks, on v_mfma_f32_16x16x4_f32 (full fp32 products and sums).  A workgroup takes 16 of the
// query rows that share a kv head of a sequence, and a part of the keys: two 64-key chunks per wave, cut at absolute positions.
// Its waves walk the part's chunks w, w + W with a running (max, sum, weighted values) per row and meet in LDS.  A row of one part
// (1024 positions; head size 128: 512) is finished there, the parts of a longer one are merged by k_attn_combine: a row's order
// of sums depends on its position alone, whatever the launch.  (The chunk kernels above for long sequences in small batches, this
// one for the rest, would give it two; five rows at 960 / 2048 / 8000 positions: 23 / 27 / 29 us with head size 64 where they
// take 23 / 39 / 73, 33 / 35 / 45 with head size 128: 52 / 55 / 115.  With values and keys requested together, 64: 23 / 26 / 28,
// and four heads of size 32 14.7 / 18.2 / 20.3 where they were 17.6 / 21.0 / 23.6; 128: no difference.)  Scores and outputs are computed
// transposed: a lane holds one row's scores of the keys 4 kg .. 4 kg + 3 of a tile, which is what the product with the
// values wants from it, and both operands come from the cache as 16 bytes per lane (dims of a key, tokens of a dim).
// A chain of launch, block table, cache, merge bounds it: 6.1 us at five rows and 68 cached positions, where the two kernels
// above take 7.2 + 3.0 (a vector-unit version of this kernel took 7.9: twice the instructions, fetched cold on every launch).
template <int HD>
constexpr int att_f32_waves() { return HD <= 64 ? 8 : 4; }
template <int HD>
constexpr int att_f32_part() { return 2 * att_f32_waves<HD>(); }      // chunks of a part

template <int HD>
__global__ void __launch_bounds__(att_f32_waves<HD>() * WAVE) k_attn_f32(AttnArgs a) {
  constexpr int W = att_f32_waves<HD>(), PC = att_f32_part<HD>(), DT = HD / 16;
  __shared__ float po[W][16][HD + 4];
  __shared__ float pm[W][16], pl[W][16];
  const int kvh = blockIdx.y, brel = blockIdx.z, seq = a.rows.seq0 + brel;
  const int part = blockIdx.x % a.nparts, r0 = blockIdx.x / a.nparts * 16, c0 = part * PC;
  const int G = a.nq / a.kv.nkv, nrows = a.rows.R * G, m_first = brel * a.rows.R;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int li = lane & 15, kg = lane >> 4;
  const float* pool = (const float*)a.kv.pool;
  auto q_of = [&](int r, int& m) {                         // query row r of the group: its row of the forward and its values
    const int j = r / G;
    m = m_first + j;
    return ((size_t)m * a.nq + kvh * G + r - j * G) * HD;
  };
  int m;
  const f32x4* qp = (const f32x4*)(a.q + q_of(min(r0 + li, nrows - 1), m)) + kg;
  const int pos = a.rows.pos[m], pos_max = a.rows.pos[m_first + a.rows.R - 1];
  if (c0 * ATT_CHUNK > pos_max) return;                    // no row of the sequence reaches the part
  f32x4 q[DT];
#pragma unroll
  for (int s = 0; s < DT; ++s) q[s] = qp[s * 4];
  f32x4 o[DT];
#pragma unroll
  for (int s = 0; s < DT; ++s) o[s] = f32x4{0, 0, 0, 0};
  float mrow = -INFINITY, lrow = 0.f;
  const int c_end = min(c0 + PC, a.nchunks);
  for (int c = c0 + wave; c < c_end; c += W) {
    const int p0 = c * ATT_CHUNK;
    const int32_t* tab = a.kv.table + (size_t)seq * a.kv.mbps;
    f32x4 k[4][DT];
    int blk[4];                                            // a tile of 16 keys is a block
#pragma unroll
    for (int t = 0; t < 4; ++t) blk[t] = tab[min(c * 4 + t, a.kv.mbps - 1)];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const f32x4* kp = (const f32x4*)(pool + kv_offset(a.kv, a.layer, 0, max(blk[t], 0), kvh, li)) + kg;
#pragma unroll
      for (int s = 0; s < DT; ++s) k[t][s] = kp[s * 4];
    }
    f32x4 v[DT][4];                                        // (requested with the keys: their latency is then that of one load, not of two)
#pragma unroll
    for (int s = 0; s < DT; ++s)
#pragma unroll
      for (int t = 0; t < 4; ++t)
        v[s][t] = *(const f32x4*)(pool + kv_offset(a.kv, a.layer, 1, max(blk[t], 0), kvh, 0) + (s * 16 + li) * 16 + kg * 4);
    if (p0 > pos_max) break;
    f32x4 w[4];
    float mx = mrow;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      w[t] = f32x4{0, 0, 0, 0};
#pragma unroll
      for (int s = 0; s < DT; ++s)
#pragma unroll
        for (int e = 0; e < 4; ++e) w[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(k[t][s][e], q[s][e], w[t], 0, 0, 0);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        w[t][e] = p0 + t * 16 + kg * 4 + e <= pos ? (blk[t] >= 0 ? w[t][e] * a.scale : 0.f) : -INFINITY;
        mx = fmaxf(mx, w[t][e]);
      }
    }
    mx = fmaxf(mx, __shfl_xor(mx, 16, WAVE));
    mx = fmaxf(mx, __shfl_xor(mx, 32, WAVE));
    const float base = mx == -INFINITY ? 0.f : mx;         // (no key of the chunk is the row's: all weights are 0)
    const float keep = expf(mrow - base);
    float sum = 0.f;
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) { w[t][e] = expf(w[t][e] - base); sum += w[t][e]; }
    sum += __shfl_xor(sum, 16, WAVE);
    sum += __shfl_xor(sum, 32, WAVE);
    lrow = lrow * keep + sum;
    mrow = mx;
#pragma unroll
    for (int s = 0; s < DT; ++s) {
      o[s] *= keep;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int pv = p0 + t * 16 + kg * 4;
#pragma unroll
        for (int e = 0; e < 4; ++e)                        // what lies beyond may never have been written
          o[s] = __builtin_amdgcn_mfma_f32_16x16x4f32(blk[t] >= 0 && pv + e <= pos_max ? v[s][t][e] : 0.f, w[t][e], o[s], 0, 0, 0);
      }
    }
  }
#pragma unroll
  for (int s = 0; s < DT; ++s) *(f32x4*)&po[wave][li][s * 16 + kg * 4] = o[s];
  if (kg == 0) { pm[wave][li] = mrow; pl[wave][li] = lrow; }
  __syncthreads();
  for (int i = threadIdx.x; i < 16 * (HD / 4); i += W * WAVE) {
    const int r = i / (HD / 4), d = (i - r * (HD / 4)) * 4;
    if (r0 + r >= nrows) break;
    int mm;
    const size_t at = q_of(r0 + r, mm);
    const int row_pos = a.rows.pos[mm];
    if (c0 * ATT_CHUNK > row_pos) continue;                // (no key of the part is the row's, and its merge does not look here)
    float mx = -INFINITY, l = 0.f;
#pragma unroll
    for (int x = 0; x < W; ++x) mx = fmaxf(mx, pm[x][r]);  // (the part's first position is the row's: finite)
    f32x4 acc = {0, 0, 0, 0};
#pragma unroll
    for (int x = 0; x < W; ++x) {
      const float f = expf(pm[x][r] - mx);
      l = fmaf(pl[x][r], f, l);
      acc += *(const f32x4*)&po[x][r][d] * f;
    }
    if (row_pos < PC * ATT_CHUNK) {
      *(f32x4*)((float*)a.out + at + d) = acc / l;
    } else {
      const size_t pidx = at / HD * a.NC + part;
      *(f32x4*)(a.o_part + pidx * HD + d) = acc;
      if (d == 0) { a.ml_part[pidx * 2] = mx; a.ml_part[pidx * 2 + 1] = l; }
    }
  }
}

// ------------------------------------------------------------------------------------------------ matrix-core variant
// The same operation for bf16 caches with 16-token blocks and head_dim 64 or 128.  The query rows that share keys - R rows
// of a sequence x the G query heads of a group - form tiles of 16.  A workgroup takes WQ tiles and a part of the keys
// (`part_keys`, cut at absolute positions; a multiple of WK chunks, so that no key group walks into the next part); its waves are WQ
// tiles x WK key groups, and key group k walks the part's 64-key chunks k, k + WK, .. with a running (reference, sum, weighted values)
// per row.  The key groups meet once in LDS.  Where one part covers all keys the row is finished here; else its partial goes to memory
// and k_attn_combine_parts merges the parts in ascending order.
//
// S is computed transposed, S^T = K Q^T, and so is O^T = V^T P^T: a lane then holds scores and outputs of ONE query row
// (lane % 16), so the row maximum needs two cross-lane steps instead of sixteen, and P goes from the accumulators
// into the second product without leaving the registers: accumulator (tile h, register r) of lane group g is row
// 4 g + r of the key tile, and the keys are assigned to the rows of the two key tiles of a 32-key pair such that this is
// key 8 g + 4 h + r - the eight keys whose values lane group g holds in a value fragment.
// The row sum is P times a matrix of ones, with P as hi + lo as in the product with the values: numerator and denominator
// weigh with the same numbers.  Against 64 bits, the partials are off by 3.7e-6 to 1.4e-5 (2-norm, relative; 46 combinations of
// head size, 64 to 4000 cached positions, 1 to 64 sequences and scores of spread 0.5 to 6), which is the 2^-17 of the split
// operands: 0.998 times (geometric mean) what fp32 sums of the unsplit weights give, and 1.000 times what accumulators that
// start at zero give instead of minus the maximum.  (The fp32 sums cost 5 % with head size 128, nothing with 64.)
// Keys and values go from the paged cache to LDS with direct loads, a chunk ahead.  What bounds a long prefix is issue: beside the
// 16x16x32 matrix instructions (36 per wave and chunk, 16 cycles each) a SIMD issues about two vector instructions for nothing, and
// a wave has 80 a chunk, half of them for the split of P, and 16 exponentials.  With few keys per workgroup it is the chain of
// dependent latencies, and the code itself, fetched cold by every launch.
// So there are two loops.  Eight waves (4 tiles x 2 key groups, or 2 x 4: the launch's choice) take short parts: one copy of the code,
// the reference is the running maximum.  The other (LAZY) takes prompts whose parts have more than 16 chunks, with head size 64 on sixteen waves of a compute
// unit (4 x 4, 8 x 2 or two workgroups of 4 x 2: pick_attn_mfma) to overlap matrix and vector instructions, and the reference, the maximum of the row's first chunk, moves only to a score that exceeds it by ATT_LAZY, so that
// the usual chunk asks each lane for its own largest score and no more (some row of sixteen has a new maximum in most chunks: a
// maximum across lanes and 40 instructions of scaling).  The heaviest key then weighs anything up to 2^8 instead of 1, which the
// truncating split holds exactly; the split of later chunks rounds hi to nearest in return (error against 64 bits 0.85 times the other
// form's over 24 shapes; 1.02 times without).  1024 rows of the 0.5B shape at 0 / 1024 / 3072 cached positions: 14.6 / 22.8 / 38.7 us, with
// 4 x 2 15.8 / 25.0 / 47.1; the same loop with 4 x 2 14.6 / 24.2 / 43.1 but 0.5 us more for the batches' launches; 97 rows 7.7 against
// 6.1.  (Those times are of the kernel alone.  Where the line lies between the forms: pick_attn_mfma.)  Two row tiles per wave, which read keys and values half as often, took as long with as many waves and a quarter longer with half.
constexpr float ATT_LAZY = 8.0f;                         // weights may reach 2^8 before the reference moves (fp32 sums and the hi + lo split of
                                                         // a weight are as exact at any scale)

template <int HD, int WQ, int WK, bool LAZY>
__global__ void __launch_bounds__(WQ * WK * 64, LAZY && HD == 64 ? 4 : WQ * WK / 4) k_attn_mfma(AttnArgs a) {
  constexpr int KS = HD / 32, DT = HD / 16;
  constexpr int NB = 8 / WQ;                               // blocks that a wave loads of a chunk: half of a key group's waves keys, half values
  static_assert(WQ == 2 || WQ == 4 || WQ == 8, "");
  extern __shared__ u32x4 kvs[];                           // [key group][keys, values][buffer][block][KS][64]
  // (LAZY: the last rows, which reach the most keys, first: a long prompt's launch has more workgroups than fit, and the short ones fill its end)
  const int part = blockIdx.x % a.nparts, tgroup = LAZY ? a.n_tg - 1 - blockIdx.x / a.nparts : blockIdx.x / a.nparts, kvh = blockIdx.y, brel = blockIdx.z;
  const int seq = a.rows.seq0 + brel;
  const int R = a.rows.R, nkv = a.kv.nkv, G = a.nq / nkv, RG = R * G, m_first = brel * R;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wq = wave % WQ, kg = wave / WQ;
  const int g = lane >> 4, c16 = lane & 15;
  const int r0 = 16 * (tgroup * WQ + wq);                  // first of this wave's query rows
  // (constant address space: what the whole wave needs is read with scalar loads, which do not queue behind the loads in flight)
  typedef const __attribute__((address_space(4))) int32_t* const_i32;
  const const_i32 row_pos = (const_i32)(uintptr_t)(a.rows.pos + m_first);
  const const_i32 table = (const_i32)(uintptr_t)(a.kv.table + (size_t)seq * a.kv.mbps);
  // rows ascend in position: what the workgroup's last row, and this wave's first and last, reach
  const int wg_reach = row_pos[(min(16 * WQ * (tgroup + 1), RG) - 1) / G];
  const int pbase = part * a.part_keys;
  if (pbase > wg_reach) return;                            // (the whole workgroup)
  const bool has_rows = r0 < RG;
  const int pos_lo = has_rows ? row_pos[r0 / G] : 0;
  const int reach = has_rows ? row_pos[(min(r0 + 16, RG) - 1) / G] : -1;
  const int nch = min(a.part_keys >> 6, ((wg_reach - pbase) >> 6) + 1);           // chunks of the part that some row reaches
  const int nit = (nch + WK - 1) / WK;

  // Direct loads: each brings 1 KB of consecutive memory of one block (sixteen lanes that touch sixteen rows would load at a
  // quarter of the rate).  Keys are parked row by row with the 16-byte units of row t of a block permuted by XOR with
  // (t & 3) + 4 (t / 8), so that the rows of a key tile read their units from distinct banks; values as they are, dim by dim.
  const bool values = wq >= WQ / 2;
  const int b0 = NB * (wq % (WQ / 2));                     // first of this wave's blocks of a chunk
  const size_t block_elems = (size_t)nkv * 16 * HD, plane = (size_t)a.kv.n_blocks * block_elems;
  const bf16_t* pool = (const bf16_t*)a.kv.pool + (size_t)(2 * a.layer + (values ? 1 : 0)) * plane + (size_t)kvh * 16 * HD;
  int voff[KS];
  {
    constexpr int UPR = 4 * KS;                            // 16-byte units of a cached row
#pragma unroll
    for (int i = 0; i < KS; ++i) {
      const int t = (64 / UPR) * i + lane / UPR, unit = (lane % UPR) ^ ((t & 3) | ((t >> 1) & 4));
      voff[i] = values ? i * 512 + lane * 8 : t * HD + unit * 8;
          }
  }
  const int last_bi = min(a.kv.mbps - 1, wg_reach >> 4);
  int blk[NB];                                             // block ids of what this wave requests next
  auto look_up = [&](int it) {                             // ... which is its share of this key group's chunk of iteration `it`
    const int bi = (pbase >> 4) + 4 * (it * WK + kg) + b0;
#pragma unroll
    for (int t = 0; t < NB; ++t) blk[t] = table[min(bi + t, last_bi)];
  };
  u32x4* my = kvs + (size_t)kg * (4 * 4 * KS * 64);
  auto request = [&](int it) {
    u32x4* dst = my + ((values ? 2 : 0) + (it & 1)) * (4 * KS * 64) + b0 * (KS * 64);
#pragma unroll
    for (int t = 0; t < NB; ++t)
#pragma unroll
      for (int i = 0; i < KS; ++i)
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(pool + (size_t)max(blk[t], 0) * block_elems + voff[i]),      // (masked keys may read any block)
                                         (__attribute__((address_space(3))) void*)(dst + (t * KS + i) * 64), 16, 0, 0);
  };
  // query row c16 of the tile, scaled into the base-2 domain and split
  const int qr = r0 + c16;
  const bool qok = qr < RG;
  const int j = qok ? qr / G : 0, gq = qok ? qr - j * G : 0;
  const int m = m_first + j, hq = kvh * G + gq;
  const int pos = qok ? a.rows.pos[m] : -1;
  f32x4 q[KS][2];
  {
    const f32x4* qp = (const f32x4*)(a.q + ((size_t)m * a.nq + hq) * HD + g * 8);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) { q[ks][0] = qp[8 * ks]; q[ks][1] = qp[8 * ks + 1]; }
  }
  asm volatile("" ::: "memory");                           // (requested ahead of the keys, which wait for the block table; split while those travel: 0.5 us a launch)
  look_up(0);
  request(0);
  look_up(min(1, nit - 1));
  SplitA qf[KS];
  {
    const float scale2 = a.scale * 1.4426950408889634f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qf[ks] = split_bf16(__builtin_bit_cast(u32x4, q[ks][0] * scale2), __builtin_bit_cast(u32x4, q[ks][1] * scale2));
  }
  // running state of a row: the reference mrow of its weights, and o and l (all four registers of l hold the row's sum: P times a matrix of ones)
  float mrow = 0.f;
  f32x4 o[DT], l = {0, 0, 0, 0};
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) o[dt] = f32x4{0, 0, 0, 0};
  const bf16x8 ones = __builtin_bit_cast(bf16x8, u32x4{0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u});
  // (`first`: a bool, or its value as a type where the first chunk is code of its own)
  auto chunk = [&](int it, auto& first) {
    constexpr bool later = std::is_same<decltype(first), std::false_type&>::value;
    // the chunk has arrived, and every wave of the group has read the one whose buffer the next request overwrites
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (it + 1 < nit) { request(it + 1); look_up(min(it + 2, nit - 1)); }
    const int kbase = pbase + 64 * (it * WK + kg);
    if (kbase > reach) return;                             // (uniform over the wave; always so for a wave without rows)
    // Scores minus the row's reference (the accumulators start at -mrow).  Element (tile t, register r): key
    // kbase + 32 (t / 2) + 8 g + 4 (t % 2) + r of row c16.  Independent chains of matrix-core instructions side by side.
    const u32x4* kk = my + (it & 1) * (4 * KS * 64) + (8 * (c16 >> 2) + (c16 & 3)) * (4 * KS);       // row 8 (c16 / 4) + c16 % 4 of a pair
    const u32x4* vv = my + (2 + (it & 1)) * (4 * KS * 64) + (g >> 1) * (KS * 64) + 2 * c16 + (g & 1);
    bf16x8 kf[4][KS];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) kf[t][ks] = __builtin_bit_cast(bf16x8, kk[(t >> 1) * (2 * KS * 64) + (t & 1) * (16 * KS) + ((4 * ks + g) ^ (c16 & 7))]);
    f32x4 s[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) s[t] = f32x4{-mrow, -mrow, -mrow, -mrow};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int t = 0; t < 4; ++t) s[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[t][ks], qf[ks].lo, s[t], 0, 0, 0);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int t = 0; t < 4; ++t) s[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[t][ks], qf[ks].hi, s[t], 0, 0, 0);
    if (kbase + 63 > pos_lo) {
      const int left = pos - kbase - 8 * g;
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (32 * (t >> 1) + 4 * (t & 1) + r > left) s[t][r] = -INFINITY;
    }
    float mx = s[0][0];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) mx = fmaxf(mx, s[t][r]);
    constexpr float keep = LAZY ? ATT_LAZY : 0.f;
    if (!LAZY) mx = max_over_groups(mx);                   // (taken in most chunks: better ahead of the branch)
    if (first || __any(mx > keep)) {                       // the first scores, or larger ones: what is there shrinks
      if (LAZY) mx = max_over_groups(mx);
      const float up = first ? (mx == -INFINITY ? 0.f : mx) : LAZY ? (mx > keep ? mx : 0.f) : fmaxf(mx, 0.f), alpha = first ? 0.f : __builtin_amdgcn_exp2f(-up);
      if constexpr (!LAZY) first = false;
      mrow += up;
      l *= alpha;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) o[dt] *= alpha;
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) s[t][r] -= up;
    }
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) s[t][r] = __builtin_amdgcn_exp2f(s[t][r]);
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const SplitA pf = later ? split_bf16_near(s[2 * p], s[2 * p + 1]) : split_bf16(__builtin_bit_cast(u32x4, s[2 * p]), __builtin_bit_cast(u32x4, s[2 * p + 1]));
      bf16x8 vf[DT];
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) vf[dt] = __builtin_bit_cast(bf16x8, vv[p * (2 * KS * 64) + dt * 32]);
      l = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, pf.lo, l, 0, 0, 0);
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) o[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[dt], pf.lo, o[dt], 0, 0, 0);
      l = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, pf.hi, l, 0, 0, 0);
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) o[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[dt], pf.hi, o[dt], 0, 0, 0);
    }
  };
  if constexpr (LAZY) {
    std::true_type first;
    std::false_type later;
    chunk(0, first);
    for (int it = 1; it < nit; ++it) chunk(it, later);
  } else {
    bool first = true;
    for (int it = 0; it < nit; ++it) chunk(it, first);
  }
  if (l[0] == 0.f) mrow = -1e30f;                          // no key of the row in this key group
  // key groups 1 .. WK-1 hand their state over, group 0 adds them in ascending order
  __syncthreads();
  f32x4* xch = (f32x4*)kvs;                                // [key group - 1][wq][DT + 1][64]
  constexpr int XT = (DT + 1) * 64;
  if (kg > 0) {
    f32x4* x = xch + (size_t)((kg - 1) * WQ + wq) * XT + lane;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) x[dt * 64] = o[dt];
    x[DT * 64] = f32x4{mrow, l[0], 0.f, 0.f};
  }
  __syncthreads();
  if (kg > 0 || !qok) return;
  float lr = l[0];
#pragma unroll
  for (int k = 1; k < WK; ++k) {
    const f32x4* x = xch + (size_t)((k - 1) * WQ + wq) * XT + lane;
    const f32x4 ml = x[DT * 64];
    const float mnew = fmaxf(mrow, ml[0]), wa = __builtin_amdgcn_exp2f(mrow - mnew), wb = __builtin_amdgcn_exp2f(ml[0] - mnew);
    mrow = mnew;
    lr = lr * wa + ml[1] * wb;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) o[dt] = o[dt] * wa + x[dt * 64] * wb;
  }
  if (pbase > pos) return;                                 // the row does not reach the part (the merge reads no such partial)
  if (a.nparts == 1) {                                     // dims 16 dt + 4 g .. + 3 of the finished row
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
      const f32x4 y = o[dt] / lr;
      bf16_t* out = (bf16_t*)a.out + split_index(m, hq * HD + 16 * dt + 4 * g, a.split_kt);
      *(uint2*)out = hi_pairs(y);
      *(uint2*)(out + 512) = lo_pairs(y);
    }
    return;
  }
  const size_t pidx = ((size_t)m * a.nq + hq) * a.NC + part;
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) *(f32x4*)(a.o_part + pidx * HD + 16 * dt + 4 * g) = o[dt];
  if (g == 0) { a.ml_part[pidx * 2] = mrow; a.ml_part[pidx * 2 + 1] = lr; }
}

// Merges a row's part partials (base-2 references) in ascending part order: HD / 4 lanes per (row, query head), four dims each.
// A chain of two loads once the first parts' no longer wait for the row's position: 16 sequences x 7 rows 4.3 -> 3.9 us a launch.
template <int HD>
__global__ void __launch_bounds__(BLOCK) k_attn_combine_parts(AttnArgs a) {
  constexpr int L = HD / 4;
  const int rh = blockIdx.x * (BLOCK / L) + threadIdx.x / L, d = (threadIdx.x % L) * 4;
  if (rh >= a.rows.M * a.nq) return;
  const int m = rh / a.nq, hq = rh - m * a.nq;
  const int pos = a.rows.pos[m];
  const size_t base = (size_t)rh * a.NC;
  float mx = -INFINITY, l = 0.f;
  f32x4 o = {0, 0, 0, 0};
  float2 ml[4];
  f32x4 x[4];
  auto load = [&](int p0) {                                // four parts' loads in flight; the first four do not wait for the position
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int p = min(p0 + u, a.nparts - 1);             // (what lies in parts that the row does not reach is not looked at)
      ml[u] = *(const float2*)(a.ml_part + (base + p) * 2);
      x[u] = *(const f32x4*)(a.o_part + (base + p) * HD + d);
    }
  };
  load(0);
  asm volatile("" ::: "memory");                           // (else they sink below the loop's first test)
  const int np = pos / a.part_keys + 1;
  for (int p0 = 0; p0 < np; p0 += 4) {
    if (p0) load(p0);
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (p0 + u < np) {
        const float mnew = fmaxf(mx, ml[u].x), wa = __builtin_amdgcn_exp2f(mx - mnew), wb = __builtin_amdgcn_exp2f(ml[u].x - mnew);
        mx = mnew;
        l = l * wa + ml[u].y * wb;
        o = o * wa + x[u] * wb;
      }
  }
  const f32x4 y = o / l;
  bf16_t* out = (bf16_t*)a.out + split_index(m, hq * HD + d, a.split_kt);
  *(uint2*)out = hi_pairs(y);
  *(uint2*)(out + 512) = lo_pairs(y);
}

}  // namespace ssd
