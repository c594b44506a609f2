// Row kernels around the vocabulary: embedding gather + row bookkeeping, residual add + RMSNorm,
// warp + softmax, and the acceptance / resampling / commit kernel (Eq. 5-6, Alg. 1).
#pragma once
#include "common.h"

namespace ssd {

// ------------------------------------------------------------------------------------------ rows + embed
struct EmbedArgs {
  KvView kv;
  Rows rows;
  int pcap;                 // pending slots at the head of each sequence's rows (0 for a prefill chunk)
  int n_seqs;
  const int32_t* tokens;    // explicit tokens [n_seqs][tok_stride] for rows j >= pcap
  int tok_stride;
  const void* embed;        // [n_embed][d]
  int n_embed, d;
  float* h;                 // [M][d]
  const float* gain;        // of the first layer's norm
  float eps;
  bf16_t* xn;               // the normalised rows as split rows (null: the next kernel normalises)
};

// RMSNorm of a row whose columns 4 tid .. + 3 (+ 4 blockDim ..) a workgroup's threads hold, the first four of each thread in v0 and
// the rest in memory (hr); g0: the gain of those four, requested with what the kernel reads first; ss: the thread's share of the sum of
// squares.
__device__ __forceinline__ f32x4 first_gain(const float* gain, int d) {
  return (int)threadIdx.x * 4 < d ? *(const f32x4*)(gain + threadIdx.x * 4) : f32x4{0, 0, 0, 0};
}
__device__ __forceinline__ void norm_row(const float* hr, f32x4 v0, f32x4 g0, float ss, const float* gain, float eps, bf16_t* xn, int m, int d,
                                         float* s16) {
  ss = wave_sum(ss);
  if ((threadIdx.x & 63) == 0) s16[threadIdx.x >> 6] = ss;
  __syncthreads();
  float tot = 0.f;
  for (int w = 0; w < (int)blockDim.x >> 6; ++w) tot += s16[w];
  const float inv = 1.0f / sqrtf(tot / (float)d + eps);
  for (int i = threadIdx.x * 4; i < d; i += blockDim.x * 4) {
    const bool held = i == (int)threadIdx.x * 4;
    f32x4 v = held ? v0 : *(const f32x4*)(hr + i);
    const f32x4 gn = held ? g0 : *(const f32x4*)(gain + i);
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = v[r] * inv * gn[r];
    bf16_t* o = xn + split_index(m, i, d >> 5);
    *(uint2*)o = hi_pairs(v);
    *(uint2*)(o + 512) = lo_pairs(v);
  }
}

// One workgroup per row: resolve the row's token and position, copy its embedding into the residual stream and normalise it
// for the first layer.  One more workgroup reserves the cache blocks the forward will write (sequences in ascending order).
// The kernel is a chain of dependent reads (state, token, embedding, norm), so the reservation is a chain of its own beside
// it and the norm no launch of its own: a forward is 4 us shorter, a prefill chunk of 1024 rows another 8.
template <typename WT>
__global__ void __launch_bounds__(1024) k_embed(EmbedArgs e) {
  if ((int)blockIdx.x == e.rows.M) {
    __shared__ int scan[1024 + 16], slot[1024];
    for (int b0 = 0; b0 < e.n_seqs; b0 += blockDim.x) {
      const bool in = b0 + (int)threadIdx.x < e.n_seqs;
      const int s = e.rows.seq0 + (in ? b0 + (int)threadIdx.x : 0);
      const int o = e.pcap ? e.pcap - e.kv.n_pend[s] : 0;
      kv_reserve_all(e.kv, in, s, e.kv.len[s] + e.rows.R - o, scan, slot);
    }
    return;
  }
  __shared__ float s16[16];
  const f32x4 g0 = e.xn ? first_gain(e.gain, e.d) : f32x4{0, 0, 0, 0};
  const int m = blockIdx.x;
  const int brel = m / e.rows.R, j = m - brel * e.rows.R;
  const int seq = e.rows.seq0 + brel;
  const int npend = e.pcap ? e.kv.n_pend[seq] : 0;
  const int off = e.pcap - npend;                          // leading rows that carry nothing
  const int len = e.kv.len[seq];
  int tok, pos, active;
  if (j < off) { tok = e.kv.pend[seq * 2]; pos = len; active = 0; }
  else {
    pos = len + (j - off); active = 1;
    tok = j < e.pcap ? e.kv.pend[seq * 2 + (j - off)] : e.tokens[(size_t)brel * e.tok_stride + (j - e.pcap)];
  }
  tok = min(max(tok, 0), e.n_embed - 1);
  if (threadIdx.x == 0) { e.rows.pos[m] = pos; e.rows.active[m] = active; }
  const typename WT::T* src = (const typename WT::T*)e.embed + (size_t)tok * e.d;
  float* hr = e.h + (size_t)m * e.d;
  f32x4 v0 = {0, 0, 0, 0};
  float ss = 0.f;
  for (int i = threadIdx.x * 4; i < e.d; i += blockDim.x * 4) {
    const f32x4 v = {WT::ld(src + i), WT::ld(src + i + 1), WT::ld(src + i + 2), WT::ld(src + i + 3)};
    *(f32x4*)(hr + i) = v;
    if (i == (int)threadIdx.x * 4) v0 = v;
#pragma unroll
    for (int r = 0; r < 4; ++r) ss = fmaf(v[r], v[r], ss);
  }
  if (e.xn) norm_row(hr, v0, g0, ss, e.gain, e.eps, e.xn, m, e.d, s16);
}

// h[m] += sum of the k-split partials of the previous GEMM (ascending split order); xn[m] = RMSNorm(h[m]) * gain, as fp32 rows
// or as split rows (common.h) for the matrix-core GEMMs.  One workgroup per row, four consecutive columns per thread; a
// row of up to 4 * blockDim columns stays in registers between the two passes.  What bounds it is latency: the row, its partials
// (NP >= n_part; those that are missing repeat the last one's address and are not added) and the gain are requested together, one trip to memory
// instead of three (112 rows of width 896 4.2 -> 3.8 us, 1024 7.9 -> 6.9).
template <int NP>
__global__ void __launch_bounds__(1024) k_add_norm(float* h, const float* part, int n_part, size_t part_stride, const float* gain,
                                                   float eps, bf16_t* xn, int d) {
  __shared__ float s16[16];
  const int m = blockIdx.x;
  float* hr = h + (size_t)m * d;
  const f32x4 g0 = first_gain(gain, d);
  f32x4 v0 = {0, 0, 0, 0};
  float ss = 0.f;
  for (int i = threadIdx.x * 4; i < d; i += blockDim.x * 4) {
    f32x4 v = *(const f32x4*)(hr + i);
    const float* pp = part + (size_t)m * d + i;
    f32x4 x[NP];
#pragma unroll
    for (int u = 0; u < NP; ++u) x[u] = *(const f32x4*)(pp + (size_t)min(u, n_part - 1) * part_stride);
    asm volatile("" ::: "memory");                         // (else each load sinks to its sum)
#pragma unroll
    for (int u = 0; u < NP; ++u)
      if (u < n_part) v += x[u];
    *(f32x4*)(hr + i) = v;
    if (i == (int)threadIdx.x * 4) v0 = v;
#pragma unroll
    for (int r = 0; r < 4; ++r) ss = fmaf(v[r], v[r], ss);
  }
  norm_row(hr, v0, g0, ss, gain, eps, xn, m, d, s16);
}

// ------------------------------------------------------------------------------------------ warp + softmax
__device__ __forceinline__ uint32_t order_key(float f) {      // larger float <-> larger key
  const uint32_t u = __float_as_uint(f + 0.0f);              // (-0 is +0: they tie)
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ __forceinline__ float key_order(uint32_t k) {      // its inverse
  return __uint_as_float(k & 0x80000000u ? k & 0x7FFFFFFFu : ~k);
}

struct WarpArgs {
  const float* logits;   // [rows][ld]
  int ld, V;
  float temperature;
  int top_k, greedy;
  float* probs;          // [rows][V] or strided
  size_t probs_stride;
};

constexpr int SBLOCK = 1024;          // threads of the two sampler kernels (16 waves): short unrolled loops, small code
constexpr int SPER = 16;              // elements per thread at most: vocab <= 16384.  The kernels are instantiated for 1, 8 and 16: the
                                      // loops over a thread's elements are unrolled to that count, and what a vocabulary does not fill costs
constexpr int TOPK_CAND = 1024;       // top-k candidates that are ranked in LDS

// Reductions over the 16 waves of a sampler workgroup through 16 LDS entries, which are this reduction's alone (a later one that
// reused them would need a barrier more); all threads get the result.
__device__ __forceinline__ float sblock_max(float v, float* s16) {
  v = wave_max(v);
  if ((threadIdx.x & 63) == 0) s16[threadIdx.x >> 6] = v;
  __syncthreads();
  float r = s16[0];
#pragma unroll
  for (int i = 1; i < 16; ++i) r = fmaxf(r, s16[i]);
  return r;
}
__device__ __forceinline__ float sblock_sum(float v, float* s16) {      // fixed order: waves ascending
  v = wave_sum(v);
  if ((threadIdx.x & 63) == 0) s16[threadIdx.x >> 6] = v;
  __syncthreads();
  float r = s16[0];
#pragma unroll
  for (int i = 1; i < 16; ++i) r += s16[i];
  return r;
}

// One workgroup per row.  Top-k keeps exactly k entries: everything above the k-th largest value, and of the
// entries equal to it the ones with the lowest indices.
template <int SP>
__device__ __forceinline__ void warp_softmax_row(const WarpArgs w, const int row, float* lds_probs = nullptr) {
  __shared__ float max16[16], sum16[16];
  __shared__ int i16[16];
  __shared__ int cnt16[2][16];
  __shared__ unsigned long long cand[TOPK_CAND];
  __shared__ __align__(16) uint32_t group_max[SBLOCK / 8];
  __shared__ uint32_t sh_kth, sh_best;
  __shared__ int sh_n, sh_idxmax;
  const int tid = threadIdx.x;
  const float* x = w.logits + (size_t)row * w.ld;
  float* p = w.probs + (size_t)row * w.probs_stride;
  const int V = w.V;
  // the row is read once into registers (all loads in flight together)
  float xv[SP];
#pragma unroll
  for (int e = 0; e < SP; ++e) {
    const int i = tid + e * SBLOCK;
    xv[e] = i < V ? x[i] : -INFINITY;
  }

  if (w.greedy) {                                            // one-hot at the arg-max, lowest index on ties
    float best = -INFINITY; int bi = 0x7fffffff;
#pragma unroll
    for (int e = 0; e < SP; ++e) { if (xv[e] > best) { best = xv[e]; bi = tid + e * SBLOCK; } }
    const float mx = sblock_max(best, max16);
    int cand = (best == mx) ? bi : 0x7fffffff;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) cand = min(cand, __shfl_xor(cand, o, WAVE));
    if ((tid & 63) == 0) i16[tid >> 6] = cand;
    __syncthreads();
    int arg = i16[0];
#pragma unroll
    for (int i = 1; i < 16; ++i) arg = min(arg, i16[i]);
#pragma unroll
    for (int e = 0; e < SP; ++e) {
      const int i = tid + e * SBLOCK;
      if (i < V) {
        p[i] = (i == arg) ? 1.0f : 0.0f;
        if (lds_probs) lds_probs[i] = (i == arg) ? 1.0f : 0.0f;
      }
    }
    return;
  }

  // The cut of the top-k set, in three steps.
  //  1. A lower bound of the k-th largest key: the k-th largest of the maxima of 128 disjoint groups of entries (eight threads'
  //     each) is reached by at least k entries.  Eight threads rank a group's maximum against the others, two barriers in all.
  //     Logits without order over the vocabulary leave little more than k entries above it (k = 25: about 28, k = 50: 62).
  //  2. Where more than `cap` entries reach the bound (k > 128, or large entries that share groups), a binary search from there
  //     over the order-preserving integer keys for a threshold that between k and `cap` reach (a step counts with wave ballots: no
  //     atomics, one barrier).
  //  3. The candidates are collected in LDS and ranked against each other by (value, index), four threads per candidate.
  // (112 rows of 6564 with k = 25: 8.9 us, where the search alone, about eight steps from zero, took 12.8, and a radix select by LDS
  // histograms 44, serialised on the few leading bytes that logits share.  One row with its draw: 11.9 against 17.0.)
  uint32_t kth = 0;          // keep keys > kth, and keys == kth with index <= idxmax
  int idxmax = 0x7fffffff;
  const bool use_k = w.top_k > 0 && w.top_k < V;
  float best = -INFINITY;    // the thread's largest entry, with top-k the row's
  if (use_k) {
    const int k = w.top_k;
    const int cap = k <= 128 ? 256 : k <= TOPK_CAND / 2 ? TOPK_CAND : 0;   // 0: search down to the exact key
    uint32_t key[SP], top = 0;
#pragma unroll
    for (int e = 0; e < SP; ++e) {
      const bool in = tid + e * SBLOCK < V;
      key[e] = in ? order_key(xv[e]) : 0u;                   // (padding: below every number)
      top = max(top, key[e]);
    }
    // groups of eight lanes: pairs, quads, half rows (common.h)
    top = max(top, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)top, 0xB1, 0xF, 0xF, true));
    top = max(top, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)top, 0x4E, 0xF, 0xF, true));
    top = max(top, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)top, 0x141, 0xF, 0xF, true));
    if ((tid & 7) == 0) group_max[tid >> 3] = top;
    if (tid == 0) { sh_n = 0; sh_kth = 0; }
    __syncthreads();
    {                                                        // rank of this group's maximum, ties by the group's number
      const int g = tid >> 3, g0 = (tid & 7) * 16;
      const uint32_t mine = group_max[g];
      int rank = 0;
#pragma unroll
      for (int j = 0; j < 16; j += 4) {
        const u32x4 o = *(const u32x4*)&group_max[g0 + j];
#pragma unroll
        for (int i = 0; i < 4; ++i) rank += o[i] > mine || (o[i] == mine && g0 + j + i < g);
      }
      rank += __builtin_amdgcn_update_dpp(0, rank, 0xB1, 0xF, 0xF, true);
      rank += __builtin_amdgcn_update_dpp(0, rank, 0x4E, 0xF, 0xF, true);
      rank += __builtin_amdgcn_update_dpp(0, rank, 0x141, 0xF, 0xF, true);
      if ((tid & 7) == 0 && rank == 0) sh_best = mine;
      if ((tid & 7) == 0 && rank == k - 1) sh_kth = mine;    // (no group where k exceeds their number: the bound stays 0)
    }
    __syncthreads();
    int turn = 0;
    auto reach = [&](uint32_t t) {                           // entries with key >= t (t > 0)
      int c = 0;
#pragma unroll
      for (int e = 0; e < SP; ++e) c += __popcll(__ballot(key[e] >= t));
      turn ^= 1;
      if ((tid & 63) == 0) cnt16[turn][tid >> 6] = c;
      __syncthreads();                                       // (the other buffer is rewritten a step, and a barrier, later)
      int n = 0;
#pragma unroll
      for (int i = 0; i < 16; ++i) n += cnt16[turn][i];
      return n;
    };
    uint32_t lo = sh_kth, hi = sh_best;
    best = key_order(hi);
    int c_lo = lo ? reach(lo) : V, c_hi = 0;
    if (c_lo > cap) {
      c_hi = reach(hi);
      if (c_hi >= k) { lo = hi; c_lo = c_hi; c_hi = 0; }     // k or more entries equal the maximum
      else {
        while (c_lo > cap && hi - lo > 1) {
          const uint32_t mid = lo + ((hi - lo) >> 1);
          const int c = reach(mid);
          if (c >= k) { lo = mid; c_lo = c; }
          else { hi = mid; c_hi = c; }
        }
      }
    }
    if (c_lo <= cap) {
#pragma unroll
      for (int e = 0; e < SP; ++e)
        if (tid + e * SBLOCK < V && key[e] >= lo)
          cand[atomicAdd(&sh_n, 1)] = ((unsigned long long)key[e] << 32) | (uint32_t)~(tid + e * SBLOCK);
      __syncthreads();
      const int n = min(sh_n, TOPK_CAND);
      for (int c0 = 0; c0 < n; c0 += SBLOCK / 4) {
        const int c = c0 + (tid >> 2);
        const unsigned long long mine = c < n ? cand[c] : 0ull;
        int rank = 0;
        for (int j = tid & 3; j < n; j += 4) rank += cand[j] > mine;
        rank += __shfl_xor(rank, 1, WAVE);
        rank += __shfl_xor(rank, 2, WAVE);
        if (c < n && rank == k - 1 && (tid & 3) == 0) { sh_kth = (uint32_t)(mine >> 32); sh_idxmax = (int)~(uint32_t)mine; }
      }
      __syncthreads();
      kth = sh_kth;
      idxmax = sh_idxmax;
    } else {                                                 // `lo` is the k-th key: k - c_hi of the entries equal to it survive
      kth = lo;
      if (c_lo > k) {                                        // a tie straddles the cut: rare, resolved serially
        if (tid == 0) {
          int seen = c_hi, im = V - 1;
          for (int i = 0; i < V; ++i)
            if (order_key(x[i]) == kth && ++seen == k) { im = i; break; }
          sh_idxmax = im;
        }
        __syncthreads();
        idxmax = sh_idxmax;
      }
    }
  }
  // The kernel is bound by instruction issue (one row is four waves per SIMD of one compute unit), and a division or an exponential
  // is ten instructions and more: a temperature of 1 divides nothing, with top-k a wave passes over the steps in which it
  // holds no kept entry (at most k of the row's 16 x SP; the largest entry is kept, so the maximum is known), and the
  // division of a whole row by its sum multiplies by the reciprocal and corrects by the residual, which is the rounded quotient as
  // long as nothing is subnormal (Markstein, "Computation of elementary functions on the IBM RISC System/6000 processor", 1990).
  // One row of 6564 with its draw: 9.8 -> 8.5 us with this, reductions without LDS shuffles and three barriers less; with top-k 25 12.2 -> 11.0.
  const float T = w.temperature;
  const bool scale = T != 1.0f;
  float z[SP];
  float mx = -INFINITY;
  bool some[SP];
#pragma unroll
  for (int e = 0; e < SP; ++e) {
    const int i = tid + e * SBLOCK;
    bool keep = i < V;
    some[e] = true;
    if (use_k) {
      const uint32_t k = order_key(xv[e]);
      keep = keep && (k > kth || (k == kth && i <= idxmax));
      some[e] = __any(keep);
    }
    z[e] = keep ? xv[e] : -INFINITY;
    if (scale && some[e]) z[e] /= T;
    mx = fmaxf(mx, z[e]);
  }
  mx = use_k ? (scale ? best / T : best) : sblock_max(mx, max16);
  float sum = 0.f;
  bool tiny = false;
#pragma unroll
  for (int e = 0; e < SP; ++e) {
    if (some[e]) z[e] = (z[e] == -INFINITY) ? 0.f : expf(z[e] - mx);
    else z[e] = 0.f;
    sum += z[e];
    if (!use_k) tiny |= z[e] > 0.f && z[e] < 7.9e-31f;       // 2^-100: its quotient's residual is no longer normal
  }
  sum = sblock_sum(sum, sum16);                              // (at least 1 and at most V, unless the row has no number at its top)
  const float rcp = 1.0f / sum;
  const bool sound = sum > 0.f && sum < INFINITY;            // else every entry of the row is what the division gives
  const bool quick = !use_k && sound && !__any(tiny);
#pragma unroll
  for (int e = 0; e < SP; ++e) {
    const int i = tid + e * SBLOCK;
    float q = 0.f;
    if (quick) {
      const float q0 = z[e] * rcp;
      q = fmaf(fmaf(-q0, sum, z[e]), rcp, q0);
    } else if (some[e] || !sound) q = z[e] / sum;
    if (i < V) {
      p[i] = q;
      if (lds_probs) lds_probs[i] = q;                        // k_warp_accept: the draw reads the row from LDS
    }
  }
}

template <int SP>
__global__ void __launch_bounds__(SBLOCK) k_warp_softmax(WarpArgs w) { warp_softmax_row<SP>(w, blockIdx.x); }

// ------------------------------------------------------------------------------ acceptance + resampling
struct AcceptArgs {
  const float* pt;       // [B][K+1][V]
  size_t pt_seq_stride;  // elements between sequences
  const float* pd;       // [B][K][V]
  const int32_t* x;      // [B][K]
  const float* uniforms; // [B][K+1] or NULL -> Philox(seed, seq, step, slot)
  uint64_t seed, step;
  const int32_t* step_dev;  // when set: two words (low, high) of a device-resident cycle counter that is added to `step`, so
                         // that a captured graph of a cycle draws fresh uniforms at every replay
  int bump_step;         // the committing thread advances that counter (the last sampling kernel of a cycle without drafts)
  uint32_t launch;       // not 0: this kernel follows a forward on a.kv, the committing thread advances the cache's launch number (kv_publish_forward)
  int slot_base;         // r_i uses slot slot_base + i - 1, the emitted token slot_base + K
  int B, K, V;
  float beta;
  int32_t* n_acc;        // [B] (may be NULL)
  int32_t* next_tok;     // [B*tok_stride]
  int tok_stride;
  int32_t* flags;        // [B] or NULL
  int32_t* ticket;       // arrival counter of the workgroups of a multi-sequence commit: zero before the launch, zero after it
  // commit (kv.len == NULL: decisions only)
  KvView kv;
  int seq0;
};

// Fixed-point weight of the canonical sampler: floor(w * 2^40) for a float w < 2^23 (0 for negative ones), exactly: w * 2^40 is a shift
// of w's exponent, its upper and lower 32 bits are exact again.
__device__ __forceinline__ unsigned long long fix40(float w) {
  const float u = fmaxf(w, 0.f) * 1099511627776.0f;
  const uint32_t hi = (uint32_t)(u * 2.3283064365386963e-10f);
  const uint32_t lo = (uint32_t)fmaf((float)hi, -4294967296.0f, u);
  return ((unsigned long long)hi << 32) | lo;
}

// Exclusive prefix sum of one 64-bit value per thread over the 1024 threads of a sampler workgroup (integer: exact
// in any order).  w16: 16 entries of LDS.
__device__ __forceinline__ unsigned long long sblock_excl_scan_u64(unsigned long long v, unsigned long long* w16,
                                                                   unsigned long long* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const unsigned long long inc = wave_inclusive_scan(v);
  __syncthreads();
  if (lane == 63) w16[wave] = inc;
  __syncthreads();
  unsigned long long base = 0, tot = 0;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    if (i < wave) base += w16[i];
    tot += w16[i];
  }
  *total = tot;
  return base + inc - v;
}

// One workgroup per sequence.
//  1. lanes i < K: threshold min(1, pt_i(x_i)/pd_i(x_i)) + beta in fp32 (division only when pd > pt, so never by
//     zero), accept iff r_i < threshold; n = number of leading accepts via a wave ballot.
//  2. emitted token: inverse CDF over w_j = max(0, pt_{n+1}(j) - pd_{n+1}(j)) (n < K) or pt_{K+1}(j) (n == K), with the
//     weights in 2^40 fixed point so that the total and the prefix sums are integers (no dependence on the
//     summation tree): smallest j whose inclusive prefix exceeds floor(total * u).
//  3. the last workgroup to finish commits every sequence in ascending order: len += pending + n, pending =
//     emitted token, blocks past the new length go back to the free stack.
template <int SP>
__device__ __forceinline__ void accept_seq(const AcceptArgs a, const int b, const float* lds_row0 = nullptr) {
  __shared__ unsigned long long w16[16];
  __shared__ int sh_n, sh_tok, sh_last;
  __shared__ float sh_u;
  const int tid = threadIdx.x;
  const int K = a.K, V = a.V;
  const float* pt = a.pt + (size_t)b * a.pt_seq_stride;
  const float* pd = a.pd + (size_t)b * K * V;
  const uint32_t seq = (uint32_t)(a.seq0 + b);
  uint64_t step = a.step;
  if (a.step_dev) step += (uint64_t)(uint32_t)a.step_dev[0] | ((uint64_t)(uint32_t)a.step_dev[1] << 32);
  // A sequence commits without waiting for anyone where no other commit depends on it: a single one, and any of a step
  // without drafts, which keeps every row it has reserved blocks for and so gives none back.  Its cache state is requested
  // now (nothing but its own commit changes it), so that the commit at the end is stores only.
  const bool solo = a.kv.len != nullptr && (a.B == 1 || (a.K == 0 && !a.bump_step));
  int st_len = 0, st_npend = 0, st_owned = 0, st_top = 0, st_err = 0, st_launch = 0;
  uint32_t st_dev_err = 0;
  if (solo && tid == 0) {
    st_len = a.kv.len[seq]; st_npend = a.kv.n_pend[seq]; st_owned = a.kv.owned[seq];
    st_top = a.kv.ctl[0]; st_err = a.kv.ctl[1]; st_launch = a.kv.ctl[3]; st_dev_err = *a.kv.err;
  }

  if (tid < WAVE) {
    bool acc = false;
    if (tid < K) {
      const int xi = min(max(a.x[b * K + tid], 0), V - 1);
      const float ptx = pt[(size_t)tid * V + xi], pdx = pd[(size_t)tid * V + xi];
      const float r = a.uniforms ? a.uniforms[b * (K + 1) + tid] : philox_uniform(a.seed, seq, step, a.slot_base + tid);
      float thr;
      if (pdx > ptx) thr = __fadd_rn(__fdiv_rn(ptx, pdx), a.beta);
      else thr = __fadd_rn(1.0f, a.beta);
      acc = r < thr;
    }
    const unsigned long long rej = ~__ballot(acc);          // lanes >= K vote "reject"
    if (tid == 0) sh_n = min(__ffsll((long long)rej) - 1, K);
  }
  if (tid == WAVE)                                         // the uniform of the draw: one thread of the second wave
    sh_u = a.uniforms ? a.uniforms[b * (K + 1) + K] : philox_uniform(a.seed, seq, step, a.slot_base + K);
  __syncthreads();
  const int n = __builtin_amdgcn_readfirstlane(sh_n);       // (the row is the whole workgroup's: scalar addresses)
  const float u = sh_u;
  const float* prow = (lds_row0 && n == 0) ? lds_row0 : pt + (size_t)n * V;
  const float* drow = pd + (size_t)n * V;                   // only read when n < K
  const int per = (V + SBLOCK - 1) / SBLOCK;                // contiguous span of indices per thread (<= SP)
  const int j0 = tid * per;
  // It is read as SP entries that start at jb, of which those of the span count: a load behind a condition of its own waits for the one
  // before it, and addresses that are clamped one by one are 16 pairs of registers, which 1024 threads do not have.  (One sequence of
  // 6564 / 9000 / 16384, K = 6: 4.1 / 4.9 / 5.6 us; with both, and the spilled fixed-point weights below, 5.8 / 20 / 20.)
  const int jb = min(j0, V - SP);                           // (the instantiation has V >= SP)
  int fallback = 0;
  bool residual = n < K;
  unsigned long long total, excl, mine;
  float wgt[SP];
  for (;;) {
    // the thread's span of weights, all loads in flight together
#pragma unroll
    for (int e = 0; e < SP; ++e) wgt[e] = prow[jb + e];
    if (residual) {
      float d[SP];
#pragma unroll
      for (int e = 0; e < SP; ++e) d[e] = drow[jb + e];
#pragma unroll
      for (int e = 0; e < SP; ++e) wgt[e] = fmaxf(__fsub_rn(wgt[e], d[e]), 0.f);
    }
#pragma unroll
    for (int e = 0; e < SP; ++e)
      if (jb + e < j0 || jb + e >= j0 + per) wgt[e] = 0.f;
    mine = 0;
#pragma unroll
    for (int e = 0; e < SP; ++e) mine += fix40(wgt[e]);
    excl = sblock_excl_scan_u64(mine, w16, &total);          // sum of the spans before this thread's, and of all
    if (total == 0 && residual) { residual = false; fallback = 1; continue; }
    break;
  }
  if (total == 0) {
    if (tid == 0) sh_tok = 0;
  } else {
    const unsigned long long Ru = (unsigned long long)(u * 16777216.0f);
    const unsigned long long tgt = (__umul64hi(total, Ru) << 40) | ((total * Ru) >> 24);   // floor(total*Ru / 2^24)
    if (excl <= tgt && tgt < excl + mine) {
      unsigned long long c = excl;
      int tok = min(j0 + per, V) - 1;
      bool found = false;
#pragma unroll
      for (int e = 0; e < SP; ++e) {
        asm volatile("" : "+v"(wgt[e]));                   // (converted again by the one thread that draws, not kept by all as 64-bit numbers)
        c += fix40(wgt[e]);
        if (!found && c > tgt) { tok = jb + e; found = true; }
      }
      sh_tok = tok;
    }
  }
  __syncthreads();
  if (tid == 0) {
    if (a.n_acc) a.n_acc[b] = n;
    a.next_tok[(size_t)b * a.tok_stride] = sh_tok;
    if (a.flags) a.flags[b] = fallback;
  }
  if (a.kv.len == nullptr) return;
  if (solo) {                                              // kv_truncate + kv_publish on the values read at the start
    if (tid == 0) {
      if (a.launch && b == 0) { a.kv.ctl[3] = st_launch + 1; kv_publish_forward(a.kv, a.launch); }
      if (a.bump_step && a.step_dev) {
        const uint64_t nx = step - a.step + 1;
        ((int32_t*)a.step_dev)[0] = (int32_t)(uint32_t)nx;
        ((int32_t*)a.step_dev)[1] = (int32_t)(uint32_t)(nx >> 32);
      }
      a.kv.mirror[2 * a.kv.max_seqs] = st_err;
      a.kv.mirror[2 * a.kv.max_seqs + 1] = (int32_t)st_dev_err;
      if (st_dev_err) return;                              // the forward did not finish: its logits mean nothing, commit nothing
      const int new_len = st_len + st_npend + n;
      const int keep = ceil_div(new_len, a.kv.bt);
      if (a.B == 1) {
        int own = st_owned, top = st_top;
        while (own > keep) {
          --own;
          a.kv.free_stack[top++] = a.kv.table[seq * a.kv.mbps + own];
          a.kv.table[seq * a.kv.mbps + own] = -1;
        }
        a.kv.owned[seq] = own;
        a.kv.ctl[0] = top;
      }
      a.kv.len[seq] = new_len;
      a.kv.pend[seq * 2] = sh_tok;
      a.kv.n_pend[seq] = 1;
      a.kv.mirror[2 * seq] = new_len;
      a.kv.mirror[2 * seq + 1] = 1;
    }
    return;
  }
  // ---- commit by the last workgroup to arrive
  if (tid == 0) {
    __threadfence();
    const int arrived = atomicAdd(a.ticket, 1);
    sh_last = (arrived == a.B - 1);
  }
  __syncthreads();
  if (!sh_last) return;                                    // (the whole workgroup)
  __threadfence();
  const bool failed = *a.kv.err != 0;                      // the forward did not finish: commit nothing
  if (tid == 0) {
    *a.ticket = 0;
    if (a.launch) kv_bump_launch(a.kv, a.launch);
    if (a.bump_step && a.step_dev) {
      const uint64_t nx = step - a.step + 1;
      ((int32_t*)a.step_dev)[0] = (int32_t)(uint32_t)nx;
      ((int32_t*)a.step_dev)[1] = (int32_t)(uint32_t)(nx >> 32);
    }
    if (failed) kv_publish_flags(a.kv);
  }
  if (failed) return;
  __shared__ int c16[16];
  const bool in = tid < a.B;                               // one thread per sequence (at most MAX_ROWS = SBLOCK of them)
  const int sq = a.seq0 + (in ? tid : 0);
  const int nn = in && a.n_acc ? ((volatile int32_t*)a.n_acc)[tid] : 0;
  const int tok = in ? ((volatile int32_t*)a.next_tok)[(size_t)tid * a.tok_stride] : 0;
  kv_truncate_all(a.kv, in, sq, a.kv.len[sq] + a.kv.n_pend[sq] + nn, c16);
  if (in) {
    a.kv.pend[sq * 2] = tok;
    a.kv.n_pend[sq] = 1;
    kv_publish_seq(a.kv, sq);
  }
  if (tid == 0) kv_publish_flags(a.kv);
}

template <int SP>
__global__ void __launch_bounds__(SBLOCK) k_accept(AcceptArgs a) { accept_seq<SP>(a, blockIdx.x); }

// One row per sequence (a draft step, an autoregressive step): the row's distribution and the token drawn from it in
// one launch.  The probabilities go to memory (the caller wants the row) and, for the draw, through LDS (the halves
// assign elements to threads differently); the arithmetic is that of the two kernels above, bit for bit.
template <int SP>
__global__ void __launch_bounds__(SBLOCK) k_warp_accept(WarpArgs w, AcceptArgs a) {
  constexpr bool STAGE = SP <= 8;                           // 32 KB of LDS; the larger instantiation re-reads the row from memory
  __shared__ float row_probs[STAGE ? SP * SBLOCK : 1];
  float* lds_row = (STAGE && a.K == 0) ? row_probs : nullptr;   // K == 0: the row of the draw is the row just computed
  warp_softmax_row<SP>(w, blockIdx.x, lds_row);
  __threadfence_block();
  __syncthreads();
  accept_seq<SP>(a, blockIdx.x, lds_row);
}

// ------------------------------------------------------------------------------------------ small state kernels
// Truncate one sequence and (optionally) set its pending token from a value or from device memory.  new_len >= 0 is a
// rollback: a target beyond the cached length is refused (the state stays, KV_ERR_ROLLBACK is raised).  add_len is
// the commit of a prefill chunk.  after_forward (kv_publish_forward's `launch`): the kernel follows a forward on this cache (advances its launch number;
// commits nothing if that forward did not finish).
__global__ void __launch_bounds__(BLOCK) k_kv_set(KvView kv, int seq, int new_len, int add_len, int set_pending, int pending_value,
                                                  const int32_t* pending_ptr, uint32_t after_forward) {
  const int tid = threadIdx.x, len = kv.len[seq], own = kv.owned[seq], top = kv.ctl[0];
  const bool failed = *kv.err != 0, refused = new_len > len;
  const int target = new_len >= 0 ? new_len : len + add_len, keep = ceil_div(target, kv.bt);
  __syncthreads();                                         // every thread has read the state
  if (tid == 0 && after_forward) kv_bump_launch(kv, after_forward);
  if (failed || refused) {
    if (tid == 0) {
      if (!failed) kv.ctl[1] |= KV_ERR_ROLLBACK;
      kv_publish_flags(kv);
    }
    return;
  }
  int32_t* table = kv.table + (size_t)seq * kv.mbps;
  for (int i = keep + tid; i < own; i += BLOCK) {          // highest table index first onto the stack
    kv.free_stack[top + own - 1 - i] = table[i];
    table[i] = -1;
  }
  if (tid) return;
  if (own > keep) { kv.owned[seq] = keep; kv.ctl[0] = top + own - keep; }
  kv.len[seq] = target;
  if (set_pending) {
    kv.pend[seq * 2] = pending_ptr ? *pending_ptr : pending_value;
    kv.n_pend[seq] = 1;
  }
  kv_publish(kv, seq);
}

// Draft cache after a verification of K drafts (see ssd_kv_follow): one workgroup, one thread per sequence.
__global__ void k_kv_follow(KvView kv, int n_seqs, int K, const int32_t* n_acc, const int32_t* next_tok,
                            const int32_t* x, int32_t* step_dev, int replayed) {
  __shared__ int w16[16];
  const int s = threadIdx.x;
  if (step_dev && s == 0) {                                // last kernel of a captured cycle: the next replay is the next step
    const int32_t cycles = kv.ctl[6] + 1;
    const uint64_t nx = ((uint64_t)(uint32_t)step_dev[0] | ((uint64_t)(uint32_t)step_dev[1] << 32)) + 1;
    step_dev[0] = (int32_t)(uint32_t)nx;
    step_dev[1] = (int32_t)(uint32_t)(nx >> 32);
    if (replayed) {
      kv.ctl[6] = cycles;
      kv.mirror[2 * kv.max_seqs + MIRROR_CYCLE] = cycles;
    }
  }
  if (*kv.err) {
    if (s == 0) kv_publish_flags(kv);
    return;
  }
  const bool in = s < n_seqs;
  const int n = in ? n_acc[s] : 0, len = in ? kv.len[s] : 0;
  kv_truncate_all(kv, in, s, n < K ? len - (K - 1 - n) : len, w16);
  if (in) {
    kv.pend[s * 2] = n < K ? next_tok[s] : x[s * K + K - 1];
    if (n >= K) kv.pend[s * 2 + 1] = next_tok[s];
    kv.n_pend[s] = n < K ? 1 : 2;
    kv_publish_seq(kv, s);
  }
  if (s == 0) kv_publish_flags(kv);
}

__global__ void k_kv_init(KvView kv) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < kv.n_blocks) kv.free_stack[i] = kv.n_blocks - 1 - i;       // lowest id on top
  if (i < kv.max_seqs) {
    kv.len[i] = 0; kv.n_pend[i] = 0; kv.pend[2 * i] = 0; kv.pend[2 * i + 1] = 0; kv.owned[i] = 0;
    kv.mirror[2 * i] = 0; kv.mirror[2 * i + 1] = 0;
  }
  if (i < kv.max_seqs * kv.mbps) kv.table[i] = -1;
  if (i == 0) {
    kv.ctl[0] = kv.n_blocks; kv.ctl[1] = 0; kv.ctl[2] = 0; kv.ctl[3] = 1; kv.ctl[4] = 0; kv.ctl[5] = 0; kv.ctl[6] = 0;
    kv.mirror[2 * kv.max_seqs] = 0; kv.mirror[2 * kv.max_seqs + 1] = 0;
  }
}

// Clears the sticky error state (the caller has re-zeroed the barrier words and the barrier-free forward's workspace on the same stream)
// and restarts the launch numbering; sequence state is left as it is.
__global__ void k_kv_clear_error(KvView kv) {
  if (threadIdx.x || blockIdx.x) return;
  kv.ctl[1] = 0; kv.ctl[2] = 0; kv.ctl[3] = 1;
  *kv.err = 0u;
  kv_publish_flags(kv);
}

// Clears n 32-bit words (a kernel, not a memset: callers may be capturing the stream).
__global__ void k_zero_words(int32_t* p, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}

// Test hook: raise device error bits / set the launch number (see ssd_kv_test_hook).
__global__ void k_kv_poke(KvView kv, uint32_t err_bits, int launch_no) {
  if (threadIdx.x || blockIdx.x) return;
  if (err_bits) *kv.err = *kv.err | err_bits;
  if (launch_no > 0) kv.ctl[3] = launch_no;
}

// Rotary table: (cos, sin)(pos * base^(-2i/hd)) evaluated in fp64, rounded once to fp32.
__global__ void k_rope_table(float2* tab, int max_pos, int half, double base) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= max_pos * half) return;
  const int pos = i / half, f = i - pos * half;
  const double ang = (double)pos * pow(base, -(double)f / (double)half);
  tab[i] = make_float2((float)cos(ang), (float)sin(ang));
}

}  // namespace ssd
