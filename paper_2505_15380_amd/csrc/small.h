// The fp32 forward of a few rows as one launch: the phases of gemm.h's k_gemm_f32 and attention.h's k_attn_f32, with their bits, on workgroups that
// hand over to each other as dataflow.h describes (words that are zero while they are not there, two sets that launches take in turn).
//
// Three kinds of workgroups, three hand-overs a layer: a kv head of a sequence (its query, key and value projections, then attention), 32 columns of the
// SwiGLU output (the whole output projection of the rows first: at these widths every workgroup computes it sooner than it could be handed
// on), 32 columns of the down projection.  A workgroup keeps its item for the whole launch, so the weights of the next layer are requested while it
// waits, and a wave polls its operands straight into the registers that the matrix instructions read.  A wave's k-steps, the order of its
// products and of the waves' sums, and the walk over the keys are those of the two kernels: a row has the same bits whichever way computed it.
//
// What bounds it is one workgroup's chain: 0.7 to 1.5 us for a hand-over, 2.2 for the projections of a kv head, 3.4 for its attention (single waves issuing fp32
// matrix instructions and exponentials), 3 for the other two.  A cycle of the two models of widths 128 and 64 with four drafts, 64 positions: 188 us
// with one launch per operator, 47 launches; 136 with 12.  The line to the launches per operator is where a workgroup has a compute unit and an
// item to itself; a verification of 64 rows of the wider one takes 72 there and 52 here.
#pragma once
#include "attention.h"
#include "dataflow.h"

namespace ssd {

constexpr int SF_MAX_ROWS = 64;                            // rows of a launch
constexpr int SF_MAX_D = 256, SF_MAX_FFN = 512;            // inputs of a projection that four waves share, eight: at most four steps of 16 each
constexpr int SF_MAX_GROUP = 8;                            // query heads of a kv head
constexpr int SF_HD = 32, SF_HP = SF_HD + 4;               // head size; words from one row of a head to the next in LDS

struct SArgs {
  int n_layers, d, nq, nkv, ffn, vocab, n_embed;
  float eps, scale;
  const float* embed;
  const float* final_norm;
  const float* head;
  const float2* rope;
  PLayer layer0;
  size_t layer_stride;
  KvView kv;
  Rows rows;
  int pcap, n_seqs, tok_stride, with_head;
  const int32_t* tokens;
  uint32_t* tw;                 // two sets of words
  size_t st_set;                // words of a set: per layer [cap][attention | h after attention | SwiGLU | h after the MLP]
  int cap;                      // rows that the workspace has room for
  u64* state;                   // the last launch that has gone through its layers: its number, then (rows of the one before it << 16 | rows << 1 | set)
  u64* rowblk;                  // [SF_MAX_ROWS]
  float* logits;
  uint32_t* bar;
  int tiles, recip_tiles, recip_seqs, recip_T, recip_R, recip_G;         // attention's row tiles; 2^16 / it, / n_seqs, / row tiles, / rows, / heads of a group, rounded up
  int first_gu, first_down, first_end;   // workgroups: attention's from 0, gate / up's, the down projection's; at first_end the one that reserves blocks
};

// n / d for n d < 2^16 (a division is forty instructions, and the launch's first loads wait for it)
__device__ __forceinline__ int sf_div(int n, int recip) { return (int)((uint32_t)(n * recip) >> 16); }

// What a row needs of the cache's state, every candidate requested at once (one trip to memory instead of three in a row); none of it changes in the launch.
struct SfRow {
  int j, len, npend, p0, p1, tx;
  __device__ __forceinline__ SfRow(const SArgs& a, int m) {
    const int b = sf_div(m, a.recip_R), seq = a.rows.seq0 + b;
    j = m - b * a.rows.R;
    len = ld_state(a.kv.len + seq);
    npend = a.pcap ? ld_state(a.kv.n_pend + seq) : 0;
    p0 = a.pcap ? ld_state(a.kv.pend + seq * 2) : 0;
    p1 = a.pcap > 1 ? ld_state(a.kv.pend + seq * 2 + 1) : 0;
    tx = j >= a.pcap ? ld_state(a.tokens + (size_t)b * a.tok_stride + (j - a.pcap)) : 0;
  }
  __device__ __forceinline__ int token(const SArgs& a) const {
    const int off = a.pcap - npend, x0 = p0, x1 = p1, xt = tx, pend = j > off ? x1 : x0;
    return min(max(j < a.pcap ? pend : xt, 0), a.n_embed - 1);
  }
};

// The words of a layer's buffers.
struct SfWords {
  uint32_t *attn, *mid, *act, *out;
  __device__ __forceinline__ SfWords(const SArgs& a, uint32_t* set, int l) {
    const size_t c = a.cap, nqd = (size_t)a.nq * SF_HD;
    attn = set + (size_t)l * c * (nqd + 2 * a.d + a.ffn);
    mid = attn + c * nqd;
    act = mid + c * a.d;
    out = act + c * a.ffn;
  }
};

// Gives up after a while, or when another workgroup has.
__device__ __forceinline__ bool sf_give_up(long& spins, uint32_t* err) {
  if (++spins > DF_SPIN_LIMIT || ((spins & 63) == 0 && __hip_atomic_load(err, __ATOMIC_RELAXED, AG) != 0)) {
    __hip_atomic_store(err, 1u, __ATOMIC_RELAXED, AG);
    return true;
  }
  __builtin_amdgcn_s_sleep(1);
  return false;
}

// k-steps [kb, ke) of wave `wave` of the nw that share a projection of K inputs (see k_gemm_f32).
__device__ __forceinline__ void sf_steps(int K, int wave, int& nw, int& kb, int& ke) {
  const int steps = K >> 4;
  nw = min(GF_MAX_WAVES, max(4, (steps + 3) >> 2));
  const int per = steps / nw, rem = steps - per * nw;
  kb = wave * per + min(wave, rem);
  ke = kb + per + (wave < rem ? 1 : 0);
}
// (Through descriptors, here and below: a load is then an instruction and a scalar addition, not five.)
__device__ __forceinline__ f32x4 sf_ld(df_rsrc r, int lane_off, int off) { return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, lane_off, off, 0)); }
struct SfWeights { f32x4 x0[4], x1[4]; };
__device__ __forceinline__ void sf_weights(const void* W0, const void* W1, int N, int K, int t0, int t1, int kb, int ke, int lane, SfWeights& w) {
  const df_rsrc r0 = df_make_rsrc(W0), r1 = df_make_rsrc(W1);
  const int li = lane & 15, at = (lane >> 4) * 16, o0 = min(t0 * 16 + li, N - 1) * (4 * K) + at, o1 = min(t1 * 16 + li, N - 1) * (4 * K) + at;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    if (kb + u >= ke) break;                               // (scalar: a step more, of rows in 16 places each, costs its way through the L1)
    w.x0[u] = sf_ld(r0, o0, (kb + u) * 64);
    w.x1[u] = sf_ld(r1, o1, (kb + u) * 64);
  }
}
__device__ __forceinline__ void sf_gain(const float* gain, int kb, int ke, int lane, f32x4 (&g)[4]) {
  const df_rsrc r = df_make_rsrc(gain);
#pragma unroll
  for (int u = 0; u < 4; ++u)
    if (kb + u < ke) g[u] = sf_ld(r, (lane >> 4) * 16, (kb + u) * 64);
}

// A wave's operands: the four k of its lane group in each of its steps, of row `row` of the words A [..][K]; p0, p1: two more words of this thread (or
// null), awaited in the same polls.
__device__ __forceinline__ bool sf_poll(const uint32_t* A, int row, int K, int kb, int ke, int lane, u32x4 (&x)[4], const uint32_t* p0, const uint32_t* p1, float& h0, float& h1, uint32_t* err) {
  uint32_t b0 = 1u, b1 = 1u;
  if (p0) { b0 = ld_val(p0); b1 = ld_val(p1); }
  const df_rsrc rs = df_make_rsrc(A);
  uint32_t at = 4u * (uint32_t)(row * K + (lane >> 4) * 4);
  auto off = [&](int u) { return at + 64u * (uint32_t)(kb + u); };
  bool ok = true;
#pragma unroll
  for (int u = 0; u < 4; ++u) x[u] = kb + u < ke ? ld_words2(rs, off(u)) : u32x4{1u, 1u, 1u, 1u};
  for (long spins = 0;;) {
    bool late = min(b0, b1) == 0u;
#pragma unroll
    for (int u = 0; u < 4; ++u) late = late || df_any_zero(x[u]);
    if (!late) break;
    if (sf_give_up(spins, err)) { ok = false; break; }
    asm volatile("" : "+v"(at) : : "memory");              // (the words may have changed)
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (df_any_zero(x[u])) x[u] = ld_words2(rs, off(u));
    if (p0 && b0 == 0u) b0 = ld_val(p0);
    if (p0 && b1 == 0u) b1 = ld_val(p1);
  }
  h0 = __uint_as_float(b0);
  h1 = __uint_as_float(b1);
  return ok;
}

// A wave's products with two column tiles, with the gain of the norm before (k_gemm_f32's order); ss: the lane's sum of squares.
template <bool GAIN>
__device__ __forceinline__ void sf_products(const u32x4 (&x)[4], const SfWeights& w, const f32x4 (&gn)[4], int kb, int ke, float& ss, float (*red)[256], int lane) {
  f32x4 acc0 = {0, 0, 0, 0}, acc1 = {0, 0, 0, 0};
  ss = 0.f;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    if (kb + u >= ke) break;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      float y = __uint_as_float(x[u][j]);
      if (GAIN) { ss = fmaf(y, y, ss); y *= gn[u][j]; }
      acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(y, w.x0[u][j], acc0, 0, 0, 0);
      acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(y, w.x1[u][j], acc1, 0, 0, 0);
    }
  }
  const int o = (lane >> 4) * 64 + (lane & 15);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    red[0][o + 16 * r] = acc0[r];
    red[1][o + 16 * r] = acc1[r];
  }
}
__device__ __forceinline__ void sf_squares(float ss, float* red_ss, int lane) {
  ss += __shfl_xor(ss, 16, WAVE); ss += __shfl_xor(ss, 32, WAVE);
  if (lane < 16) red_ss[lane] = ss;
}
// The sums of the nw (<= NW) waves of an item, of a thread's row and column, in wave order.
template <int NW>
__device__ __forceinline__ void sf_sum(const float (*red)[2][256], int nw, int e, float& v0, float& v1) {
  float x[NW][2];
#pragma unroll
  for (int i = 0; i < NW; ++i) { x[i][0] = red[i][0][e]; x[i][1] = red[i][1][e]; }
  v0 = 0.f; v1 = 0.f;
#pragma unroll
  for (int i = 0; i < NW; ++i)
    if (i < nw) { v0 += x[i][0]; v1 += x[i][1]; }
}
__device__ __forceinline__ float sf_inv(const float (*red_ss)[16], int row, int K, float eps) {      // (of four waves)
  float x[4], tot = 0.f;
#pragma unroll
  for (int i = 0; i < 4; ++i) x[i] = red_ss[i][row];
#pragma unroll
  for (int i = 0; i < 4; ++i) tot += x[i];
  return 1.0f / sqrtf(tot / (float)K + eps);
}
// Bias and rotation, rounded where gemm_epilogue_f32 is (there the compiler makes these two fused operations of its expressions).
__device__ __forceinline__ void sf_bias_rotate(float& v0, float& v1, const float* bias, int n0, bool rotate, float2 cs) {
#pragma clang fp contract(off)
  if (bias) { v0 += bias[n0]; v1 += bias[n0 + SF_HD / 2]; }
  const float y0 = v1 * cs.y, y1 = v0 * cs.y, x0 = fmaf(v0, cs.x, -y0), x1 = fmaf(v1, cs.x, y1);
  if (rotate) { v0 = x0; v1 = x1; }
}
__device__ __forceinline__ float sf_scaled(float v, float inv) {
#pragma clang fp contract(off)
  return v * inv;
}

struct SfLds {
  float red[2][8][2][256];                                 // rounds take the two in turn: one barrier each
  float red_ss[8][16];
  union {
    struct { float po[8][16][SF_HP], pm[8][16], pl[8][16], q[SF_MAX_GROUP][16][SF_HP], kn[16][SF_HP], vn[16][SF_HP]; } at;
    float mid[16][SF_MAX_D + 4];
  };
  int dead;
};

// The keys and values of a wave's chunk, as they are in the pool (of a block that this launch reserves whatever is there: its positions come from LDS).
struct SfChunk { f32x4 k[4][2], v[2][4]; };
__device__ __forceinline__ void sf_blocks(const SArgs& a, int seq, int c, int (&blk)[4]) {
#pragma unroll
  for (int t = 0; t < 4; ++t) blk[t] = ld_state(a.kv.table + (size_t)seq * a.kv.mbps + min(c * 4 + t, a.kv.mbps - 1));
}
__device__ __forceinline__ void sf_load_chunk(const SArgs& a, int layer, int kvh, const int (&blk)[4], int lane, SfChunk& x) {
  const float* pool = (const float*)a.kv.pool;
  const df_rsrc rk = df_make_rsrc(pool + kv_offset(a.kv, layer, 0, 0, kvh, 0)), rv = df_make_rsrc(pool + kv_offset(a.kv, layer, 1, 0, kvh, 0));
  const int li = lane & 15, kg = lane >> 4, ko = li * (4 * SF_HD) + kg * 16, vo = li * 64 + kg * 16;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int id = min(max(__builtin_amdgcn_readfirstlane(blk[t]), 0), a.kv.n_blocks - 1) * (a.kv.nkv * 64 * SF_HD);      // (a plane has less than 2^31 bytes)
#pragma unroll
    for (int s = 0; s < 2; ++s) { x.k[t][s] = sf_ld(rk, ko + 64 * s, id); x.v[s][t] = sf_ld(rv, vo + 1024 * s, id); }
  }
}

// ---- A kv head of a sequence and 16 of its query rows.
__device__ __forceinline__ void sf_attention(const SArgs& a, uint32_t* set, uint32_t tag, const SfRow& mine, const int (&blk0)[4], int b, int kvh, int r0, SfLds& s) {
  constexpr int W = att_f32_waves<SF_HD>();
  static_assert(W == 8, "");
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), half = wave >> 2;
  const int G = a.nq / a.nkv, R = a.rows.R, nrows = R * G, m_first = b * R, seq = a.rows.seq0 + b, nqd = a.nq * SF_HD, N = nqd + 2 * a.nkv * SF_HD, items = G + 2;
  uint32_t* err = a.bar + 64;
  const int len = __builtin_amdgcn_readfirstlane(mine.len), off = a.pcap - __builtin_amdgcn_readfirstlane(mine.npend), nact = R - off, pos_max = len + nact - 1;
  auto pos_of = [&](int j) { return j < off ? len : len + (j - off); };
  int nw, kb, ke;
  sf_steps(a.d, wave & 3, nw, kb, ke);                     // (nw = 4)
  const int tok0 = mine.token(a);
  const int jq = sf_div(min(r0 + ((int)threadIdx.x & 15), nrows - 1), a.recip_G);        // the lane's query row: row of the sequence
  int blk = -1;
  for (int l = 0; l < a.n_layers; ++l) {
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));                          // (its parts are worked out again in each layer: there are no registers to keep them)
    const int lane = tid & 63, li = lane & 15, kg = lane >> 4, half_t = tid >> 8, m_lane = m_first + min(li, R - 1);
    const int e = tid & 255, row = e >> 4, col = e & 15;    // of an item's results
    const float2 cs = a.rope[(size_t)pos_of(min(row, R - 1)) * (SF_HD / 2) + col];
    const PLayer Y = layer_ptrs(a, l);
    const SfWords lw(a, set, l);
    auto head_of = [&](int i) { return i < G ? kvh * G + i : i == G ? a.nq + kvh : a.nq + a.nkv + kvh; };
    auto weights = [&](int rd, SfWeights& w) {
      const int h = head_of(min(2 * rd + half, items - 1));
      sf_weights(Y.wqkv, Y.wqkv, N, a.d, 2 * h, 2 * h + 1, kb, 2 * rd + half < items ? ke : kb, lane, w);
    };
    SfWeights wa, wb;
    f32x4 gn[4];
    weights(0, wa);
    sf_gain(Y.ln1, kb, ke, lane, gn);
    weights(1, wb);
    SfChunk x;
    if (wave * ATT_CHUNK <= pos_max) sf_load_chunk(a, l, kvh, blk0, lane, x);
    u32x4 A[4];
    float h0, h1;
    if (l == 0) {
#pragma unroll
      for (int u = 0; u < 4; ++u) A[u] = *(const u32x4*)(a.embed + (size_t)tok0 * a.d + (min(kb + u, ke - 1) * 4 + kg) * 4);
    } else if (!sf_poll(SfWords(a, set, l - 1).out, m_lane, a.d, kb, ke, lane, A, nullptr, nullptr, h0, h1, err)) {
      s.dead = 1;
    }
    float inv = 0.f;
    auto round = [&](int rd, const SfWeights& w) {
      float ss;
      sf_products<true>(A, w, gn, kb, ke, ss, s.red[rd & 1][wave], lane);
      if (rd == 0) sf_squares(ss, s.red_ss[wave], lane);
      __syncthreads();
      if (rd == 0) inv = sf_inv(s.red_ss, row, a.d, a.eps);
      const int i = 2 * rd + half_t, head = head_of(i);
      float v0, v1;
      sf_sum<4>(s.red[rd & 1] + 4 * half_t, 4, e, v0, v1);
      v0 = sf_scaled(v0, inv); v1 = sf_scaled(v1, inv);
      if (i >= items || row >= R) return;
      sf_bias_rotate(v0, v1, Y.bqkv, head * SF_HD + col, i <= G, cs);
      float* to = i < G ? s.at.q[i][row] : i == G ? s.at.kn[row] : s.at.vn[row];
      to[col] = v0;
      to[col + SF_HD / 2] = v1;
    };
    for (int rd = 0; 2 * rd < items; rd += 2) {
      if (rd) { weights(rd, wa); weights(rd + 1, wb); }
      round(rd, wa);
      if (2 * rd + 2 < items) round(rd + 1, wb);
    }
    __syncthreads();
    if (s.dead) return;
    const int gq = min(r0 + li, nrows - 1) - jq * G, pos = pos_of(jq);
    f32x4 q[2], o[2];
#pragma unroll
    for (int d = 0; d < 2; ++d) { q[d] = *(const f32x4*)&s.at.q[gq][jq][d * 16 + kg * 4]; o[d] = f32x4{0, 0, 0, 0}; }
    float mrow = -INFINITY, lrow = 0.f;
    for (int c = wave; c * ATT_CHUNK <= pos_max; c += W) {
      const int p0 = c * ATT_CHUNK, nt = min(4, ((pos_max - p0) >> 4) + 1);      // blocks that any row sees: the others' weights are 0
      if (c != wave) {
        int ids[4];
        sf_blocks(a, seq, c, ids);
        sf_load_chunk(a, l, kvh, ids, lane, x);
      }
      if (p0 + ATT_CHUNK > len) {                          // this launch's positions among them
        // (all of them are read, and taken where they are: reads behind conditions of their own wait one for another)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          if (t >= nt || p0 + 16 * t + 15 < len) continue;
          const int jn = p0 + 16 * t + li - len;
          const bool is = (unsigned)jn < (unsigned)nact;
          const int at = off + min(max(jn, 0), nact - 1);
#pragma unroll
          for (int d = 0; d < 2; ++d) {
            const f32x4 y = *(const f32x4*)&s.at.kn[at][d * 16 + kg * 4];
#pragma unroll
            for (int r = 0; r < 4; ++r) x.k[t][d][r] = is ? y[r] : x.k[t][d][r];
          }
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int je = p0 + 16 * t + kg * 4 + r - len;
            const bool ie = (unsigned)je < (unsigned)nact;
            const int ae = off + min(max(je, 0), nact - 1);
#pragma unroll
            for (int d = 0; d < 2; ++d) {
              const float y = s.at.vn[ae][d * 16 + li];
              x.v[d][t][r] = ie ? y : x.v[d][t][r];
            }
          }
        }
      }
      f32x4 wt[4];
      float mx = mrow;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        wt[t] = f32x4{0, 0, 0, 0};
        if (t >= nt) continue;
#pragma unroll
        for (int d = 0; d < 2; ++d)
#pragma unroll
          for (int r = 0; r < 4; ++r) wt[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(x.k[t][d][r], q[d][r], wt[t], 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          wt[t][r] = p0 + t * 16 + kg * 4 + r <= pos ? wt[t][r] * a.scale : -INFINITY;
          mx = fmaxf(mx, wt[t][r]);
        }
      }
      mx = fmaxf(mx, __shfl_xor(mx, 16, WAVE));
      mx = fmaxf(mx, __shfl_xor(mx, 32, WAVE));
      const float base = mx == -INFINITY ? 0.f : mx;
      const float keep = expf(mrow - base);
      float sum = 0.f;
#pragma unroll
      for (int t = 0; t < 4; ++t)
        if (t < nt)
#pragma unroll
          for (int r = 0; r < 4; ++r) { wt[t][r] = expf(wt[t][r] - base); sum += wt[t][r]; }
      sum += __shfl_xor(sum, 16, WAVE);
      sum += __shfl_xor(sum, 32, WAVE);
      lrow = lrow * keep + sum;
      mrow = mx;
#pragma unroll
      for (int d = 0; d < 2; ++d) o[d] *= keep;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        if (t >= nt) continue;
        if (p0 + 16 * t + 15 > pos_max)                    // what lies beyond may never have been written
#pragma unroll
          for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int d = 0; d < 2; ++d) x.v[d][t][r] = p0 + t * 16 + kg * 4 + r <= pos_max ? x.v[d][t][r] : 0.f;
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int d = 0; d < 2; ++d) o[d] = __builtin_amdgcn_mfma_f32_16x16x4f32(x.v[d][t][r], wt[t][r], o[d], 0, 0, 0);
      }
    }
#pragma unroll
    for (int d = 0; d < 2; ++d) *(f32x4*)&s.at.po[wave][li][d * 16 + kg * 4] = o[d];
    if (kg == 0) { s.at.pm[wave][li] = mrow; s.at.pl[wave][li] = lrow; }
    __syncthreads();
    if (tid < 16 * (SF_HD / 4) && r0 + (tid >> 3) < nrows) {
      const int r = tid >> 3, d = (tid & 7) * 4, j = sf_div(r0 + r, a.recip_G);
      float mx = -INFINITY, den = 0.f;
#pragma unroll
      for (int y = 0; y < W; ++y) mx = fmaxf(mx, s.at.pm[y][r]);
      f32x4 acc = {0, 0, 0, 0};
#pragma unroll
      for (int y = 0; y < W; ++y) {
        const float f = expf(s.at.pm[y][r] - mx);
        den = fmaf(s.at.pl[y][r], f, den);
        acc += *(const f32x4*)&s.at.po[y][r][d] * f;
      }
      acc /= den;
      df_put_partial(df_make_rsrc(lw.attn), 4u * (uint32_t)((m_first + j) * nqd + (kvh * G + r0 + r - j * G) * SF_HD + d), acc);
    }
    // ---- the new keys and values into the cache, behind everything that somebody waits for: row and dim of this thread
    if (r0 == 0) {
      const int j = tid >> 5, d = tid & 31;
      if (j >= off && j < R) {
        if (l == 0) {
          u64 w = ld_word(a.rowblk + m_first + j);
          for (long spins = 0; (uint32_t)(w >> 32) != tag; w = ld_word(a.rowblk + m_first + j))
            if (sf_give_up(spins, err)) { w = 0xFFFFFFFFull; break; }
          blk = (int)(uint32_t)w;
        }
        if (blk >= 0) {
          float* pool = (float*)a.kv.pool;
          const int tok = pos_of(j) & 15;
          pool[kv_offset(a.kv, l, 0, blk, kvh, 0) + tok * SF_HD + d] = s.at.kn[j][d];
          pool[kv_offset(a.kv, l, 1, blk, kvh, 0) + d * 16 + tok] = s.at.vn[j][d];
        }
      }
    }
    __syncthreads();
  }
}

// ---- 32 columns of the SwiGLU output of 16 rows, behind the whole output projection of these rows; then columns of the head.
__device__ __forceinline__ void sf_gate_up(const SArgs& a, uint32_t* set, const SfRow& mine, int item, int m0, bool first, int i, int n, SfLds& s) {
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), li = lane & 15, kg = lane >> 4, half = wave >> 2, half_t = tid >> 8;
  const int M = a.rows.M, L = a.n_layers, T = (M + 15) >> 4, nqd = a.nq * SF_HD, pairs = a.d >> 5;
  const int e = tid & 255, row = e >> 4, col = e & 15, m = m0 + row;
  uint32_t* err = a.bar + 64;
  int nw, kb, ke, kbo, keo;
  sf_steps(nqd, wave & 3, nw, kbo, keo);                   // (nw = 4 for both)
  sf_steps(a.d, wave & 3, nw, kb, ke);
  const int kbp = kbo < keo ? kbo : 0, kep = kbo < keo ? keo : 1;      // a wave without a step awaits attention all the same: it reads what that depends on
  const int m_lane = min(m0 + li, M - 1);
  const float* er = a.embed + (size_t)mine.token(a) * a.d;
  const f32x4 none[4] = {};
  u32x4 A[4];
  float h0, h1;
  for (int l = 0; l < L; ++l) {
    const PLayer Y = layer_ptrs(a, l);
    const SfWords lw(a, set, l);
    const uint32_t* res = l ? SfWords(a, set, l - 1).out + (size_t)m * a.d : nullptr;       // the residual stream that enters the layer
    SfWeights wa, wb, wg;
    f32x4 gn[4];
    auto weights = [&](int rd, SfWeights& w) {
      const int p = min(2 * rd + half, pairs - 1);
      sf_weights(Y.wo, Y.wo, a.d, nqd, 2 * p, 2 * p + 1, kbo, 2 * rd + half < pairs ? keo : kbo, lane, w);
    };
    weights(0, wa);
    weights(1, wb);
    const int g16 = min(2 * item + half, (a.ffn >> 4) - 1);
    sf_weights(Y.wgate, Y.wup, a.ffn, a.d, g16, g16, kb, ke, lane, wg);
    sf_gain(Y.ln2, kb, ke, lane, gn);
    // the residual rows (long there once a word of attention is: it depends on the whole row)
    uint32_t ra[2], rb[2];
    auto residual = [&](int rd, uint32_t (&r)[2]) {
      const int n0 = 32 * min(2 * rd + half_t, pairs - 1) + col;
      r[0] = r[1] = 1u;
      if (m >= M) return;
      if (res) { r[0] = ld_val(res + n0); r[1] = ld_val(res + n0 + 16); }
      else { r[0] = __float_as_uint(er[n0]); r[1] = __float_as_uint(er[n0 + 16]); }
    };
    if (!res) { residual(0, ra); residual(1, rb); }
    const uint32_t* first_res = res && m < M ? res + 32 * min(half_t, pairs - 1) + col : nullptr;
    if (!sf_poll(lw.attn, m_lane, nqd, kbp, kep, lane, A, first_res, first_res ? first_res + 16 : nullptr, h0, h1, err)) s.dead = 1;
    if (res) { ra[0] = __float_as_uint(h0); ra[1] = __float_as_uint(h1); residual(1, rb); }
    auto round = [&](int rd, const SfWeights& w, const uint32_t (&r)[2]) {
      const int p = 2 * rd + half_t, n0 = 32 * p + col;
      float ss;
      sf_products<false>(A, w, none, kbo, keo, ss, s.red[rd & 1][wave], lane);
      const float r0 = __uint_as_float(r[0]), r1 = __uint_as_float(r[1]);
      __syncthreads();
      float v0, v1;
      sf_sum<4>(s.red[rd & 1] + 4 * half_t, 4, e, v0, v1);
      if (p >= pairs) return;
      v0 = r0 + v0;
      v1 = r1 + v1;
      s.mid[row][n0] = v0;
      s.mid[row][n0 + 16] = v1;
      if (first && m < M) {                                // the residual of the down projection
        uint32_t* to = lw.mid + (size_t)m * a.d;
        st_val(to + n0, float_word(v0));
        st_val(to + n0 + 16, float_word(v1));
      }
    };
    int rounds = 0;
    for (int rd = 0; 2 * rd < pairs; rd += 2) {
      if (rd) { weights(rd, wa); weights(rd + 1, wb); residual(rd, ra); residual(rd + 1, rb); }
      round(rd, wa, ra);
      ++rounds;
      if (2 * rd + 2 < pairs) { round(rd + 1, wb, rb); ++rounds; }
    }
    __syncthreads();
    if (s.dead) return;
#pragma unroll
    for (int u = 0; u < 4; ++u) A[u] = *(const u32x4*)&s.mid[li][(min(kb + u, ke - 1) * 4 + kg) * 4];
    float ss;
    sf_products<true>(A, wg, gn, kb, ke, ss, s.red[rounds & 1][wave], lane);
    sf_squares(ss, s.red_ss[wave], lane);
    __syncthreads();
    const float inv = sf_inv(s.red_ss, row, a.d, a.eps);
    float v0, v1;
    sf_sum<4>(s.red[rounds & 1] + 4 * half_t, 4, e, v0, v1);
    v0 = sf_scaled(v0, inv); v1 = sf_scaled(v1, inv);
    const int n0 = (2 * item + half_t) * 16 + col;
    if (m < M && n0 < a.ffn) st_val(lw.act + (size_t)m * a.ffn + n0, float_word(v0 / (1.0f + expf(-v0)) * v1));
    __syncthreads();
  }
  if (!a.with_head) return;
  const SfWords lw(a, set, L - 1);
  const int heads = (a.vocab + 31) >> 5, hp = (heads + 1) >> 1;          // items of 32 columns; two to a workgroup
  for (int x = i; x < hp * T; x += n) {
    const int t = x / hp, h = 2 * (x - t * hp) + half, ht = 2 * (x - t * hp) + half_t, mm = t * 16 + row, c0 = ht * 32 + col;
    SfWeights w;
    f32x4 gn[4];
    sf_weights(a.head, a.head, a.vocab, a.d, 2 * h, 2 * h + 1, kb, ke, lane, w);
    sf_gain(a.final_norm, kb, ke, lane, gn);
    if (!sf_poll(lw.out, min(t * 16 + li, M - 1), a.d, kb, ke, lane, A, nullptr, nullptr, h0, h1, err)) s.dead = 1;
    float ss;
    sf_products<true>(A, w, gn, kb, ke, ss, s.red[0][wave], lane);
    sf_squares(ss, s.red_ss[wave], lane);
    __syncthreads();
    if (s.dead) return;
    const float inv = sf_inv(s.red_ss, row, a.d, a.eps);
    float v0, v1;
    sf_sum<4>(s.red[0] + 4 * half_t, 4, e, v0, v1);
    v0 = sf_scaled(v0, inv); v1 = sf_scaled(v1, inv);
    if (mm < M) {
      float* lo = a.logits + (size_t)mm * a.vocab;
      if (c0 < a.vocab) lo[c0] = v0;
      if (c0 + 16 < a.vocab) lo[c0 + 16] = v1;
    }
    __syncthreads();
  }
}

// ---- 32 columns of the down projection of 16 rows.
__device__ __forceinline__ void sf_down(const SArgs& a, uint32_t* set, int item, int m0, SfLds& s) {
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), M = a.rows.M;
  const int e = tid & 255, m = m0 + (e >> 4), n0 = item * 32 + (e & 15);
  const bool mine = tid < 256 && m < M;
  int nw, kb, ke;
  sf_steps(a.ffn, wave, nw, kb, ke);                       // (nw <= 8)
  const f32x4 none[4] = {};
  for (int l = 0; l < a.n_layers; ++l) {
    const SfWords lw(a, set, l);
    float h0 = 0.f, h1 = 0.f;
    if (wave < nw) {
      const PLayer Y = layer_ptrs(a, l);
      SfWeights w;
      sf_weights(Y.wdown, Y.wdown, a.d, a.ffn, 2 * item, 2 * item + 1, kb, ke, lane, w);
      const uint32_t* res = mine ? lw.mid + (size_t)m * a.d + n0 : nullptr;
      u32x4 A[4];
      if (!sf_poll(lw.act, min(m0 + (lane & 15), M - 1), a.ffn, kb, ke, lane, A, res, res ? res + 16 : nullptr, h0, h1, a.bar + 64)) s.dead = 1;
      float ss;
      sf_products<false>(A, w, none, kb, ke, ss, s.red[l & 1][wave], lane);
    }
    __syncthreads();
    if (s.dead) return;
    if (!mine) continue;
    float v0, v1;
    sf_sum<8>(s.red[l & 1], nw, e, v0, v1);
    uint32_t* to = lw.out + (size_t)m * a.d + n0;
    st_val(to, float_word(h0 + v0));
    st_val(to + 16, float_word(h1 + v1));
  }
}

__global__ void __launch_bounds__(PBLOCK) k_forward_f32(SArgs a) {
  __shared__ __attribute__((aligned(16))) SfLds s;
  const int tid = threadIdx.x, wg = blockIdx.x;
  if (tid == 0) s.dead = 0;
  const int M = a.rows.M, L = a.n_layers, T = (M + 15) >> 4;
  const int tag_v = ld_state(a.kv.ctl + 3);
  const u64 state_v = ld_word(a.state);
  if (wg == a.first_end) {
    df_reserve_blocks(a, tag_v, true);
    return;
  }
  // which item this is, and what of the cache's state it needs: one trip to memory with the two above
  const bool att = wg < a.first_gu;
  const int at_t = sf_div(wg, a.recip_tiles), at_kvh = sf_div(at_t, a.recip_seqs), b = at_t - at_kvh * a.n_seqs;
  const int gu = max(wg - a.first_gu, 0), gu_item = sf_div(gu, a.recip_T), gu_m0 = (gu - gu_item * T) * 16;
  const SfRow mine(a, att ? b * a.rows.R + min(tid & 15, a.rows.R - 1) : min(gu_m0 + ((tid & 255) >> 4), M - 1));
  int blk[4] = {0, 0, 0, 0};
  if (att) sf_blocks(a, a.rows.seq0 + b, tid >> 6, blk);
  const uint32_t tag = (uint32_t)__builtin_amdgcn_readfirstlane(tag_v);
  if (!df_tag_ok(tag)) {                                   // numbering exhausted: do nothing; the host must clear the workspace
    if (wg == 0 && tid == 0) __hip_atomic_fetch_or(a.bar + 64, DEV_ERR_TAGS, __ATOMIC_RELAXED, AG);
    return;
  }
  const uint32_t last_tag = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)state_v), last = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(state_v >> 32));
  const uint32_t which = last_tag == tag ? last & 1u : ~last & 1u;
  // (The state may already be this launch's: with several row tiles its last layer does not depend on the workgroups of the others, and one that begins
  // only now still has its share of the launch before to zero.)
  const int old_rows = (int)(last_tag == tag ? last >> 16 : (last & 0xFFFFu) >> 1);
  uint32_t* set = a.tw + which * a.st_set;
  __syncthreads();
  if (att) {
    sf_attention(a, set, tag, mine, blk, b, at_kvh, (wg - at_t * a.tiles) * 16, s);
    // The words that the launch before left in its set become zeros, by the workgroups whose item is not the launch's last.
    uint32_t* old = a.tw + (which ^ 1u) * a.st_set;
    auto zero = [&](uint32_t* p, int words) {
      const df_rsrc r = df_make_rsrc(p);
      for (int x = (wg * PBLOCK + tid) * 4; x < words; x += a.first_gu * PBLOCK * 4) __builtin_amdgcn_raw_buffer_store_b128(u32x4{0u, 0u, 0u, 0u}, r, x * 4, 0, 16 /* sc1 */);
    };
    for (int l = 0; l < L && old_rows; ++l) {
      const SfWords ow(a, old, l);
      zero(ow.attn, old_rows * a.nq * SF_HD);
      zero(ow.mid, old_rows * a.d);
      zero(ow.act, old_rows * a.ffn);
      zero(ow.out, old_rows * a.d);
    }
  } else if (wg < a.first_down) {
    sf_gate_up(a, set, mine, gu_item, gu_m0, gu_item == 0, gu, a.first_down - a.first_gu, s);
  } else {
    const int i = wg - a.first_down, item = sf_div(i, a.recip_T);
    sf_down(a, set, item, (i - item * T) * 16, s);
    if (wg == a.first_down && tid == 0) __hip_atomic_store(a.state, (u64)tag | (u64)((uint32_t)old_rows << 16 | (uint32_t)M << 1 | which) << 32, __ATOMIC_RELAXED, AG);
  }
}

}  // namespace ssd
