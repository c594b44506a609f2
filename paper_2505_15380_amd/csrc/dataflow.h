// The decoder forward of one verification (Eq. 4) as one persistent kernel WITHOUT grid barriers between phases.
//
// Phases per layer: QKV (+bias, rotary, cache append) -> attention (in parts, then their merge, for long prefixes)
// -> output projection (+residual) -> MLP (gate/up + SwiGLU + down projection fused inside a workgroup) -> sum of the
// MLP partials (+residual).  Weights are packed as matrix-core fragments; a unit of 4 waves takes an item.
//
// Dependent phases are ordered by the data itself: everything a workgroup hands to another workgroup is made of 4-byte words that are
// zero while they are not there.  A value that is zero goes out as -0, as an operand with the upper half -0, or with a bit beside it:
// the same value to whoever reads it.  Words are stored and loaded with agent-scope accesses, up to four with one instruction past the same caches; a
// consumer repeats the loads that brought a zero.  A word is observed whole, so one that is not zero is the payload.  No
// store has to be acknowledged before a flag is raised, no counter is shared, and a dependency costs one store plus one load instead of the
// chain of memory round trips of a barrier.  (With a tag beside every word, a launch number to compare, nothing had to be zeroed, but
// the bytes were twice as many, and they are what a hand-over waits for: per layer 5 rows 17.6 -> 16.3 us without them, 9 rows 20.7 -> 18.8, one
// row 14.3 -> 13.8; in the partials of the MLP alone, 11 MB a layer with five rows, another 1.5 and 4.)
//
// Every word is written once per launch: each layer and phase has its own buffers.  There are two sets of them, which launches take in
// turn; while it waits, a launch zeroes the rows that the last one left in the other set.  Launches on one cache workspace are ordered by the
// stream, so a launch finds its set zero.  Which set is its own, and how many rows the other has, it reads from a word that the last launch left.
// The MLP's partials, ffn/32 per output, are too many to wait for the next launch: the workgroup that has summed one puts the zero
// back, and two buffers take the layers in turn.  The zeros of layer l have reached memory before their workgroup publishes its sums of layer
// l + 1; an MLP item of layer l + 2 begins after operands that depend on all of those; so no zero overtakes a partial, and a partial
// that is not zero is this layer's.  A launch whose wait times out leaves words behind; the workspace is cleared before the cache is used again.
//
// Two kinds of words are 8 bytes {payload, tag}, the tag being the launch's number: the attention's partial results, for which
// the workspace has room by the longest context and which few launches use, and the blocks of the new keys.  They need no zeros.  For a 64-bit access
// the memory model promises that a word is observed whole.  That each aligned 8-byte half of a 16-byte access is whole as well is a property
// of this hardware, where a lane's 16 bytes are one piece of one cache line in every request.
//
// Payloads: a GEMM operand value x is hi | lo << 16 with hi = upper 16 bits of x and lo = bf16(x - hi) (the two
// bf16 whose sum the matrix core consumes); residual rows, sums of squares and partial results are fp32 bits; new
// keys / values are bf16 bits.
//
// A workgroup stages the operand rows it needs in LDS once (all its threads poll in parallel, four words of each of 2, 4, 6, 8
// or 10 rows in flight: the kernel is instantiated for SB = 2, 4, 10, 16, 18 and the host picks the smallest that holds the launch's rows in one
// flight, 18 for more) and feeds the matrix cores from LDS.  The weights of an item are requested at the entry of its phase, into
// registers, before that wait: workgroups arrive at a phase before its operands do, so the wait hides the HBM latency.
// The phases with few items (QKV, attention, output projection) run on workgroups of their own, beyond those that
// take the MLP items, so that no workgroup is late for the MLP, the phase every workgroup waits for.
// Polling costs fabric bandwidth that the producers' stores need: a wave whose first flight fails first watches a
// single word with long sleeps, and polls in earnest only from then on.
//
// Attention never reads this launch's new keys from the cache pool: the QKV phase stores them in the pool for
// later launches and, as words, in a side buffer; a wave whose 64-key chunk reaches the new positions patches its key
// fragments from that buffer at the same slots the pool would have supplied, and its values in LDS, through which that
// chunk's go.  A row's bits do not depend on how many rows are verified together.
//
// There is no grid barrier: phase 0 (row bookkeeping, embedding, block reservation) hands over like every other phase.
// All waits are bounded; a timeout raises the error word and every workgroup leaves; the kernel that follows the
// forward then commits nothing and copies the word to the host-mapped mirror, where the next call on the cache finds it.
//
// The launch number is not a kernel argument: it is read from the cache's control words, and the kernel that follows
// every forward on the stream advances it, so a captured graph of launches can be replayed.
#pragma once
#include "persistent.h"

namespace ssd {

typedef unsigned long long u64;
constexpr int DF_ATT_ROWS = 256;          // query rows of a sequence (rows x heads of a group): at most 16 tiles of 16
constexpr int DF_NPF = 5;                 // attention parts merged per flight
constexpr long DF_SPIN_LIMIT = 1L << 18;
// LDS words: staging | sums of squares | unit reduction buffers, overlaid by the attention buffers of the two units
constexpr int DF_SQ_WORDS = 1024;
constexpr int DF_RED_WORDS = 2 * 2048;
constexpr int DF_QS = 68;                 // words from one row to the next of the queries and of the merge buffers in LDS: rows 64
                                          // words apart would put a fragment's 16 rows into the same banks
// The two forms of the kernel: head size 64 (k_forward_dataflow), and 128 for wider models (k_forward_wide).
struct DfNarrow {
  static constexpr bool WIDE = false;
  static constexpr int HD = 64, HDL = 6, NH = 1;   // head size, its logarithm, and in how many pieces of 64 dims the attention's output is taken
  static constexpr int PF = PF_K;         // k-tiles of weights a wave of a unit keeps requested
  static constexpr int XB = PF_K;         // k-tiles whose operands it reads from LDS at once
  static constexpr int AW = 21504;        // LDS words of the operand staging area (84 KB)
  static constexpr int QW = DF_QS;        // words from one row of the queries to the next in LDS
  static constexpr int DN = 7;            // down-projection output tiles a wave keeps prefetched
  static constexpr int ACT_PITCH = 36;    // words from one row of a workgroup's SwiGLU output to the next
  static constexpr int TR = AW + DF_SQ_WORDS + DF_RED_WORDS;                        // the MLP's partials on their way out: per wave [8 rows][DN tiles][16]
  static constexpr int KN = 16 * QW, VN = KN + 512, MO = VN + 512, MO_WAVE = 16 * DF_QS, ML = MO + 8 * MO_WAVE, V2 = ML + 256;   // Q | new K | new V | merge O | merge m,l |
  static constexpr int ATT_WORDS = V2 + 8 * 2048;                                   // values of a chunk per wave
  static constexpr int LDS_WORDS = TR + 8 * 8 * DN * 16;
  static constexpr int AW8 = AW, RS = AW + DF_SQ_WORDS;
};
// Head size 128.  28 layers of width 1536 behind 1024 positions, against one launch per operator, seven a layer: one row 1316 -> 636 us, five 1349 -> 743, eight
// 1376 -> 840, thirteen 1408 -> 1146.  Bound by the weights, 94 MB a layer: the registers and LDS of the MLP's 140 workgroups hold 70 of them while they wait, the
// rest streams when their operands are there.  Every wave has 12 k-tiles of width 1536 in flight (96 registers) and 12 tiles of the down projection (48).
// The MLP's partials go out over the staged operands, which nothing reads any more, and a wave's share of attention over the values that it has read.
struct DfWide {
  static constexpr bool WIDE = true;
  static constexpr int HD = 128, HDL = 7, NH = 2, PF = 12, XB = 2, AW = 16 * 1540, QW = 132, DN = 12, ACT_PITCH = 68, TR = 0;
  static constexpr int MAX_K = 4 * 32 * PF;                // inputs of a projection: a wave keeps all of its k-tiles requested
  static constexpr int KN = 16 * QW, VN = KN + 1024, ML = VN + 512, V2 = ML + 256, MO = V2, MO_WAVE = 4096;                     // Q | new K | new V (64 dims) | merge m,l |
  static constexpr int ATT_WORDS = V2 + 8 * 4096;                                                                               // values of two chunks per wave, then merge O
  static constexpr int LDS_WORDS = 37952;
  static constexpr int AW8 = 8 * 1540, RS = AW8 + DF_SQ_WORDS;           // operands of up to 8 rows; where sum tasks meet
};
static_assert(DfNarrow::ATT_WORDS <= DfNarrow::LDS_WORDS && DfNarrow::LDS_WORDS <= 39 * 1024, "");
// The staging area of an instantiation, and how many of a wave's tiles of the down projection the wide form has in LDS behind it and what it is followed by.
template <int SB, class S>
constexpr int df_aw() { return SB <= 16 ? S::AW8 : S::AW; }
template <int SB, class S>
constexpr int df_wl() { return df_aw<SB, S>() + DF_SQ_WORDS + DF_RED_WORDS; }
template <int SB>
constexpr int df_lds_tiles() { return SB <= 16 ? 10 : 0; }
static_assert(DfWide::ATT_WORDS <= DfWide::LDS_WORDS && 8 * 8 * DfWide::DN * 16 <= DfWide::AW8 && DfWide::LDS_WORDS <= 39 * 1024 &&
              df_wl<16, DfWide>() + df_lds_tiles<16>() * 2048 <= DfWide::LDS_WORDS && df_wl<18, DfWide>() + df_lds_tiles<18>() * 2048 <= DfWide::LDS_WORDS, "");
template <int PF>
struct DfPre { u32x4 b0[PF], b1[PF]; };   // weight fragments of a wave's first PF k-tiles, two tiles

// Which single word a wave watches after a failed first flight (see df_wait_hint): the phases with many consumers (QKV, attention, MLP)
// watch a word of their OWN operands, the output projection one of the preceding phase's.  (The MLP watching a word of the phase before: one row
// 1.1 us a layer more, nine rows 2.4; QKV so 1.5 and 1.1; attention so 1.0 at nine rows of 4096 positions, where 40 workgroups
// polled beside the ones they waited for.  The output projection watching its own: one row 0.15 more.)
constexpr int DF_HINT_SLEEP = 2;

struct DArgs {
  int n_layers, d, nq, nkv, ffn, vocab, n_embed;
  float eps, scale;
  const bf16_t* embed;
  const float* final_norm;
  const void* head;
  const float2* rope;
  PLayer layer0;
  size_t layer_stride;
  KvView kv;
  Rows rows;
  int pcap, n_seqs, tok_stride, with_head;
  const int32_t* tokens;
  uint32_t* tw;           // base of the workspace; the members below, up to the parts, point into the first of its two sets
  uint32_t* h;            // [2L+1][PR][d]      fp32: residual stream entering layer l at 2l, after attention at 2l+1
  uint32_t* hg;           // [2L+1][PR][d]      operand: h times the gain of the RMSNorm that consumes it
  uint32_t* sq;           // [2L+1][PR][d/8]    fp32: sums of squares of h over 32 columns (after the MLP: over df_sq_cols columns)
  uint32_t* q;            // [L][PR][nq*HD]     operand: rotated queries (HD: head size)
  uint32_t* kvn;          // [L][PR][2][nkv*HD] bf16 (| 1 << 16): this launch's keys (rotated) and values
  uint32_t* attn;         // [L][PR][nq*HD]     operand: attention output
  size_t st_set;          // words from one set to the other
  u64* state;             // the last launch: its number, then (rows << 1 | set)
  u64* att_p;             // [L][PR][nq][NP][HD/4][6] fp32: per part and 4-dim chunk: 4 weighted values, max, sum
  float* part;            // [2][row][d/C][ffn/32][C]: down-projection partials of one 32-column slice of the SwiGLU output each (buffer =
                          // layer parity; C = df_sum_cols, 8 take the room of 16).  What a sum task reads is contiguous: with a
                          // row per workgroup, 112 KB apart, its pieces and all workgroups' stores fell on few memory channels
  size_t st_part;
  u64* rowblk;            // [16] per row: the pool block that takes the row's new key and value (-1: none), from the reservation
  float* logits;
  size_t st_h, st_sq, st_q, st_kvn, st_att_p;   // strides in words
  int NP, n_parts;        // parts that the workspace has room for, and that this launch has workgroups for
  int g_mlp;              // workgroups [0, g_mlp) take the MLP items; the phases with few items start on the workgroups after them
  int small_stride;       // 2: a small-phase item has a workgroup to itself; 1: two items per workgroup
  uint32_t* bar;          // [64] error flag (sticky until the host reads it); [0], [32] belong to the kernel with grid barriers
  unsigned long long* trace;
  // the wide form
  int o_stride;           // small_stride of the output projection's items
  int mlp_tiles;          // k-tiles of the down projection (32 columns of the SwiGLU output) that an MLP workgroup takes
  int n_sum;              // partials of an output of the down projection
  int recip_d, recip_q;   // 2^16 / pieces of 512 words in a row of d or nq * HD words, rounded up
};

// Tagged words.
__device__ __forceinline__ u64 ld_word(const u64* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, AG); }
__device__ __forceinline__ void st_word(u64* p, uint32_t payload, uint32_t tag) {
  __hip_atomic_store(p, (u64)payload | ((u64)tag << 32), __ATOMIC_RELAXED, AG);
}
// Words without a tag, zero while they are not there, and the forms that are never zero.
__device__ __forceinline__ uint32_t ld_val(const uint32_t* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, AG); }
__device__ __forceinline__ void st_val(uint32_t* p, uint32_t bits) { __hip_atomic_store(p, bits, __ATOMIC_RELAXED, AG); }
__device__ __forceinline__ void st_val2(uint32_t* p, uint32_t x0, uint32_t x1) { __hip_atomic_store((u64*)p, (u64)x0 | ((u64)x1 << 32), __ATOMIC_RELAXED, AG); }     // (8-byte aligned)
__device__ __forceinline__ uint32_t float_word(float x) { return __float_as_uint(x) ? __float_as_uint(x) : 0x80000000u; }
// Two consecutive tagged words (16-byte aligned) with one store: a word is still stored by one instruction, and each has its tag.  (The
// s_nop: store data of more than 8 bytes must not be overwritten by the next two vector instructions.)
__device__ __forceinline__ void st_words2(u64* p, uint32_t x0, uint32_t x1, uint32_t tag) {
  const u32x4 a = {x0, tag, x1, tag};
  asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" ::"v"(p), "v"(a) : "memory");
}
__device__ __forceinline__ uint32_t split_payload(float x) {
  const uint32_t u = __float_as_uint(x), h = u & 0xFFFF0000u;
  return (h >> 16) | ((uint32_t)f_to_bf16(x - __uint_as_float(h)) << 16);
}
__device__ __forceinline__ uint32_t operand_word(float x) {
  const uint32_t p = split_payload(x);
  return p ? p : 0x8000u;
}
__device__ __forceinline__ bool df_any_zero(const u32x4 x) { return min(min(x[0], x[1]), min(x[2], x[3])) == 0u; }

// A workgroup that arrives at a phase long before its operands would poll them the whole time, and the polls of all
// such workgroups load the fabric that the producers' stores travel through.  After a first failed flight a wave
// therefore watches one word (see DF_HINT_SLEEP) with a single address and long sleeps, and resumes the full polling when that
// word is there.  Purely a hint: bounded, and nothing depends on what it saw.
__device__ __forceinline__ void df_wait_hint(const uint32_t* word, uint32_t* err) {
  for (int i = 0; i < (1 << 14); ++i) {
    if (ld_val(word) != 0u) return;
    if ((i & 63) == 63 && __hip_atomic_load(err, __ATOMIC_RELAXED, AG) != 0) return;
    __builtin_amdgcn_s_sleep(DF_HINT_SLEEP);
  }
}

// Two consecutive words with one 16-byte agent-scope load; `off`: bytes from the descriptor's base.
typedef __amdgpu_buffer_rsrc_t df_rsrc;
__device__ __forceinline__ df_rsrc df_make_rsrc(const void* base) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)base, (short)0, (int)0xFFFFFFE0u, 0x00027000);
}
__device__ __forceinline__ u32x4 ld_words2(df_rsrc r, uint32_t off) { return __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 16 /* sc1 */); }

// Loads the pairs of words at off(at, i) (bytes; ~0: none) until every tag is this launch's.  False on a timeout.  (Offsets are worked out again
// from `at` for a repeated load instead of being kept in registers.)
template <int N, typename OFF>
__device__ __forceinline__ bool poll_pairs(df_rsrc r, uint32_t at, OFF off, uint32_t tag, u32x4 (&v)[N], uint32_t* err) {
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = off(at, i) != 0xFFFFFFFFu ? ld_words2(r, off(at, i)) : u32x4{0u, tag, 0u, tag};
  long spins = 0;
  for (;;) {
    bool all = true;
#pragma unroll
    for (int i = 0; i < N; ++i) all = all && v[i][1] == tag && v[i][3] == tag;
    if (all) return true;
    if (++spins > DF_SPIN_LIMIT || ((spins & 63) == 0 && __hip_atomic_load(err, __ATOMIC_RELAXED, AG) != 0)) {
      __hip_atomic_store(err, 1u, __ATOMIC_RELAXED, AG);
      return false;
    }
    __builtin_amdgcn_s_sleep(1);
    asm volatile("" : "+v"(at) : : "memory");              // (the words may have changed)
#pragma unroll
    for (int i = 0; i < N; ++i)
      if (v[i][1] != tag || v[i][3] != tag) v[i] = ld_words2(r, off(at, i));
  }
}

// Loads four untagged words each at off(at, i) until all are there.  False on a timeout.
template <int N, typename OFF>
__device__ __forceinline__ bool poll_quads(df_rsrc r, uint32_t at, OFF off, u32x4 (&v)[N], uint32_t* err, const uint32_t* hint) {
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = off(at, i) != 0xFFFFFFFFu ? ld_words2(r, off(at, i)) : u32x4{1u, 1u, 1u, 1u};
  for (long spins = 0;;) {
    bool late = false;
#pragma unroll
    for (int i = 0; i < N; ++i) late = late || df_any_zero(v[i]);
    if (!late) return true;
    if (spins == 0) df_wait_hint(hint, err);
    if (++spins > DF_SPIN_LIMIT || ((spins & 63) == 0 && __hip_atomic_load(err, __ATOMIC_RELAXED, AG) != 0)) {
      __hip_atomic_store(err, 1u, __ATOMIC_RELAXED, AG);
      return false;
    }
    __builtin_amdgcn_s_sleep(1);
    asm volatile("" : "+v"(at) : : "memory");              // (the words may have changed)
#pragma unroll
    for (int i = 0; i < N; ++i)
      if (df_any_zero(v[i])) v[i] = ld_words2(r, off(at, i));
  }
}

// Columns of a task of df_reduce_phase, and of a sum of squares that it publishes.
template <int SB>
constexpr int df_sum_cols() { return SB == 2 ? 8 : SB <= 10 ? 32 : 64; }
template <int SB>
constexpr int df_sq_cols() { return SB == 2 ? 8 : 32; }
// Wide form (SB = 4, 16, 18): loads of four words a thread has in flight, of 512-word pieces dealt out to four quarters of a workgroup: 2, 8 and 16 rows of 1536.
template <int SB>
constexpr int df_flight() { return SB == 4 ? 2 : SB == 16 ? 6 : 12; }

// ------------------------------------------------------------------------------------------------ GEMM phases
struct DPhase {
  const uint32_t* A;           // operand rows [PR][K]
  const uint32_t* sq;          // [PR][K/32] sums of squares of the un-gained rows (nullptr: no RMSNorm)
  const void* W0;
  const void* W1;
  int N, K, gs, items;    // gs: k-splits, always 1 here (the field the shared k-range helper reads)
  int shift, stride;      // item i of round 0 runs on unit (shift + stride * i) % units
  const uint32_t* hint;        // the word to watch while there is nothing (see df_wait_hint), or null
  int layer;
  const float* bias;
  const uint32_t* h_in;        // PE_RESID: residual input and outputs
  uint32_t* h_out;
  uint32_t* hg_out;
  uint32_t* sq_out;
  const float* gain_next;
  uint32_t* out;               // PE_QKV: q
  uint32_t* kvn;               // PE_QKV: side buffer of the new keys / values
  float* logits;          // PE_LOGITS
};

// Every request of this thread that the compiler knows of has come back.  Its own waits count requests, stores among them, but not the
// stores of st_words2; where it believes that some path has left a register with a request pending, it waits for a count that those
// stores have grown past, which is a wait for their acknowledgement: 0.8 us and more behind the MLP's.  So each phase says, where its operands
// are there and before it stores, that nothing is pending, on every path (with five rows the sums' operands are there 0.3 us earlier).
__device__ __forceinline__ void df_loads_done() { __builtin_amdgcn_s_waitcnt(0x0F70); }   // vmcnt(0)

// Operand words of rows [0, M) (K words each, the rows contiguous) -> As, and the rows' sums of squares [M][nsq] -> sqs.  In As a
// row has K + 4 words: of every eight consecutive k the hi halves (four words), then the lo halves, as the matrix core takes them.  (With the words
// as they come a lane read both halves of its operand and picked one: twice the LDS reads, which took 900 cycles of a phase, and eight
// permutations a k-tile.)  The whole workgroup polls in parallel, four words per load, a row per half of it.  What bounds it are a thread's
// instructions and the bytes, so a thread has the same columns of every second row: a row's place is then one scalar offset for the load and one
// sum for the LDS write, and rows that are not there are skipped by scalar branches.  Of eight waves an eighth idles at 896 columns.  (With the
// words dealt out over all threads as they lie, each request has a row to find and a limit to keep: five rows 0.8 us a layer more, nine rows
// 1.6, one row 0.2.)  Lanes without words are masked out: a load costs the cycles of its return path even where all its lanes are out of
// range (five rows 513 -> 543 us with such loads instead of the mask).  A thread's first sum of squares rides in the flight, and so do, RES, two
// more words (x0, x1, or null) that come back in xo0, xo1; whatever is late is asked for again together, so that
// nothing costs a round trip of its own after the operands.  (Watching a word per producer first, and requesting the
// operands once all of them are there, saves polls but adds that round trip: 0.8 us a layer more with one row, 0.9 with five or nine.)
template <int SB, bool RES>
__device__ __forceinline__ bool stage_operand(const DArgs& a, const uint32_t* A, int K, const uint32_t* sq, int nsq, uint32_t* As, float* sqs, int tid,
                                              const uint32_t* x0, const uint32_t* x1, float& xo0, float& xo1, const uint32_t* hint) {
  constexpr int SP = SB == 4 ? 2 : (SB + 3) / 4;           // rows in flight of each half of the workgroup
  const int M = a.rows.M, nS = sq ? M * nsq : 0;
  const df_rsrc rs = df_make_rsrc(a.tw);
  const uint32_t a_off = (uint32_t)(A - a.tw) * 4u;
  const int half = __builtin_amdgcn_readfirstlane(tid >> 8), c = tid & 255;
  uint32_t* err = a.bar + 64;
  bool ok = true;
  auto give_up = [&](long& spins) -> bool {
    if (spins == 0 && hint) df_wait_hint(hint, err);                   // far too early: wait cheaply
    if (++spins > DF_SPIN_LIMIT || ((spins & 63) == 0 && __hip_atomic_load(err, __ATOMIC_RELAXED, AG) != 0)) {
      __hip_atomic_store(err, 1u, __ATOMIC_RELAXED, AG);
      ok = false;
      return true;
    }
    __builtin_amdgcn_s_sleep(1);
    return false;
  };
  uint32_t w = 1u, h0 = 1u, h1 = 1u;
  if (!RES && tid < nS) w = ld_val(sq + tid);
  if (RES && x0) {
    h0 = ld_val(x0);
    h1 = ld_val(x1);
  }
  for (int c0 = 0; c0 < K >> 2; c0 += 256)
    for (int r0 = 0; r0 < M; r0 += 2 * SP) {
      const bool on = c0 + c < K >> 2;
      uint32_t at = (uint32_t)(c0 + c) * 16u;
      auto row = [&](int u) { return r0 + 2 * u + half; };
      auto request = [&](int u) -> u32x4 {
        return __builtin_amdgcn_raw_buffer_load_b128(rs, (int)at, (int)(a_off + (uint32_t)(row(u) * K) * 4u), 16 /* sc1 */);
      };
      u32x4 v[SP];
#pragma unroll
      for (int u = 0; u < SP; ++u) v[u] = on && row(u) < M ? request(u) : u32x4{1u, 1u, 1u, 1u};
      for (long spins = 0;;) {
        bool late = RES ? min(h0, h1) == 0u : w == 0u;
#pragma unroll
        for (int u = 0; u < SP; ++u) late = late || df_any_zero(v[u]);
        if (!late || give_up(spins)) break;
        asm volatile("" : "+v"(at) : : "memory");          // (the words may have changed)
#pragma unroll
        for (int u = 0; u < SP; ++u)
          if (df_any_zero(v[u])) v[u] = request(u);
        if (!RES && w == 0u) w = ld_val(sq + tid);
        if (RES && h0 == 0u) h0 = ld_val(x0);
        if (RES && h1 == 0u) h1 = ld_val(x1);
      }
      df_loads_done();
      if (on) {
        uint32_t* to = As + (r0 + half) * (K + 4) + 4 * (c0 + c) - 2 * (c & 1);
#pragma unroll
        for (int u = 0; u < SP; ++u)
          if (row(u) < M) {
            *(uint2*)(to + 2 * u * (K + 4)) = make_uint2(__builtin_amdgcn_perm(v[u][1], v[u][0], 0x05040100u), __builtin_amdgcn_perm(v[u][3], v[u][2], 0x05040100u));
            *(uint2*)(to + 2 * u * (K + 4) + 4) = make_uint2(__builtin_amdgcn_perm(v[u][1], v[u][0], 0x07060302u), __builtin_amdgcn_perm(v[u][3], v[u][2], 0x07060302u));
          }
      }
    }
  if (!RES) {
    if (tid < nS) sqs[tid] = __uint_as_float(w);
    for (int i = PBLOCK + tid; i < nS; i += PBLOCK) {      // (more than 512 sums)
      w = ld_val(sq + i);
      for (long spins = 0; w == 0u && !give_up(spins);) w = ld_val(sq + i);
      sqs[i] = __uint_as_float(w);
    }
  }
  if (RES) {
    xo0 = __uint_as_float(h0);
    xo1 = __uint_as_float(h1);
  }
  return ok;
}

// The same for the wide form, whose rows are longer than half a workgroup takes at once: the words are dealt out as pieces of 512, and each
// quarter of the workgroup takes every fourth of them, so that all rows of a launch are in one flight (five rows of width 1536: 15 pieces, four loads a
// thread).  A piece's place is scalar arithmetic, as above.
template <int FL, bool RES>
__device__ __forceinline__ bool stage_operand_wide(const DArgs& a, const uint32_t* A, int K, const uint32_t* sq, int nsq, uint32_t* As, float* sqs, int tid,
                                                   const uint32_t* x0, const uint32_t* x1, float& xo0, float& xo1, const uint32_t* hint) {
  const int M = a.rows.M, nS = sq ? M * nsq : 0, per_row = (K + 511) >> 9, pieces = M * per_row, recip = K == a.d ? a.recip_d : a.recip_q;
  const df_rsrc rs = df_make_rsrc(a.tw);
  const uint32_t a_off = (uint32_t)(A - a.tw) * 4u;
  const int quarter = __builtin_amdgcn_readfirstlane(tid >> 7), c = (tid & 127) * 4;
  uint32_t* err = a.bar + 64;
  bool ok = true;
  auto give_up = [&](long& spins) -> bool {
    if (spins == 0 && hint) df_wait_hint(hint, err);
    if (++spins > DF_SPIN_LIMIT || ((spins & 63) == 0 && __hip_atomic_load(err, __ATOMIC_RELAXED, AG) != 0)) {
      __hip_atomic_store(err, 1u, __ATOMIC_RELAXED, AG);
      ok = false;
      return true;
    }
    __builtin_amdgcn_s_sleep(1);
    return false;
  };
  uint32_t w = 1u, h0 = 1u, h1 = 1u;
  if (!RES && tid < nS) w = ld_val(sq + tid);
  if (RES && x0) {
    h0 = ld_val(x0);
    h1 = ld_val(x1);
  }
  int p0 = quarter;
  do {                                                     // (a quarter without a piece, one or two in all, still awaits its threads' residual words)
    auto row = [&](int u) { return (p0 + 4 * u) * recip >> 16; };      // (exact: fewer than 2^8 pieces)
    auto col = [&](int u) { return (p0 + 4 * u - row(u) * per_row) * 512; };
    uint32_t at = (uint32_t)c * 4u;
    auto request = [&](int u) -> u32x4 {
      return __builtin_amdgcn_raw_buffer_load_b128(rs, (int)at, (int)(a_off + (uint32_t)(row(u) * K + col(u)) * 4u), 16 /* sc1 */);
    };
    u32x4 v[FL];
#pragma unroll
    for (int u = 0; u < FL; ++u) v[u] = p0 + 4 * u < pieces && col(u) + c < K ? request(u) : u32x4{1u, 1u, 1u, 1u};
    for (long spins = 0;;) {
      bool late = RES ? min(h0, h1) == 0u : w == 0u;
#pragma unroll
      for (int u = 0; u < FL; ++u) late = late || df_any_zero(v[u]);
      if (!late || give_up(spins)) break;
      asm volatile("" : "+v"(at) : : "memory");            // (the words may have changed)
#pragma unroll
      for (int u = 0; u < FL; ++u)
        if (df_any_zero(v[u])) v[u] = request(u);
      if (!RES && w == 0u) w = ld_val(sq + tid);
      if (RES && h0 == 0u) h0 = ld_val(x0);
      if (RES && h1 == 0u) h1 = ld_val(x1);
    }
    df_loads_done();
#pragma unroll
    for (int u = 0; u < FL; ++u)
      if (p0 + 4 * u < pieces && col(u) + c < K) {
        uint32_t* to = As + row(u) * (K + 4) + col(u) + c - ((c & 4) >> 1);
        *(uint2*)to = make_uint2(__builtin_amdgcn_perm(v[u][1], v[u][0], 0x05040100u), __builtin_amdgcn_perm(v[u][3], v[u][2], 0x05040100u));
        *(uint2*)(to + 4) = make_uint2(__builtin_amdgcn_perm(v[u][1], v[u][0], 0x07060302u), __builtin_amdgcn_perm(v[u][3], v[u][2], 0x07060302u));
      }
    p0 += 4 * FL;
  } while (p0 < pieces);
  if (!RES) {
    if (tid < nS) sqs[tid] = __uint_as_float(w);
    for (int i = PBLOCK + tid; i < nS; i += PBLOCK) {      // (more than 512 sums)
      w = ld_val(sq + i);
      for (long spins = 0; w == 0u && !give_up(spins);) w = ld_val(sq + i);
      sqs[i] = __uint_as_float(w);
    }
  }
  if (RES) {
    xo0 = __uint_as_float(h0);
    xo1 = __uint_as_float(h1);
  }
  return ok;
}
template <int SB, class S, bool RES>
__device__ __forceinline__ bool df_stage(const DArgs& a, const uint32_t* A, int K, const uint32_t* sq, int nsq, uint32_t* As, float* sqs, int tid,
                                         const uint32_t* x0, const uint32_t* x1, float& xo0, float& xo1, const uint32_t* hint) {
  if constexpr (S::WIDE) return stage_operand_wide<df_flight<SB>(), RES>(a, A, K, sq, nsq, As, sqs, tid, x0, x1, xo0, xo1, hint);
  else return stage_operand<SB, RES>(a, A, K, sq, nsq, As, sqs, tid, x0, x1, xo0, xo1, hint);
}

// hi / lo fragments (8 consecutive k each) of a lane from 8 staged payload words
__device__ __forceinline__ void split_words(const u32x4 w0, const u32x4 w1, u32x4& hi, u32x4& lo) {
  hi = u32x4{__builtin_amdgcn_perm(w0[1], w0[0], 0x05040100u), __builtin_amdgcn_perm(w0[3], w0[2], 0x05040100u),
             __builtin_amdgcn_perm(w1[1], w1[0], 0x05040100u), __builtin_amdgcn_perm(w1[3], w1[2], 0x05040100u)};
  lo = u32x4{__builtin_amdgcn_perm(w0[1], w0[0], 0x07060302u), __builtin_amdgcn_perm(w0[3], w0[2], 0x07060302u),
             __builtin_amdgcn_perm(w1[1], w1[0], 0x07060302u), __builtin_amdgcn_perm(w1[3], w1[2], 0x07060302u)};
}
__device__ __forceinline__ void frag_from_lds(const uint32_t* p, u32x4& hi, u32x4& lo) {
  split_words(*(const u32x4*)p, *(const u32x4*)(p + 4), hi, lo);
}

// Clock samples per workgroup and phase, only in builds with -DSSD_TRACE (see ssd_trace_barriers).
#ifdef SSD_TRACE
#define DF_STAMP(slot) do { if (a.trace && threadIdx.x == 0) a.trace[(size_t)blockIdx.x * 512 + (slot)] = wall_clock64(); } while (0)
#define DF_STAMP2(k) do { if (a.trace && threadIdx.x == 0) a.trace[(size_t)blockIdx.x * 512 + 256 + (slot - 2) / 10 * 10 + (k)] = wall_clock64(); } while (0)
#else
#define DF_STAMP(slot) do { } while (0)
#define DF_STAMP2(k) do { } while (0)
#endif

// Item of round 0 that `unit` takes when items start at unit `shift` and take every `stride`-th unit (stride 2: one
// item per workgroup, its other unit idles, so the item's waves have their SIMDs to themselves); a huge number where none.
__device__ __forceinline__ int df_item_of_unit(int unit, int shift, int NU, int stride = 1) {
  int i = unit - shift;
  if (i < 0) i += NU;
  if (stride == 2) return (i & 1) ? 0x3FFFFFFF : (i >> 1);
  return i;
}

// Products of a wave's k-tiles [kb, ke) with two weight tiles (the first PF_K k-tiles' weights are in wl) into acc0, acc1: element
// (r, lane) = (row 4 g + r, column lane % 16).  The hi and the lo halves of the operands have a sum each, which meet at the
// end.  Up to 8 rows (PACK) one instruction takes both: rows 0 .. 7 of its operand are the hi halves, 8 .. 15 the lo halves, and
// the sums meet across the wave's halves (df_meet: what does not need them comes in between); only rows 0 .. 7 of the result mean anything then.  Half the matrix and half the
// unpacking instructions: gate / up of one row 1.0 -> 0.7 us of a layer, QKV 1.6 -> 1.2.
template <bool PACK, class S>
__device__ __forceinline__ void df_products(const uint32_t* As, int K, int M, int kb, int ke, int lane, const DfPre<S::PF>& wl, const u32x4* w0,
                                            const u32x4* w1, f32x4& acc0, f32x4& acc1) {
  // (lanes of rows that are not there take the last one: what they yield is never looked at)
  const uint32_t* p = As + min(PACK ? lane & 7 : lane & 15, M - 1) * (K + 4) + (lane >> 4) * 8 + (PACK ? (lane & 8) >> 1 : 0);
  f32x4 lo0 = f32x4{0, 0, 0, 0}, lo1 = f32x4{0, 0, 0, 0};
  constexpr int XB = S::XB;
#define DF_MULTIPLY(X, Y, B0, B1)                                                                                            \
  {                                                                                                                          \
    const bf16x8 bv0 = __builtin_bit_cast(bf16x8, B0), bv1 = __builtin_bit_cast(bf16x8, B1), fx = __builtin_bit_cast(bf16x8, X); \
    if (!PACK) {                                                                                                             \
      const bf16x8 fl = __builtin_bit_cast(bf16x8, Y);                                                                       \
      lo0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fl, bv0, lo0, 0, 0, 0);                                                  \
      lo1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fl, bv1, lo1, 0, 0, 0);                                                  \
    }                                                                                                                        \
    acc0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fx, bv0, acc0, 0, 0, 0);                                                  \
    acc1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fx, bv1, acc1, 0, 0, 0);                                                  \
  }
#pragma unroll
  for (int u0 = 0; u0 < S::PF; u0 += XB) {
    // all operand fragments first (their LDS latencies overlap), then the products; in the wide form some at a time, there are no registers for all
    u32x4 x[XB], y[XB];                                    // hi and lo halves (PACK: the lane's one of them)
#pragma unroll
    for (int u = 0; u < XB; ++u) {
      const int kt = min(kb + u0 + u, ke - 1);
      x[u] = *(const u32x4*)(p + kt * 32);
      if (!PACK) y[u] = *(const u32x4*)(p + kt * 32 + 4);
    }
#pragma unroll
    for (int u = 0; u < XB; ++u)
      if (kb + u0 + u < ke) DF_MULTIPLY(x[u], y[u], wl.b0[u0 + u], wl.b1[u0 + u])
    if (S::WIDE) __builtin_amdgcn_sched_barrier(0);        // (or the reads of all of them are put first)
  }
  for (int kt = S::WIDE ? ke : kb + S::PF; kt < ke; ++kt) {          // waves with more than PF k-tiles (wide: none have)
    const u32x4 xk = *(const u32x4*)(p + kt * 32), yk = PACK ? xk : *(const u32x4*)(p + kt * 32 + 4);
    const u32x4 b0 = __builtin_nontemporal_load(w0 + (size_t)kt * 64), b1 = __builtin_nontemporal_load(w1 + (size_t)kt * 64);
    DF_MULTIPLY(xk, yk, b0, b1)
  }
#undef DF_MULTIPLY
  if (!PACK) {
    acc0 += lo0;
    acc1 += lo1;
  }
}
template <bool PACK>
__device__ __forceinline__ void df_meet(f32x4& acc0, f32x4& acc1) {
  if (PACK) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(acc0[r]), __float_as_uint(acc0[r]), false, false);
      const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(acc1[r]), __float_as_uint(acc1[r]), false, false);
      acc0[r] = __uint_as_float(a[0]) + __uint_as_float(a[1]);
      acc1[r] = __uint_as_float(b[0]) + __uint_as_float(b[1]);
    }
  }
}
// Rows that the products' PACK form takes; the instantiations for few words in flight use it.
template <int SB>
constexpr bool df_pack() { return SB <= 16; }
constexpr int DF_PACK_ROWS = 8;

// Column tiles of an item: of QKV the tiles of 16 columns that a rotation pairs, of the others two consecutive ones.
template <int EPI, class S, typename PH>
__device__ __forceinline__ bool df_gemm_item(const PH& ph, int item, int& t0, int& t1, int& split) {
  if (!S::WIDE || EPI != PE_QKV) return gemm_item<EPI>(ph, item, t0, t1, split);
  t0 = 0; t1 = 0; split = 0;
  if (item >= ph.items) return false;
  t0 = (item >> 2) * 8 + (item & 3);
  t1 = t0 + 4;
  return true;
}

// One GEMM phase (QKV, output projection, head); the caller skips it for a workgroup none of whose units has an
// item.  The weight fragments of the unit's item are requested at entry, into registers, before the wait for the
// operands: units arrive well before their operands do, so the weights' HBM latency is hidden by that wait.
// Returns true if the workgroup has to leave (timeout somewhere in the grid).
template <int EPI, int SB, class S>
__device__ __forceinline__ bool df_gemm_phase(const DArgs& a, const DPhase& ph, uint32_t* lds, const int* srow, int* sdead,
                                              int slot) {
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int usel = wave >> 2, uw = wave & 3, ut = tid & 255;
  const int unit = blockIdx.x * 2 + usel, NU = gridDim.x * 2;
  const int uitem = df_item_of_unit(unit, ph.shift, NU, ph.stride);
  uint32_t* As = lds;
  float* sqs = (float*)(lds + df_aw<SB, S>());
  float (*red)[2][256] = (float (*)[2][256])((float*)(lds + df_aw<SB, S>() + DF_SQ_WORDS) + usel * 2048);
  const int M = a.rows.M;
  const int KT = ph.K >> 5, ntiles = (ph.N + 15) >> 4;
  const int g = lane >> 4;
  const int row = ut >> 4, col = ut & 15;
  const int rounds = (ph.items + NU - 1) / NU;
  for (int rd = 0; rd < rounds; ++rd) {
    const int item = rd * NU + uitem;
    int t0, t1, split, kb = 0, ke = 0;
    const bool valid = df_gemm_item<EPI, S>(ph, item, t0, t1, split);
    if (valid) wave_krange(ph, 0, uw, kb, ke);
    const bool has1 = t1 < ntiles;
    const bool live = valid && row < M;
    const int n0 = t0 * 16 + col, n1 = t1 * 16 + col;
    const u32x4* w0 = (const u32x4*)ph.W0 + (size_t)t0 * KT * 64 + lane;
    const u32x4* w1 = (const u32x4*)ph.W1 + (size_t)(has1 ? t1 : t0) * KT * 64 + lane;
    DfPre<S::PF> wl;
    if (valid) {
#pragma unroll
      for (int u = 0; u < S::PF; ++u) {
        const int kt = (kb + u < ke) ? kb + u : kb;
        wl.b0[u] = __builtin_nontemporal_load(w0 + (size_t)kt * 64);
        wl.b1[u] = __builtin_nontemporal_load(w1 + (size_t)kt * 64);
      }
    }
    // ---- epilogue operands that do not depend on the product: requested with the weights
    float bias0 = 0.f, bias1 = 0.f, gn0 = 0.f, gn1 = 0.f;
    float2 cs = float2{1.f, 0.f};
    int pos = 0, active = 0, rblk = -1;
    if (EPI == PE_QKV && live) {
      if (ph.bias) { bias0 = ph.bias[n0]; bias1 = ph.bias[n0 + S::HD / 2]; }
      pos = srow[row]; active = srow[16 + row]; rblk = srow[32 + row];
      cs = a.rope[(size_t)pos * (S::HD / 2) + (n0 & (S::HD - 1))];
    }
    if (EPI == PE_RESID && live) { gn0 = ph.gain_next[n0]; gn1 = ph.gain_next[n1]; }
    // ---- operands (both units of the workgroup consume the same rows); the unit that finishes residual rows takes
    //      its residual inputs in the same flight
    const bool res = EPI == PE_RESID && live;
    const uint32_t *hx0 = res ? ph.h_in + (size_t)row * ph.N + n0 : nullptr, *hx1 = res ? ph.h_in + (size_t)row * ph.N + n1 : nullptr;
    float hv0 = 0.f, hv1 = 0.f;
    bool ok = true;
    if (rd == 0) ok = df_stage<SB, S, EPI == PE_RESID>(a, ph.A, ph.K, ph.sq, ph.K / df_sq_cols<SB>(), As, sqs, tid, hx0, hx1, hv0, hv1, ph.hint);
    if (!ok) *sdead = 1;
    __syncthreads();
    df_loads_done();
    if (*sdead) return true;
    if (rd == 0) DF_STAMP(slot);
    // ---- products
    f32x4 acc0 = f32x4{0, 0, 0, 0}, acc1 = f32x4{0, 0, 0, 0};
    if (valid) df_products<df_pack<SB>(), S>(As, ph.K, M, kb, ke, lane, wl, w0, w1, acc0, acc1);
    float inv = 1.0f;                                      // (while the matrix cores work)
    if (ph.sq) {
      float sq = 0.f;
      if (row < M)                                         // sums over 32 columns, as the halves of df_reduce_phase's tree
        for (int p = col; p < KT; p += 16) {
          if (df_sq_cols<SB>() == 8) {
            const f32x4 q = *(const f32x4*)(sqs + (row * KT + p) * 4);
            sq += (q[0] + q[1]) + (q[2] + q[3]);
          } else {
            sq += sqs[row * KT + p];
          }
        }
      inv = 1.0f / sqrtf(row16_sum(sq) / (float)ph.K + a.eps);
    }
    df_meet<df_pack<SB>()>(acc0, acc1);
    const int obase = (g * 4) * 16 + (lane & 15);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      red[uw][0][obase + r * 16] = acc0[r];
      red[uw][1][obase + r * 16] = acc1[r];
    }
    __syncthreads();
    float v0 = (red[0][0][ut] + red[1][0][ut]) + (red[2][0][ut] + red[3][0][ut]);
    float v1 = (red[0][1][ut] + red[1][1][ut]) + (red[2][1][ut] + red[3][1][ut]);
    if (ph.sq) { v0 *= inv; v1 *= inv; }
    if (EPI == PE_QKV) {
      if (live) {
        const int head = n0 >> S::HDL, dd = n0 & (S::HD - 1);          // dd < HD / 2
        v0 += bias0; v1 += bias1;
        if (head < a.nq + a.nkv) {
          const float r0 = v0 * cs.x - v1 * cs.y, r1 = v1 * cs.x + v0 * cs.y;
          v0 = r0; v1 = r1;
        }
        if (head < a.nq) {
          uint32_t* qo = ph.out + (size_t)row * (a.nq * S::HD) + head * S::HD + dd;
          st_val(qo, operand_word(v0));
          st_val(qo + S::HD / 2, operand_word(v1));
        } else {
          const int which = head < a.nq + a.nkv ? 0 : 1;
          const int kvh = head - a.nq - which * a.nkv;
          const bf16_t b0 = f_to_bf16(v0), b1 = f_to_bf16(v1);
          uint32_t* ko = ph.kvn + ((size_t)row * 2 + which) * (a.nkv * S::HD) + kvh * S::HD + dd;
          st_val(ko, b0 | 0x10000u);
          st_val(ko + S::HD / 2, b1 | 0x10000u);
          if (active && rblk >= 0) {
            bf16_t* base = (bf16_t*)a.kv.pool + kv_offset(a.kv, ph.layer, which, rblk, kvh, 0);
            const int tok = pos & 15;
            if (which == 0) { st_ag(base + tok * S::HD + dd, b0); st_ag(base + tok * S::HD + dd + S::HD / 2, b1); }
            else { st_ag(base + dd * 16 + tok, b0); st_ag(base + (dd + S::HD / 2) * 16 + tok, b1); }
          }
        }
      }
    } else if (EPI == PE_LOGITS) {
      if (live) {
        if (n0 < ph.N) ph.logits[(size_t)row * ph.N + n0] = v0;
        if (has1 && n1 < ph.N) ph.logits[(size_t)row * ph.N + n1] = v1;
      }
    } else {  // PE_RESID: N == d (a multiple of 32): residual, and the operand / statistics of the next RMSNorm
      if (valid) {
        const int pair = t0 >> 1;
        float q2 = 0.f;
        if (row < M) {
          v0 += hv0;
          v1 += hv1;
          st_val(ph.h_out + (size_t)row * ph.N + n0, float_word(v0));
          st_val(ph.h_out + (size_t)row * ph.N + n1, float_word(v1));
          st_val(ph.hg_out + (size_t)row * ph.N + n0, operand_word(v0 * gn0));
          st_val(ph.hg_out + (size_t)row * ph.N + n1, operand_word(v1 * gn1));
          q2 = v0 * v0 + v1 * v1;
        }
        q2 = row16_sum(q2);
        if (col == 0 && row < M) st_val(ph.sq_out + (size_t)row * (ph.N >> 5) + pair, float_word(q2));
      }
    }
    if (rd == 0) DF_STAMP(slot + 1);
    __syncthreads();
  }
  return false;
}

// Brings the weights of the unit's QKV item into the chip's cache, a word of each 128-byte line: for a workgroup that sums partials just before (16
// rows), with nothing to do until they come.  It requests the item's weights when its sum is out, and from memory they would arrive later
// than the operands (0.6 us a layer).
template <class S>
__device__ __forceinline__ void df_touch_weights(const DArgs& a, const DPhase& ph) {
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int NU = gridDim.x * 2, KT = ph.K >> 5, ntiles = (ph.N + 15) >> 4;
  int t0, t1, split;
  if (!df_gemm_item<PE_QKV, S>(ph, df_item_of_unit(blockIdx.x * 2 + (wave >> 2), ph.shift, NU, ph.stride), t0, t1, split)) return;
  const uint32_t* w0 = (const uint32_t*)ph.W0 + (size_t)t0 * KT * 256;
  const uint32_t* w1 = (const uint32_t*)ph.W0 + (size_t)(t1 < ntiles ? t1 : t0) * KT * 256;
  uint32_t x = 0u;
  for (int i = tid & 255; i < KT * 8; i += 256) x |= w0[i * 32] | w1[i * 32];
  asm volatile("" ::"v"(x));
}

// ------------------------------------------------------------------------------------------------ fused MLP
// Gate/up + SwiGLU + down projection inside one workgroup: its two units produce 32 consecutive columns of the
// SwiGLU output, which is exactly one k-tile of the down projection; the workgroup multiplies it with that k-tile of
// every output tile (8 waves x DN tiles) and publishes a partial of the whole row.  The SwiGLU output never
// leaves the workgroup, and one dependency per layer disappears; the price is ffn/32 partials per output.
constexpr int df_part_pitch(int C) { return C == 8 ? 64 : 4 * C; }     // bytes from one partial of C columns to the next
template <int DN>
struct WDown { u32x4 b[DN]; };

// (a zero would be a partial that is not there)
__device__ __forceinline__ void df_put_partial(df_rsrc r, uint32_t at, const f32x4 x) {
  u32x4 b = __builtin_bit_cast(u32x4, x);
#pragma unroll
  for (int i = 0; i < 4; ++i) b[i] = b[i] ? b[i] : 0x80000000u;
  __builtin_amdgcn_raw_buffer_store_b128(b, r, (int)at, 0, 16 /* sc1 */);
}

// Fragments (n-tile wave + 8 i, k-tile kt2) of the down projection for i < DN; exactly DN loads.
template <int DN>
__device__ __forceinline__ void df_prefetch_down(const DArgs& a, const void* wdown, int kt2, WDown<DN>& wd) {
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ntiles = a.d >> 4, KTd = a.ffn >> 5;
#pragma unroll
  for (int i = 0; i < DN; ++i) {
    const int nt = min(wave + 8 * i, ntiles - 1);          // (a wave may have fewer tiles than DN, below 128 columns none)
    wd.b[i] = __builtin_nontemporal_load((const u32x4*)wdown + ((size_t)nt * KTd + kt2) * 64 + lane);
  }
}

template <int SB, class S, typename CLEAR>
__device__ __forceinline__ bool df_mlp_phase(const DArgs& a, const DPhase& ph, const void* wdown, const float* part, CLEAR clear,
                                             uint32_t* lds, uint32_t* sact, int* sdead, int slot) {
  constexpr int C = df_sum_cols<SB>(), DN = S::DN;
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int usel = wave >> 2, uw = wave & 3, ut = tid & 255;
  const int unit = blockIdx.x * 2 + usel, NU = a.g_mlp * 2;
  uint32_t* As = lds;
  float* sqs = (float*)(lds + df_aw<SB, S>());
  float (*red)[2][256] = (float (*)[2][256])((float*)(lds + df_aw<SB, S>() + DF_SQ_WORDS) + usel * 2048);
  const int M = a.rows.M;
  const int KT = ph.K >> 5, ntiles_d = a.d >> 4, KTd = a.ffn >> 5;
  const int g = lane >> 4, c16 = lane & 15;
  const int row = ut >> 4, col = ut & 15;
  const int rounds = (ph.items + NU - 1) / NU;
  for (int rd = 0; rd < rounds; ++rd) {
    const int item = rd * NU + unit;
    const bool valid = item < ph.items;
    const int kt2 = item >> 1;                          // the workgroup's k-tile of the down projection
    int kb = 0, ke = 0;
    if (valid) wave_krange(ph, 0, uw, kb, ke);
    const bool live = valid && row < M;
    const int n0 = item * 16 + col;
    // the weights of the unit's item and the workgroup's down-projection tiles: requested at entry, they arrive
    // while the workgroup waits for its operands
    DfPre<S::PF> pre;
    WDown<DN> wd;
    if (valid) {
      const u32x4* w0 = (const u32x4*)ph.W0 + (size_t)item * KT * 64 + lane;
      const u32x4* w1 = (const u32x4*)ph.W1 + (size_t)item * KT * 64 + lane;
#pragma unroll
      for (int u = 0; u < S::PF; ++u) {
        const int kt = (kb + u < ke) ? kb + u : kb;
        pre.b0[u] = __builtin_nontemporal_load(w0 + (size_t)kt * 64);
        pre.b1[u] = __builtin_nontemporal_load(w1 + (size_t)kt * 64);
      }
    }
    if ((rd * NU + blockIdx.x * 2) < ph.items) df_prefetch_down(a, wdown, kt2, wd);
    if (rd == 0) {
      df_loads_done();
      clear();
    }
    float dummy0, dummy1;
    bool ok = true;
    if (rd == 0) ok = df_stage<SB, S, false>(a, ph.A, ph.K, ph.sq, KT, As, sqs, tid, nullptr, nullptr, dummy0, dummy1, ph.hint);
    if (!ok) *sdead = 1;
    __syncthreads();
    df_loads_done();
    if (*sdead) return true;
    if (rd == 0) DF_STAMP(slot);
    f32x4 acc0 = f32x4{0, 0, 0, 0}, acc1 = f32x4{0, 0, 0, 0};
    if (valid)
      df_products<df_pack<SB>(), S>(As, ph.K, M, kb, ke, lane, pre, (const u32x4*)ph.W0 + (size_t)item * KT * 64 + lane,
                                 (const u32x4*)ph.W1 + (size_t)item * KT * 64 + lane, acc0, acc1);
    float sq = 0.f;                                        // (while the matrix cores work)
    if (row < M)
      for (int p = col; p < KT; p += 16) sq += sqs[row * KT + p];
    const float inv = 1.0f / sqrtf(row16_sum(sq) / (float)ph.K + a.eps);
    df_meet<df_pack<SB>()>(acc0, acc1);
    DF_STAMP2(0);
    const int obase = (g * 4) * 16 + (lane & 15);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      red[uw][0][obase + r * 16] = acc0[r];
      red[uw][1][obase + r * 16] = acc1[r];
    }
    __syncthreads();
    DF_STAMP2(1);
    float v0 = (red[0][0][ut] + red[1][0][ut]) + (red[2][0][ut] + red[3][0][ut]);
    float v1 = (red[0][1][ut] + red[1][1][ut]) + (red[2][1][ut] + red[3][1][ut]);
    v0 *= inv;
    v1 *= inv;
    const float actv = (live && n0 < ph.N) ? v0 / (1.0f + expf(-v0)) * v1 : 0.f;
    sact[row * 36 + usel * 16 + col] = split_payload(actv);          // [16 rows][32 columns of the workgroup's k-tile]
    __syncthreads();
    DF_STAMP2(2);
    // ---- down projection of the workgroup's 32 columns: wave takes output tiles wave, wave + 8, ...
    if ((rd * NU + blockIdx.x * 2) < ph.items) {
      u32x4 xh = u32x4{0u, 0u, 0u, 0u}, xl = xh;
      if (c16 < M) frag_from_lds(sact + c16 * 36 + g * 8, xh, xl);
      const bf16x8 ah = __builtin_bit_cast(bf16x8, xh), al = __builtin_bit_cast(bf16x8, xl);
      // Computed transposed: a lane holds four consecutive columns of row c16.  They go out by way of LDS, row by row: a wave's seven tiles of a
      // row with one store, 128 contiguous bytes per tile.  (Straight from the registers, two stores per tile of which most lanes are masked, this
      // section took 0.8 us with one row, 0.5 so; with nine rows the sums' operands are there 0.8 us earlier.)
      f32x4 acc[DN];
#pragma unroll
      for (int i = 0; i < DN; ++i)
        acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wd.b[i]), al, f32x4{0, 0, 0, 0}, 0, 0, 0);
#pragma unroll
      for (int i = 0; i < DN; ++i) acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wd.b[i]), ah, acc[i], 0, 0, 0);
      const int nW = a.ffn >> 5;
      float* tr = (float*)(lds + S::TR) + wave * (8 * DN * 16);
      const df_rsrc rp = df_make_rsrc(part);
      const uint32_t row_bytes = (uint32_t)(ceil_div(a.d, C) * nW * df_part_pitch(C));
      auto place = [&](int nt, int q) {                              // of columns 4 q .. 4 q + 3 of a tile
        const int n = nt * 16 + 4 * q;
        return (uint32_t)((n / C * nW + kt2) * df_part_pitch(C) + n % C * 4);
      };
      // half a wave stores a row: this lane's row of two, tile, and four columns of it
      const int half = lane >> 5, ti = (lane & 31) >> 2, nt_out = wave + 8 * ti;
      const bool stores = ti < DN && nt_out < ntiles_d;
      uint32_t at = place(nt_out, lane & 3) + (uint32_t)half * row_bytes;
      for (int r0 = 0; r0 < M; r0 += 8) {
        if ((c16 & 8) == r0 && c16 < M)
#pragma unroll
          for (int i = 0; i < DN; ++i) *(f32x4*)(tr + ((c16 & 7) * DN + i) * 16 + 4 * g) = acc[i];
        const float* from = tr + (half * DN + ti) * 16 + 4 * (lane & 3);
        const int re = min(M, r0 + 8);
        for (int r = r0; r < re; r += 2, from += 2 * DN * 16, at += 2 * row_bytes)
          if (stores && r + half < re) df_put_partial(rp, at, *(const f32x4*)from);
      }
      for (int nt = wave + 8 * DN; nt < ntiles_d; nt += 8) {      // wider models: the remaining tiles, not prefetched
        const bf16x8 bv = __builtin_bit_cast(bf16x8, __builtin_nontemporal_load((const u32x4*)wdown + ((size_t)nt * KTd + kt2) * 64 + lane));
        f32x4 x = f32x4{0, 0, 0, 0};
        x = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bv, al, x, 0, 0, 0);
        x = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bv, ah, x, 0, 0, 0);
        if (c16 < M) df_put_partial(rp, place(nt, g) + (uint32_t)c16 * row_bytes, x);
      }
    }
    if (rd == 0) DF_STAMP(slot + 1);
    __syncthreads();
  }
  return false;
}

// The same for the wide form: a workgroup takes `mlp_tiles` (one or two) consecutive k-tiles of the down projection: half the partials (140 of width
// 1536), and with 280 k-tiles no second round on some of 256 workgroups.  What does not fit the registers and LDS while it waits streams behind the operands, 140
// workgroups at 5 TB/s, so as much as fits is requested at entry: the first k-tile, and of the second the down projection (ten of a wave's twelve tiles to LDS
// with up to 8 rows) and four or five of its twelve k-tiles of gate / up.  Five rows of width 1536 (28 layers): 770 us with two thirds of the second's down
// projection in registers and nothing else of it, 763 with it in LDS, 754 with two k-tiles of gate / up beside, 743 with four.  (The next layer's requested before
// the sums, when nothing streams: 770, the sums wait behind it.  More than 8 rows have no room: their operands are 98 KB.)
template <int SB, class S, typename CLEAR>
__device__ __forceinline__ bool df_mlp_wide(const DArgs& a, const DPhase& ph, const void* wdown, const float* part, CLEAR clear,
                                            uint32_t* lds, uint32_t* sact, int* sdead, int slot) {
  constexpr int C = df_sum_cols<SB>(), DN = S::DN, AP = S::ACT_PITCH;
  constexpr int LD = df_lds_tiles<SB>(), G1 = SB == 4 ? 4 : SB == 16 ? 5 : 0, D2 = 8;          // of the second k-tile: tiles of the down projection in LDS, k-tiles of gate / up in registers
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int usel = wave >> 2, uw = wave & 3, ut = tid & 255;
  uint32_t* As = lds;
  float* sqs = (float*)(lds + df_aw<SB, S>());
  float (*red)[2][256] = (float (*)[2][256])((float*)(lds + df_aw<SB, S>() + DF_SQ_WORDS) + usel * 2048);
  const int M = a.rows.M;
  const int KT = ph.K >> 5, ntiles_d = a.d >> 4, KTd = a.ffn >> 5;
  const int g = lane >> 4, c16 = lane & 15;
  const int row = ut >> 4, col = ut & 15;
  const int kt0 = blockIdx.x * a.mlp_tiles;
  const bool two = a.mlp_tiles == 2 && kt0 + 1 < KTd;
  int kb, ke;
  wave_krange(ph, 0, uw, kb, ke);
  DfPre<S::PF> pre;
  WDown<DN> wd;
  u32x4 wr[DN - LD], p0[G1 + 1], p1[G1 + 1];
  uint32_t* wl = lds + df_wl<SB, S>() + wave * (LD * 256);
  const df_rsrc r0 = df_make_rsrc(ph.W0), r1 = df_make_rsrc(ph.W1), rd = df_make_rsrc(wdown);
  auto gate_up = [&](int t, int u, u32x4& x0, u32x4& x1) {            // (through descriptors: one register of addresses)
    const uint32_t o = (uint32_t)((2 * (kt0 + t) + usel) * KT + ((kb + u < ke) ? kb + u : kb)) << 10;
    x0 = __builtin_amdgcn_raw_buffer_load_b128(r0, lane * 16, (int)o, 2 /* nt */);
    x1 = __builtin_amdgcn_raw_buffer_load_b128(r1, lane * 16, (int)o, 2);
  };
  auto down_at = [&](int t, int i) { return (int)((uint32_t)(min(wave + 8 * i, ntiles_d - 1) * KTd + kt0 + t) << 10); };       // (a wave may have fewer tiles than DN)
#pragma unroll
  for (int u = 0; u < S::PF; ++u) gate_up(0, u, pre.b0[u], pre.b1[u]);
#pragma unroll
  for (int i = 0; i < DN; ++i) wd.b[i] = __builtin_amdgcn_raw_buffer_load_b128(rd, lane * 16, down_at(0, i), 2);
  if (two) {
#pragma unroll
    for (int i = 0; i < LD; ++i) load_to_lds(rd, wl + i * 256, lane * 16, down_at(1, i));
    if (SB <= 16)
#pragma unroll
      for (int i = LD; i < DN; ++i) wr[i - LD] = __builtin_amdgcn_raw_buffer_load_b128(rd, lane * 16, down_at(1, i), 2);
#pragma unroll
    for (int u = 0; u < G1; ++u) gate_up(1, u, p0[u], p1[u]);
  }
  df_loads_done();
  clear();
  float dummy0, dummy1;
  const bool ok = df_stage<SB, S, false>(a, ph.A, ph.K, ph.sq, KT, As, sqs, tid, nullptr, nullptr, dummy0, dummy1, ph.hint);
  if (!ok) *sdead = 1;
  __syncthreads();
  df_loads_done();
  if (*sdead) return true;
  DF_STAMP(slot);
  float sq = 0.f;
  if (row < M)
    for (int p = col; p < KT; p += 16) sq += sqs[row * KT + p];
  const float inv = 1.0f / sqrtf(row16_sum(sq) / (float)ph.K + a.eps);
  auto swiglu = [&](int t) {
    f32x4 acc0 = f32x4{0, 0, 0, 0}, acc1 = f32x4{0, 0, 0, 0};
    df_products<df_pack<SB>(), S>(As, ph.K, M, kb, ke, lane, pre, (const u32x4*)ph.W0 + (size_t)(2 * (kt0 + t) + usel) * KT * 64 + lane,
                                  (const u32x4*)ph.W1 + (size_t)(2 * (kt0 + t) + usel) * KT * 64 + lane, acc0, acc1);
    if (t == 0 && two) {
#pragma unroll
      for (int u = 0; u < S::PF; ++u) {
        if (u < G1) { pre.b0[u] = p0[u]; pre.b1[u] = p1[u]; }
        else gate_up(1, u, pre.b0[u], pre.b1[u]);
      }
      if (SB > 16)
#pragma unroll
        for (int i = LD; i < D2; ++i) wr[i - LD] = __builtin_amdgcn_raw_buffer_load_b128(rd, lane * 16, down_at(1, i), 2);
    }
    if (SB > 16 && t == 1)
#pragma unroll
      for (int i = D2; i < DN; ++i) wr[i - LD] = __builtin_amdgcn_raw_buffer_load_b128(rd, lane * 16, down_at(1, i), 2);
    df_meet<df_pack<SB>()>(acc0, acc1);
    const int obase = (g * 4) * 16 + (lane & 15);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      red[uw][0][obase + r * 16] = acc0[r];
      red[uw][1][obase + r * 16] = acc1[r];
    }
    __syncthreads();
    float v0 = (red[0][0][ut] + red[1][0][ut]) + (red[2][0][ut] + red[3][0][ut]);
    float v1 = (red[0][1][ut] + red[1][1][ut]) + (red[2][1][ut] + red[3][1][ut]);
    v0 *= inv;
    v1 *= inv;
    sact[row * AP + t * 32 + usel * 16 + col] = split_payload(row < M ? v0 / (1.0f + expf(-v0)) * v1 : 0.f);     // [16 rows][32 columns of each k-tile]
    __syncthreads();
  };
  f32x4 acc[DN];
  auto down = [&](int t) {
    u32x4 xh = u32x4{0u, 0u, 0u, 0u}, xl = xh;
    if (c16 < M) frag_from_lds(sact + c16 * AP + t * 32 + g * 8, xh, xl);
    const bf16x8 ah = __builtin_bit_cast(bf16x8, xh), al = __builtin_bit_cast(bf16x8, xl);
#pragma unroll
    for (int i = 0; i < DN; ++i) {
      const bf16x8 w = __builtin_bit_cast(bf16x8, t == 0 ? wd.b[i] : i < LD ? *(const u32x4*)(wl + i * 256 + lane * 4) : wr[max(i - LD, 0)]);
      acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, al, t == 0 ? f32x4{0, 0, 0, 0} : acc[i], 0, 0, 0);
      acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, ah, acc[i], 0, 0, 0);
    }
  };
  swiglu(0);
  if (two) swiglu(1);
  down(0);
  if (two) down(1);
  // partials out by way of LDS, row by row, as above: a row's tiles of a wave in 64 lanes, 16 tiles at most
  const int nW = a.n_sum;
  float* tr = (float*)(lds + S::TR) + wave * (8 * DN * 16);
  const df_rsrc rp = df_make_rsrc(part);
  const uint32_t row_bytes = (uint32_t)(ceil_div(a.d, C) * nW * df_part_pitch(C));
  auto place = [&](int nt, int q) {                                  // of columns 4 q .. 4 q + 3 of a tile
    const int n = nt * 16 + 4 * q;
    return (uint32_t)((n / C * nW + (int)blockIdx.x) * df_part_pitch(C) + n % C * 4);
  };
  const int ti = lane >> 2, nt_out = wave + 8 * ti;
  const bool stores = ti < DN && nt_out < ntiles_d;
  uint32_t at = place(nt_out, lane & 3);
  for (int r0 = 0; r0 < M; r0 += 8) {
    if ((c16 & 8) == r0 && c16 < M)
#pragma unroll
      for (int i = 0; i < DN; ++i) *(f32x4*)(tr + ((c16 & 7) * DN + i) * 16 + 4 * g) = acc[i];
    const float* from = tr + ti * 16 + 4 * (lane & 3);
    const int re = min(M, r0 + 8);
    for (int r = r0; r < re; ++r, from += DN * 16, at += row_bytes)
      if (stores) df_put_partial(rp, at, *(const f32x4*)from);
  }
  DF_STAMP(slot + 1);
  __syncthreads();
  return false;
}

// Sum of the ffn/32 down-projection partials, residual, and the operand / statistics of the next RMSNorm.  Task = (row, C
// output columns) on a whole workgroup.  Tasks go to the workgroups with MLP items first, one each.  Their first requests queue behind the
// acknowledgement of their own stores, and then nearly always find everything there; a workgroup without an MLP item that polls meanwhile
// delays those stores (five rows 1.2 us a layer more when such workgroups came first), so it watches one word of its last partial.
// The last ones to get a task are those with QKV or attention items, which begin the next layer: C = 64 for six rows and more leaves
// them without one up to 12 rows of the 0.5B shape, and gives none a second task (nine rows: 24.3 -> 20.7 us a layer, against C = 32).
// With few rows what counts is the time to take in a task's partials: C = 8 for one, or for two that are one round of tasks (one row: 1.9 us from the end of the MLP to the sum;
// with 16 columns 2.0, with 32 3.0), else 32.
// Partials of 4 bytes without a tag instead of 8 with one, and 16-byte loads: from the MLP's end to the sum five rows 3.4 -> 2.2 us, nine 3.5 -> 2.4.
// The order of a sum does not depend on C: the partials form 64 blocks of consecutive ones, summed in ascending order; eight
// blocks meet as a binary tree - in the thread, which may hold two, and between the lanes -, and eight such groups in ascending
// order in LDS.  So it is with the squares: a tree over columns whose nodes over 8 or 32 are published.
constexpr int DF_RBLOCKS = 64;
constexpr int DF_RW = 3;                  // partials of a block in flight
// Partials of an output: one per MLP workgroup's share of the SwiGLU output.
template <class S>
__device__ __forceinline__ int df_partials(const DArgs& a) { return S::WIDE ? a.n_sum : a.ffn >> 5; }
// A thread's partials in a task: four columns of one block, or of two consecutive ones.  The lanes that share a column and eight
// consecutive blocks differ in lane bits that the cheap lane exchanges reach in the order of the tree (df_sum_blocks).
template <int C>
struct DfPartials {
  static constexpr int TB = C == 64 ? 2 : 1;               // blocks
  int group, cg;                                           // eight blocks; which four columns
  int w[TB + 1];                                           // first partial of a block, and of the one after the last
  __device__ __forceinline__ DfPartials(int tid, int nW) {
    const int l = tid & 63;
    group = tid >> (C == 8 ? 4 : 6);
    cg = l & (C / 4 - 1);
    const int blk = group * 8 + (C == 64 ? l >> 4 << 1 : C == 32 ? l >> 3 : (l >> 3 & 1) | (l >> 1 & 2) | (l << 1 & 4));
#pragma unroll
    for (int t = 0; t <= TB; ++t) w[t] = group < 8 ? (blk + t) * nW / DF_RBLOCKS : 0;
  }
  __device__ __forceinline__ uint32_t at(int task, int nW) const { return (uint32_t)((task * nW + w[0]) * df_part_pitch(C) + 16 * cg); }     // in bytes
};
template <int C>
__device__ __forceinline__ float df_sum_blocks(float s) {
  if (C == 64) return sum_over_groups(s);
  s += dpp_f<0x128>(s);                                    // row_ror:8: that of lane ^ 8
  if (C == 32) return sum_over_groups(s);
  s += dpp_f<0x124>(s);                                    // row_ror:4: that of lane ^ 4 or ^ 12, which are the same now
  return s + dpp_f<0x4E>(s);                               // quad_perm: lane ^ 2
}
template <int C, class S>
__device__ __forceinline__ bool df_reduce_phase(const DArgs& a, const float* part, const uint32_t* h_in,
                                                uint32_t* h_out, uint32_t* hg_out, uint32_t* sq_out, const float* gain_next, int shift,
                                                uint32_t* lds, int* sdead, int slot) {
  constexpr int TB = DfPartials<C>::TB, CS = C < 32 ? C : 32;        // columns of a sum of squares
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int NW = gridDim.x;
  const int d = a.d, np = ceil_div(d, C), nW = df_partials<S>(a), tasks = a.rows.M * np;
  const int first = df_item_of_unit(blockIdx.x, shift >> 1, NW);       // a task has the whole workgroup
  float* rs = (float*)(lds + S::RS);                     // [8 groups of blocks][C]
  const DfPartials<C> pt(tid, nW);
  const int bs = (nW + DF_RBLOCKS - 1) / DF_RBLOCKS;
  const df_rsrc rp = df_make_rsrc(part);
  uint32_t* err = a.bar + 64;
  bool bad = false;
  for (int task = first; task < tasks; task += NW) {
    const int m = task / np, col = C * (task - m * np) + tid;
    const size_t o = (size_t)m * d + col;
    const bool some = col - tid + 4 * pt.cg < d, want_h = tid < C && col < d;      // (of the last 64 columns the second half may not be there)
    uint32_t at = pt.at(task, nW);
    f32x4 s[TB];
#pragma unroll
    for (int t = 0; t < TB; ++t) s[t] = f32x4{0, 0, 0, 0};
    uint32_t hw = 1u;
    const float gain = want_h ? gain_next[col] : 0.f;
    for (int k0 = 0; k0 < bs; k0 += DF_RW) {
      u32x4 v[TB][DF_RW];
      auto there = [&](int t, int i) { return some && pt.w[t] + k0 + i < pt.w[t + 1]; };
      auto request = [&](int t, int i) { return __builtin_amdgcn_raw_buffer_load_b128(rp, (int)(at + (uint32_t)((pt.w[t] - pt.w[0] + k0 + i) * df_part_pitch(C))), 0, 16 /* sc1 */); };
#pragma unroll
      for (int t = 0; t < TB; ++t)
#pragma unroll
        for (int i = 0; i < DF_RW; ++i) v[t][i] = there(t, i) ? request(t, i) : u32x4{1u, 1u, 1u, 1u};
      if (k0 == 0 && want_h) hw = ld_val(h_in + o);
      for (long spins = 0;;) {
        bool late = hw == 0u;
#pragma unroll
        for (int t = 0; t < TB; ++t)
#pragma unroll
          for (int i = 0; i < DF_RW; ++i) late = late || df_any_zero(v[t][i]);
        if (!late) break;
        // a workgroup that comes here from its own MLP item is not early; another one first watches a word of the last partial
        if (spins == 0 && (int)blockIdx.x >= a.g_mlp) df_wait_hint((const uint32_t*)part + (size_t)((task + 1) * nW - 1) * (df_part_pitch(C) / 4), err);
        if (++spins > DF_SPIN_LIMIT || ((spins & 63) == 0 && __hip_atomic_load(err, __ATOMIC_RELAXED, AG) != 0)) {
          __hip_atomic_store(err, 1u, __ATOMIC_RELAXED, AG);
          bad = true;
          break;
        }
        __builtin_amdgcn_s_sleep(1);
        asm volatile("" : "+v"(at) : : "memory");          // (the words may have changed)
#pragma unroll
        for (int t = 0; t < TB; ++t)
#pragma unroll
          for (int i = 0; i < DF_RW; ++i)
            if (df_any_zero(v[t][i])) v[t][i] = request(t, i);
        if (hw == 0u) hw = ld_val(h_in + o);
      }
#pragma unroll
      for (int t = 0; t < TB; ++t)
#pragma unroll
        for (int i = 0; i < DF_RW; ++i)
          if (there(t, i)) s[t] += __builtin_bit_cast(f32x4, v[t][i]);
    }
    f32x4 x = TB == 1 ? s[0] : s[0] + s[TB - 1];
#pragma unroll
    for (int i = 0; i < 4; ++i) x[i] = df_sum_blocks<C>(x[i]);
    if (pt.group < 8 && (tid & (C == 8 ? 15 : 63)) < C / 4) *(f32x4*)(rs + pt.group * C + 4 * pt.cg) = x;
    if (bad) *sdead = 1;
    // Besides this task's words: the zeros of the layer before have reached memory.  Nobody stores into their places before he has seen,
    // by way of the next layers' phases, the sums that every workgroup publishes below.
    df_loads_done();
    __syncthreads();
    if (*sdead) return true;
    if (task == first) DF_STAMP(slot);
    if (want_h) {
      float r[8];
#pragma unroll
      for (int w = 0; w < 8; ++w) r[w] = rs[w * C + tid];
      const float v = (((((((r[0] + r[1]) + r[2]) + r[3]) + r[4]) + r[5]) + r[6]) + r[7]) + __uint_as_float(hw);
      st_val(h_out + o, float_word(v));
      st_val(hg_out + o, operand_word(v * gain));
      float q2 = v * v;
#pragma unroll
      for (int off = 1; off < 16; off <<= 1)
        if (off < CS) q2 += off == 1 ? dpp_f<0xB1>(q2) : off == 2 ? dpp_f<0x4E>(q2) : off == 4 ? dpp_f<0x141>(q2) : dpp_f<0x140>(q2);       // (as row16_sum)
      if (CS == 32) {
        const auto x = __builtin_amdgcn_permlane16_swap(__float_as_uint(q2), __float_as_uint(q2), false, false);
        q2 = __uint_as_float(x[0]) + __uint_as_float(x[1]);
      }
      if ((tid & (CS - 1)) == 0) st_val(sq_out + (size_t)m * (d / CS) + col / CS, float_word(q2));
    }
    if (task == first) DF_STAMP(slot + 1);
    __syncthreads();
  }
  return false;
}

// The partials that this workgroup has read in a layer become zeros again, in the next layer, when it has nothing better to do: behind its own QKV,
// attention and output items, or when its MLP item's weights have come (right behind the sums these stores delayed the next operands).
template <int C, class S>
__device__ __forceinline__ void df_clear_partials(const DArgs& a, const float* part, int shift) {
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int NW = gridDim.x, nW = df_partials<S>(a), tasks = a.rows.M * ceil_div(a.d, C);
  const DfPartials<C> pt(tid, nW);
  const df_rsrc rp = df_make_rsrc(part);
  for (int task = df_item_of_unit(blockIdx.x, shift >> 1, NW); task < tasks; task += NW) {
    const uint32_t at = pt.at(task, nW);
    for (int k = pt.w[0]; k < pt.w[DfPartials<C>::TB]; ++k)
      __builtin_amdgcn_raw_buffer_store_b128(u32x4{0u, 0u, 0u, 0u}, rp, (int)(at + (uint32_t)((k - pt.w[0]) * df_part_pitch(C))), 0, 16 /* sc1 */);
  }
}

// The words of a layer that the launch before left in its set become zeros: by the workgroups with MLP items, while they wait.
template <class S>
__device__ __forceinline__ void df_clear_layer(const DArgs& a, const size_t set, int rows, int l) {
  if (rows == 0) return;
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  int wg = blockIdx.x;                                     // the words of one kind begin where those of another end
  auto zero = [&](uint32_t* p, int words) {
    const int n = min((words + 2047) >> 11, a.g_mlp);      // workgroups
    const df_rsrc r = df_make_rsrc(p);
    for (int i = (wg * PBLOCK + tid) * 4; i < words; i += a.g_mlp * PBLOCK * 4) __builtin_amdgcn_raw_buffer_store_b128(u32x4{0u, 0u, 0u, 0u}, r, i * 4, 0, 16 /* sc1 */);
    wg -= n;
    if (wg < 0) wg += a.g_mlp;
  };
  for (int hi = l ? 2 * l + 1 : 0; hi <= 2 * l + 2; ++hi) {
    zero(a.h + set + (size_t)hi * a.st_h, rows * a.d);
    zero(a.hg + set + (size_t)hi * a.st_h, rows * a.d);
    zero(a.sq + set + (size_t)hi * a.st_sq, rows * (a.d >> 3));
  }
  zero(a.q + set + (size_t)l * a.st_q, rows * a.nq * S::HD);
  zero(a.attn + set + (size_t)l * a.st_q, rows * a.nq * S::HD);
  zero(a.kvn + set + (size_t)l * a.st_kvn, rows * a.nkv * 2 * S::HD);
}

// ------------------------------------------------------------------------------------------------ phase 0
// Rows and embedding.  Item = row.
template <int C>
__device__ __forceinline__ void df_embed_phase(const DArgs& a, const size_t set) {
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), usel = wave >> 2, ut = tid & 255;
  const int unit = blockIdx.x * 2 + usel, NU = gridDim.x * 2;
  const int M = a.rows.M, R = a.rows.R, d = a.d;
  for (int m = unit; m < M; m += NU) {
    const int brel = m / R, j = m - brel * R;
    const int seq = a.rows.seq0 + brel;
    // every candidate is requested at once: which of them is the row's token follows from the pending count
    const int npend = a.pcap ? ld_state(a.kv.n_pend + seq) : 0;
    const int len = ld_state(a.kv.len + seq);
    const int p0 = a.pcap ? ld_state(a.kv.pend + seq * 2) : 0;
    const int p1 = a.pcap > 1 ? ld_state(a.kv.pend + seq * 2 + 1) : 0;
    const int tx = j >= a.pcap ? ld_state(a.tokens + (size_t)brel * a.tok_stride + (j - a.pcap)) : 0;
    const int off = a.pcap - npend;
    int tok, pos, active;
    if (j < off) { tok = p0; pos = len; active = 0; }
    else {
      pos = len + (j - off); active = 1;
      tok = j < a.pcap ? ((j - off) ? p1 : p0) : tx;
    }
    tok = min(max(tok, 0), a.n_embed - 1);
    if (ut == 0) { st_ag(a.rows.pos + m, pos); st_ag(a.rows.active + m, active); }
    const bf16_t* src = a.embed + (size_t)tok * d;
    const float* gain = a.layer0.ln1;
    for (int p = ut >> 5; p < (d >> 5); p += 8) {
      const int c = p * 32 + (ut & 31);
      const float v = bf16_to_f(src[c]);
      st_val(a.h + set + (size_t)m * d + c, float_word(v));
      st_val(a.hg + set + (size_t)m * d + c, operand_word(v * gain[c]));
      float sq = v * v;
#pragma unroll
      for (int o = 1; o < C; o <<= 1) sq += __shfl_xor(sq, o, WAVE);       // as df_reduce_phase leaves them
      if ((ut & (C - 1)) == 0) st_val(a.sq + set + (size_t)m * (d / C) + c / C, float_word(sq));
    }
  }
}

// Block reservation for the rows of this launch, by one workgroup: lane b of its first wave takes sequence b (at most
// 16 sequences).  Two memory round trips for all of them: the state words, then the ids (free-stack entries for new
// blocks, table entries for blocks already owned).  Sequences take from the free stack in ascending order, top first,
// as a serial walk over the sequences would.  Nothing waits for the table itself: the block that holds a row's new
// key goes out as a tagged word per row (the workgroups with QKV items, whose epilogue appends the keys and values,
// wait for it once), and attention never reads a position of this launch from the pool.  The launch therefore has no
// grid barrier.
__device__ __forceinline__ bool df_tag_ok(uint32_t tag) { return tag != 0u && tag < TAG_LIMIT; }

template <typename AR>
__device__ __forceinline__ void df_reserve_blocks(const AR& a, const int tag_v, const bool mine) {
  if (!mine || threadIdx.x >= 64) return;
  const int b = threadIdx.x, R = a.rows.R;
  const bool on = b < a.n_seqs;
  const int s = a.rows.seq0 + (on ? b : 0);
  const int top = ld_state(a.kv.ctl);
  const int np_s = a.pcap ? ld_state(a.kv.n_pend + s) : 0;
  const int len_s = ld_state(a.kv.len + s);
  const int own = ld_state(a.kv.owned + s);
  const int off = a.pcap ? a.pcap - np_s : 0;
  const int need = ceil_div(len_s + R - off, a.kv.bt);
  const uint32_t tag = (uint32_t)__builtin_amdgcn_readfirstlane(tag_v);
  if (!df_tag_ok(tag)) return;                                     // a refused launch changes nothing
  const int want = on ? max(0, need - own) : 0, room = max(0, a.kv.mbps - own);
  const int take = min(want, room);
  int before = take;                                               // blocks that lower sequences take: exclusive prefix sum
#pragma unroll
  for (int o = 1; o < 16; o <<= 1) {
    const int v = __shfl_up(before, o, WAVE);
    if (b >= o) before += v;
  }
  const int total = __shfl(before, 15, WAVE);
  before -= take;
  const int got = max(0, min(take, top - before));
  // ids of the (at most two) blocks that hold the positions of this launch's rows
  const int bi0 = len_s >> 4;
  int id[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int bi = bi0 + i;
    id[i] = -1;
    if (on && bi < own) id[i] = ld_state(a.kv.table + s * a.kv.mbps + bi);
    else if (on && bi - own < got) id[i] = ld_state(a.kv.free_stack + (top - before - 1 - (bi - own)));
  }
  if (on) {
    for (int i = 0; i < got; ++i) {
      const int bi = own + i;
      const int v = bi == bi0 ? id[0] : bi == bi0 + 1 ? id[1] : ld_state(a.kv.free_stack + (top - before - 1 - i));
      st_ag(a.kv.table + s * a.kv.mbps + bi, v);
    }
    a.kv.owned[s] = own + got;
    if (got < want) a.kv.ctl[1] = 1;
    for (int j = 0; j < R; ++j) {
      const int pos = j < off ? len_s : len_s + (j - off);
      const int bi = pos >> 4;
      const int v = bi == bi0 ? id[0] : bi == bi0 + 1 ? id[1] : -1;
      st_word(a.rowblk + b * R + j, (uint32_t)v, tag);
    }
  }
  if (b == 0) a.kv.ctl[0] = max(0, top - total);
}

// ------------------------------------------------------------------------------------------------ attention
// Item = (sequence, kv head, part of the keys, tile of 16 query rows) on a workgroup; the query rows of a sequence are its R
// rows times the G query heads of the group, row index qr = j * G + head-in-group.  Wave w takes chunks w, w + 8, w + 16 (of 64
// keys) of its part: all their scores, one maximum and one sum per row, the weighted values; the eight waves meet once in LDS.  Scores are kept
// in the base-2 domain (scale * log2 e folded in), so that the exponentials are single instructions.
//
// How a row's keys are cut follows from its position alone, so that it has the same bits alone, in a verification, in a captured
// cycle and beside any other sequence: a row below DF_ONE_PART attends in one part of up to DF_ONE_CHUNKS chunks, whose result goes
// out as operand words; any other in parts of DF_PART_CHUNKS chunks cut at absolute positions, which their workgroups merge (see the
// end of df_attn_phase).  Merging costs a hand-over and about 2.5 us per layer, a third round of chunks 1.2: hence one part as far
// as three rounds reach, and two rounds beyond.  The host only provides the workgroups, from its bound of the lengths: those
// without keys have nothing to do.  Where rows of one sequence lie on both sides of the line, part 0 walks its third round too,
// masked for the rows beyond (their maximum, sum and values keep their bits: scores of -inf, terms of 0).
constexpr int DF_ONE_CHUNKS = 24, DF_ONE_PART = 64 * DF_ONE_CHUNKS, DF_PART_CHUNKS = 16;
__host__ __device__ constexpr int df_parts(int positions) {     // parts of a row that attends to this many positions
  return positions <= DF_ONE_PART ? 1 : (positions + 64 * DF_PART_CHUNKS - 1) / (64 * DF_PART_CHUNKS);
}
struct DAttItem {
  int valid, b, kvh, part, rt, half, len, nact, off, pos_last;
  int c0, nch, nparts_b;                                 // first chunk and chunks of the part, parts of the sequence
};

// Everything here is requested at once (one memory round trip, not six): the cached length and the pending count do
// not change during the launch, and the block ids of positions below the cached length do not either.  A block all of
// whose positions are at or beyond the cached length may be reserved concurrently by this launch: whatever id is read
// for it is only checked to be inside the pool, since each of its positions is either a row of this launch (taken from
// the side buffer, never from the pool) or masked.
template <class S>
__device__ __forceinline__ DAttItem df_att_item(const DArgs& a, int item, int ntile, int* sblk) {
  DAttItem it;
  it.valid = item < a.n_seqs * a.nkv * a.n_parts * ntile * S::NH;
  it.b = 0; it.kvh = 0; it.part = 0; it.rt = 0; it.half = 0;
  if (it.valid) {
    if (S::NH > 1) it.half = item % S::NH;
    const int u = item / S::NH;
    it.rt = u % ntile;
    int t = u / ntile;
    it.b = t % a.n_seqs;
    t /= a.n_seqs;
    it.kvh = t % a.nkv;
    it.part = t / a.nkv;
  }
  const int seq = a.rows.seq0 + it.b;
  it.c0 = it.part * DF_PART_CHUNKS;
  // (only by the workgroups that have an item: a few hundred asking for the same words queue up at one channel)
  const int len_v = it.valid ? ld_state(a.kv.len + seq) : 0;
  const int npend_v = (it.valid && a.pcap) ? ld_state(a.kv.n_pend + seq) : 0;
  const int i = threadIdx.x, bi = it.c0 * 4 + i;
  int bid = -1;
  if (i < DF_ONE_CHUNKS * 4 && it.valid && bi < a.kv.mbps) bid = ld_state(a.kv.table + seq * a.kv.mbps + bi);
  it.len = __builtin_amdgcn_readfirstlane(len_v);
  const int npend = __builtin_amdgcn_readfirstlane(npend_v);
  it.off = a.pcap - npend;
  it.nact = a.rows.R - it.off;
  it.pos_last = it.len + it.nact - 1;
  const int nch = it.pos_last / 64 + 1;
  it.nparts_b = df_parts(it.pos_last + 1);
  it.nch = min(it.part == 0 && it.len < DF_ONE_PART ? DF_ONE_CHUNKS : DF_PART_CHUNKS, nch - it.c0);     // (a row stands at `len`)
  it.valid = it.valid && it.part < it.nparts_b;
  // block ids of the part's positions (masked positions may read any block)
  if (i < DF_ONE_CHUNKS * 4) sblk[i] = (bid < 0 || bid >= a.kv.n_blocks || bi * 16 > it.pos_last) ? 0 : bid;
  return it;
}

// A wave's chunk of 64 keys is computed transposed: the keys are the rows of the score tiles and the query rows their
// columns, so a lane holds, of ONE query row (lane % 16), the scores of keys 4 g .. 4 g + 3 of each of the chunk's four blocks
// (g = lane / 16).  The row's maximum and sum are in-lane operations and two exchanges between the lane groups, and the
// weights are where the product with the values wants them: its contraction takes the lane's eight keys of two blocks as
// its eight k, so the values come as 8 bytes (four tokens of a dim) from each of the two.  Nothing goes through LDS.
// (With query rows as rows of the tiles a lane had four rows' statistics, each a chain of 16-lane reductions, and the weights
// took a way through LDS: the attention of one row and 1024 keys took 5.5 us of a layer, 3.7 now.)
// Head size 128: the keys of a chunk take 64 registers, its values as many.  An item is half of the output's dims: its workgroup works out all scores, and
// weights 64 dims of the values.  Two chunks' keys are in registers, and the first one's values, the other two chunks' in LDS; the third
// chunk's keys are brought into the chip's cache and take the first one's registers when its scores are there.
template <class S>
struct DfK { u32x4 f[4][S::HD / 32]; };                  // [block][32 dims]
struct DfV { u32x4 f[2][4]; };                           // [pair of blocks][16 dims]

// Positions at or beyond the sequence's cached length hold whatever an earlier launch left there; they are patched or
// masked later, never used.
template <class S>
__device__ __forceinline__ const bf16_t* df_plane(const DArgs& a, int plane) { return (const bf16_t*)a.kv.pool + (size_t)plane * ((size_t)a.kv.n_blocks * a.kv.nkv * (16 * S::HD)); }
template <class S>
__device__ __forceinline__ void df_load_k(const DArgs& a, int layer, const int (&boff)[4], int lane, DfK<S>& k) {
  const df_rsrc r = df_make_rsrc(df_plane<S>(a, 2 * layer));           // (through a descriptor: one register of addresses)
  const int at = (lane & 15) * (2 * S::HD) + (lane >> 4) * 16;
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int ks = 0; ks < S::HD / 32; ++ks) k.f[t][ks] = __builtin_amdgcn_raw_buffer_load_b128(r, at + 64 * ks, (int)(2u * (uint32_t)boff[t]), 0);
}
// (boff: of the values, with the item's half of the dims)
template <class S>
__device__ __forceinline__ void df_load_v(const DArgs& a, int layer, const int (&boff)[4], int lane, DfV& v) {
  const df_rsrc r = df_make_rsrc(df_plane<S>(a, 2 * layer + 1));
  const int at = (lane & 15) * 32 + (lane >> 4) * 8;
#pragma unroll
  for (int ks = 0; ks < 2; ++ks)
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) {
      const auto x = __builtin_amdgcn_raw_buffer_load_b64(r, at + dt * 512, (int)(2u * (uint32_t)boff[2 * ks]), 0), y = __builtin_amdgcn_raw_buffer_load_b64(r, at + dt * 512, (int)(2u * (uint32_t)boff[2 * ks + 1]), 0);
      v.f[ks][dt] = u32x4{x[0], x[1], y[0], y[1]};
    }
}

// Positions written by this launch: their keys and values come from the side buffer, at the pool's fragment slots.
template <class S>
__device__ __forceinline__ void df_patch_k(DfK<S>& k, int kbase, int len, int nact, const bf16_t* Kn, int lane) {
  const int g = lane >> 4, c16 = lane & 15;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int jn = kbase + 16 * t + c16 - len;
    if ((unsigned)jn < (unsigned)nact)
#pragma unroll
      for (int ks = 0; ks < S::HD / 32; ++ks) k.f[t][ks] = *(const u32x4*)(Kn + jn * S::HD + 32 * ks + g * 8);
  }
}
// Values of a chunk by way of LDS: its four blocks as they are in the pool, [block][dim][token] (2 KB each, one wave's direct
// loads; the wave waits for them itself).
template <class S>
__device__ __forceinline__ void df_v_to_lds(const DArgs& a, int layer, const int (&boff)[4], int lane, uint32_t* v2) {
  const df_rsrc r = df_make_rsrc(df_plane<S>(a, 2 * layer + 1));
#pragma unroll
  for (int i = 0; i < 8; ++i) load_to_lds(r, v2 + i * 256, (int)(2u * (uint32_t)boff[i >> 1] + (uint32_t)(lane * 16 + (i & 1) * 1024)), 0);      // (32 bits: a plane has fewer than 2^31 elements)
}
__device__ __forceinline__ void df_v_from_lds(uint32_t* v2, int kbase, int len, int nact, const bf16_t* Vn, int lane, DfV& v) {
  const int g = lane >> 4, c16 = lane & 15;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  for (int jn = max(0, kbase - len); jn < min(nact, kbase + 64 - len); ++jn) {       // this launch's positions, lane = dim
    const int tok = len + jn - kbase;
    ((bf16_t*)v2)[(tok >> 4) * 1024 + lane * 16 + (tok & 15)] = Vn[jn * 64 + lane];
  }
  asm volatile("" ::: "memory");
#pragma unroll
  for (int ks = 0; ks < 2; ++ks)
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) {
      const uint2 x = *(const uint2*)(v2 + ks * 1024 + (16 * dt + c16) * 8 + g * 2);
      const uint2 y = *(const uint2*)(v2 + ks * 1024 + 512 + (16 * dt + c16) * 8 + g * 2);
      v.f[ks][dt] = u32x4{x.x, x.y, y.x, y.y};
    }
}

__device__ __forceinline__ float df_exp2(float x) { return __builtin_amdgcn_exp2f(x); }     // x <= 0 here, or -inf

// The lane's query row: maximum (base-2 domain), sum (the same in all lane groups) and weighted values, dims 16 dt + 4 g + r.
struct DfRow { float m, l; f32x4 o[4]; };

// The lane's query row: in registers, or (wide) where it is in LDS, of every eight dims the hi halves, then the lo halves.
template <class S>
struct DfQ { u32x4 hi[2], lo[2]; };
template <>
struct DfQ<DfWide> { const uint32_t* at; };

// Scores of one chunk's keys.  qpos: position of the lane's query row (-1: none).
template <class S>
__device__ __forceinline__ void df_scores(const DfK<S>& k, const DfQ<S>& q, int kbase, int qpos, bool masked, int lane, f32x4 (&s)[4]) {
  const int g = lane >> 4;
#pragma unroll
  for (int t = 0; t < 4; ++t) s[t] = f32x4{0, 0, 0, 0};
  auto product = [&](int ks, const u32x4 q) {              // (four chains side by side)
#pragma unroll
    for (int t = 0; t < 4; ++t) s[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, k.f[t][ks]), __builtin_bit_cast(bf16x8, q), s[t], 0, 0, 0);
  };
  if constexpr (S::WIDE) {
#pragma unroll
    for (int ks = 0; ks < S::HD / 32; ++ks) {
      const u32x4 lo = *(const u32x4*)(q.at + ks * 32 + 4), hi = *(const u32x4*)(q.at + ks * 32);
      product(ks, lo);
      product(ks, hi);
      __builtin_amdgcn_sched_barrier(0);
    }
  } else {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) product(ks, q.lo[ks]);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) product(ks, q.hi[ks]);
  }
  if (masked) {                                            // (wave-uniform: only chunks that reach the new positions)
    const int last = qpos - kbase - 4 * g;
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) s[t][e] = 16 * t + e <= last ? s[t][e] : -INFINITY;
  }
}
__device__ __forceinline__ float df_max16(const f32x4 (&s)[4]) {
  f32x4 m4 = s[0];
#pragma unroll
  for (int t = 1; t < 4; ++t)
#pragma unroll
    for (int e = 0; e < 4; ++e) m4[e] = fmaxf(m4[e], s[t][e]);
  return fmaxf(fmaxf(m4[0], m4[1]), fmaxf(m4[2], m4[3]));
}
// Scores -> weights against the maximum; their sum over the lane's keys.
__device__ __forceinline__ float df_weights(f32x4 (&s)[4], float sc2, float base) {
  f32x4 sum4 = f32x4{0, 0, 0, 0};
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      s[t][e] = df_exp2(fmaf(s[t][e], sc2, -base));
      sum4[e] += s[t][e];
    }
  return (sum4[0] + sum4[1]) + (sum4[2] + sum4[3]);
}
__device__ __forceinline__ void df_values(const DfV& v, const f32x4 (&s)[4], DfRow& r) {
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    const uint2 h0 = hi_pairs(s[2 * ks]), h1 = hi_pairs(s[2 * ks + 1]), l0 = lo_pairs(s[2 * ks]), l1 = lo_pairs(s[2 * ks + 1]);
    const bf16x8 ph = __builtin_bit_cast(bf16x8, u32x4{h0.x, h0.y, h1.x, h1.y}), pl = __builtin_bit_cast(bf16x8, u32x4{l0.x, l0.y, l1.x, l1.y});
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) r.o[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, v.f[ks][dt]), pl, r.o[dt], 0, 0, 0);
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) r.o[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, v.f[ks][dt]), ph, r.o[dt], 0, 0, 0);
  }
}

// A wave's rows into the merge buffers [wave][row][dim], [wave][row][max, sum]
template <class S>
__device__ __forceinline__ void df_put_row(const DfRow& r, float* MO, float* ML, int wave, int lane) {
  const int g = lane >> 4, c16 = lane & 15;
#pragma unroll
  for (int dt = 0; dt < 4; ++dt) *(f32x4*)(MO + wave * S::MO_WAVE + c16 * DF_QS + 16 * dt + 4 * g) = r.o[dt];
  if (g == 0) { ML[(wave * 16 + c16) * 2] = r.m; ML[(wave * 16 + c16) * 2 + 1] = r.l; }
}

// Merge of the waves' (ascending) share of a row: maximum, sum and the two dims d0, d0 + 1.
template <class S>
__device__ __forceinline__ void df_merge_row(const float* MO, const float* ML, int row, int d0, float& mx, float& l, float (&o)[2]) {
  mx = -INFINITY; l = 0.f; o[0] = o[1] = 0.f;
#pragma unroll
  for (int w = 0; w < 8; ++w) mx = fmaxf(mx, ML[(w * 16 + row) * 2]);
  const float base = mx == -INFINITY ? 0.f : mx;
#pragma unroll
  for (int w = 0; w < 8; ++w) {
    const float e = df_exp2(ML[(w * 16 + row) * 2] - base);
    l = fmaf(ML[(w * 16 + row) * 2 + 1], e, l);
    const float2 x = *(const float2*)(MO + w * S::MO_WAVE + row * DF_QS + d0);
    o[0] = fmaf(x.x, e, o[0]);
    o[1] = fmaf(x.y, e, o[1]);
  }
}

template <int SB, class S>
__device__ __forceinline__ bool df_attn_phase(const DArgs& a, const uint32_t tag, const size_t set, int layer, const DAttItem& it, uint32_t* lds, const int* sblk,
                                              const int* srow, int* sdead, int slot) {
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, c16 = lane & 15;
  // The wave's keys and values are requested before anything else: the queries are not there yet in any case.  The values of one
  // chunk go to LDS: the third, for which there are no registers (requested when the first keys' registers were free they held
  // the wave up for 1.2 us), or the one with new positions, which is the wave's last and is patched there (by element in
  // registers that took 1.5 us).
  const int half = S::NH == 1 ? 0 : it.half;
  constexpr int HD = S::HD, NKF = S::WIDE ? 2 : 3;
  DfK<S> kf[NKF];
  DfV vf[3];
  auto v2 = [&](int j) { return lds + S::V2 + (S::WIDE ? wave * 4096 + (j == 2 ? 2048 : 0) : wave * 2048); };
  auto fresh = [&](int j) { return 64 * (it.c0 + wave + 8 * j) + 64 > it.len; };     // the chunk reaches new positions
  auto by_lds = [&](int j) { return j >= (S::WIDE ? 1 : 2) || fresh(j); };
  auto blocks = [&](int j, int (&boff)[4]) {
#pragma unroll
    for (int t = 0; t < 4; ++t) boff[t] = (__builtin_amdgcn_readfirstlane(sblk[(wave + 8 * j) * 4 + t]) * a.kv.nkv + it.kvh) * (16 * HD);
  };
  uint32_t touched = 0u;
  auto request = [&](auto jc) {
    constexpr int j = decltype(jc)::value;
    int boff[4];
    blocks(j, boff);
    if constexpr (j < NKF) {
      df_load_k<S>(a, layer, boff, lane, kf[j]);
    } else {                                               // its registers are not free yet: a word of each 128-byte line
      const uint32_t* p = (const uint32_t*)df_plane<S>(a, 2 * layer);
#pragma unroll
      for (int t = 0; t < 4; ++t)
        if (lane < HD / 4) touched |= p[(boff[t] >> 1) + lane * 32];
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) boff[t] += half * 1024;
    if (by_lds(j)) df_v_to_lds<S>(a, layer, boff, lane, v2(j));
    else df_load_v<S>(a, layer, boff, lane, vf[j]);
  };
  const bool live0 = it.valid && wave < it.nch, live1 = it.valid && wave + 8 < it.nch, live2 = it.valid && wave + 16 < it.nch;
  if (live0) request(std::integral_constant<int, 0>());
  if (live1) request(std::integral_constant<int, 1>());
  if (live2) request(std::integral_constant<int, 2>());
  uint32_t* Qs = lds;                                  // [16 rows][HD] operand words
  bf16_t* Kn = (bf16_t*)(lds + S::KN);                 // [16][HD] new keys
  bf16_t* Vn = (bf16_t*)(lds + S::VN);                 // [16][64] new values
  float* MO = (float*)(lds + S::MO);                   // [8 waves][16][64]
  float* ML = (float*)(lds + S::ML);                   // [8 waves][16][2]
  const int R = a.rows.R, G = a.nq / a.nkv, nqd = a.nq * HD, RG = R * G;
  const int r0 = 16 * it.rt, nrt = min(16, RG - r0);                         // first query row and rows of this tile
  const bool unew = (it.c0 + it.nch) * 64 > it.len;                          // the part reaches this launch's positions
  const uint32_t* q = a.q + set + (size_t)layer * a.st_q;
  const uint32_t* kvn = a.kvn + set + (size_t)layer * a.st_kvn;
  uint32_t* attn = a.attn + set + (size_t)layer * a.st_q;
  u64* att_p = a.att_p + (size_t)layer * a.st_att_p;
  const int* rowpos = srow + it.b * R;                 // positions of the sequence's rows
  const float sc2 = a.scale * 1.44269504088896340736f;
  const int qpos = r0 + c16 < RG ? rowpos[(r0 + c16) / G] : -1;              // position of the lane's query row
  // the row and the two dims that this thread finishes when the waves meet (looked up ahead of the wait): its row of the launch, head and parts
  const int row = tid >> 5, d0 = (tid & 31) * 2, row_j = min(r0 + row, RG - 1) / G;
  const int out_m = it.b * R + row_j, out_head = it.kvh * G + min(r0 + row, RG - 1) - row_j * G;
  const int np_row = it.valid ? df_parts(rowpos[row_j] + 1) : 0;             // parts that hold keys of the row
  bool bad = false;
  // ---- the queries of the tile's rows and this launch's keys / values of the kv head
  if (it.valid) {
    constexpr int NB = SB == 2 ? 1 : S::WIDE && SB == 18 ? 3 : 2;            // requests of four words that a thread keeps in flight: one flight for 4 / all 16 new rows
    const int nQ = nrt * HD, total = nQ + (unew ? it.nact * (HD + 64) : 0);  // <= 16 HD + 16 (HD + 64) words; of the values the item's 64 dims
    auto new_word = [&](int i, int& jn, int& which, int& dd) {               // word i of the new rows: a row's keys, then its values
      if (HD == 64) { jn = i >> 7; which = (i >> 6) & 1; dd = i & 63; }
      else { jn = i / (HD + 64); dd = i - jn * (HD + 64); which = dd >= HD; dd -= which ? HD : 0; }
    };
    const df_rsrc rs = df_make_rsrc(a.tw);
    const uint32_t q_off = (uint32_t)(q - a.tw), n_off = (uint32_t)(kvn - a.tw);
    for (int base = 0; base < total; base += 4 * NB * PBLOCK) {
      u32x4 v[NB];
      auto off = [&](uint32_t t, int u) -> uint32_t {
        const int idx = base + 4 * (u * PBLOCK + (int)t);
        if (idx < nQ) {
          const int r = r0 + (idx >> S::HDL), dd = idx & (HD - 1), j = r / G, gq = r - j * G;
          return 4u * (q_off + (uint32_t)((it.b * R + j) * nqd + (it.kvh * G + gq) * HD + dd));
        }
        int jn, which, dd;
        new_word(idx - nQ, jn, which, dd);
        return idx < total ? 4u * (n_off + (uint32_t)((((it.b * R + it.off + jn) * 2 + which) * a.nkv + it.kvh) * HD + (which ? half * 64 + dd : dd))) : 0xFFFFFFFFu;
      };
      bad = !poll_quads<NB>(rs, (uint32_t)tid, off, v, a.bar + 64, q + (size_t)it.b * R * nqd + it.kvh * G * HD) || bad;
#pragma unroll
      for (int u = 0; u < NB; ++u) {
        const int idx = base + 4 * (u * PBLOCK + tid);
        if (S::WIDE && idx < nQ) {
          uint32_t* to = Qs + (idx >> S::HDL) * S::QW + (idx & (HD - 1)) - ((idx & 4) >> 1);
          *(uint2*)to = make_uint2(__builtin_amdgcn_perm(v[u][1], v[u][0], 0x05040100u), __builtin_amdgcn_perm(v[u][3], v[u][2], 0x05040100u));
          *(uint2*)(to + 4) = make_uint2(__builtin_amdgcn_perm(v[u][1], v[u][0], 0x07060302u), __builtin_amdgcn_perm(v[u][3], v[u][2], 0x07060302u));
        } else if (idx < nQ) *(u32x4*)(Qs + (idx >> S::HDL) * S::QW + (idx & (HD - 1))) = v[u];
        else if (idx < total) {
          int jn, which, dd;
          new_word(idx - nQ, jn, which, dd);
          *(uint2*)((which ? Vn + jn * 64 : Kn + jn * HD) + dd) = make_uint2(__builtin_amdgcn_perm(v[u][1], v[u][0], 0x05040100u), __builtin_amdgcn_perm(v[u][3], v[u][2], 0x05040100u));
        }
      }
    }
    for (int idx = nQ + tid; idx < 16 * HD; idx += PBLOCK) Qs[(idx >> S::HDL) * S::QW + (idx & (HD - 1))] = 0u;       // padding rows of the tile
  }
  if (bad) *sdead = 1;
  __syncthreads();
  if (*sdead) return true;
  DF_STAMP(slot);
  DfRow rs = {-INFINITY, 0.f, {f32x4{0, 0, 0, 0}, f32x4{0, 0, 0, 0}, f32x4{0, 0, 0, 0}, f32x4{0, 0, 0, 0}}};
  if (S::WIDE) asm volatile("" ::"v"(touched));
  if (live0) {
    DfQ<S> qf;
    if constexpr (S::WIDE) {
      qf.at = Qs + c16 * S::QW + g * 8;
    } else {
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) frag_from_lds(Qs + c16 * S::QW + ks * 32 + g * 8, qf.hi[ks], qf.lo[ks]);
    }
    // All scores first, one maximum and one sum over the wave's chunks, then the values: a chain of reductions across lanes once, not once per chunk.
    // (The third round is not for rows in several parts.)
    f32x4 sc[3][4];
    float mx = -INFINITY;
    auto scores = [&](auto jc) {
      constexpr int j = decltype(jc)::value;
      const int kbase = 64 * (it.c0 + wave + 8 * j);
      DfK<S>& k = kf[j % NKF];
      if (fresh(j)) df_patch_k<S>(k, kbase, it.len, it.nact, Kn, lane);
      df_scores<S>(k, qf, kbase, j < 2 || qpos < DF_ONE_PART ? qpos : -1, fresh(j) || (j == 2 && it.nparts_b > 1), lane, sc[j]);
      mx = fmaxf(mx, df_max16(sc[j]));
    };
    scores(std::integral_constant<int, 0>());
    if (S::WIDE && live2) {
      int boff[4];
      blocks(2, boff);
      df_load_k<S>(a, layer, boff, lane, kf[0]);
    }
    if (live1) scores(std::integral_constant<int, 1>());
    if (live2) scores(std::integral_constant<int, 2>());
    rs.m = max_over_groups(mx) * sc2;
    const float base = rs.m == -INFINITY ? 0.f : rs.m;     // (the row sees none of these keys: every weight is 0)
    auto values = [&](auto jc) {
      constexpr int j = decltype(jc)::value;
      rs.l += df_weights(sc[j], sc2, base);
      if (by_lds(j)) df_v_from_lds(v2(j), 64 * (it.c0 + wave + 8 * j), it.len, it.nact, Vn, lane, vf[j]);
      df_values(vf[j], sc[j], rs);
    };
    values(std::integral_constant<int, 0>());
    if (live1) values(std::integral_constant<int, 1>());
    if (live2) values(std::integral_constant<int, 2>());
    rs.l = sum_over_groups(rs.l);
  }
  DF_STAMP2(3);
  // ---- the eight waves meet (fixed order: wave 0 .. 7); a single part's rows go out as operand words
  df_put_row<S>(rs, MO, ML, wave, lane);
  __syncthreads();
  df_loads_done();
  DF_STAMP2(4);
  if (it.valid && row < nrt) {
    if (it.part < np_row) {
      float mx, l, o[2];
      df_merge_row<S>(MO, ML, row, d0, mx, l, o);
      if (np_row == 1) {
        st_val2(attn + (size_t)out_m * nqd + out_head * HD + half * 64 + d0, operand_word(o[0] / l), operand_word(o[1] / l));
      } else {
        u64* pp = att_p + (((((size_t)out_m * a.nq + out_head) * a.NP + it.part) * S::NH + half) * 16 + (d0 >> 2)) * 6;
        st_words2(pp + (d0 & 2), __float_as_uint(o[0]), __float_as_uint(o[1]), tag);
        if (!(d0 & 2)) st_words2(pp + 4, __float_as_uint(mx), __float_as_uint(l), tag);
      }
    }
  }
  // ---- merge of the parts: of the tile's rows, the workgroup of part p finishes those with row index = p mod P, two dims a thread
  if (it.valid && it.nparts_b > 1) {
    const int P = it.nparts_b;
    const int first = ((it.part - r0) % P + P) % P;                          // first row of the tile this workgroup finishes
    const int qr = r0 + first + row * P;
    if (first + row * P < nrt) {
      const int j = qr / G, gq = qr - j * G, m = it.b * R + j, head = it.kvh * G + gq;
      const int np = df_parts(rowpos[j] + 1);
      if (np > 1) {
        const df_rsrc rs = df_make_rsrc(att_p);
        const uint32_t p_off = 8u * (uint32_t)(((m * a.nq + head) * a.NP * S::NH + half) * 96 + (d0 >> 2) * 6);
        float mx = -INFINITY, l = 0.f, o0 = 0.f, o1 = 0.f;
        for (int p0 = 0; p0 < np; p0 += DF_NPF) {
          u32x4 v[DF_NPF * 2];                               // per part: the two values; maximum and sum
          auto off = [&](uint32_t at, int i) -> uint32_t {
            return i / 2 < np - p0 ? at + (uint32_t)((p0 + i / 2) * (768 * S::NH) + (i % 2 ? 32 : (d0 & 2) * 8)) : 0xFFFFFFFFu;
          };
          bad = !poll_pairs<DF_NPF * 2>(rs, p_off, off, tag, v, a.bar + 64) || bad;
          float gm = mx;
#pragma unroll
          for (int p = 0; p < DF_NPF; ++p)
            if (p0 + p < np) gm = fmaxf(gm, __uint_as_float(v[2 * p + 1][0]));
          if (p0 > 0) {                                      // more than DF_NPF parts: rescale what is already summed
            const float e = df_exp2(mx - gm);
            l *= e;
            o0 *= e;
            o1 *= e;
          }
          mx = gm;
#pragma unroll
          for (int p = 0; p < DF_NPF; ++p)
            if (p0 + p < np) {
              const float e = df_exp2(__uint_as_float(v[2 * p + 1][0]) - mx);
              l = fmaf(__uint_as_float(v[2 * p + 1][2]), e, l);
              o0 = fmaf(__uint_as_float(v[2 * p][0]), e, o0);
              o1 = fmaf(__uint_as_float(v[2 * p][2]), e, o1);
            }
        }
        st_val2(attn + (size_t)m * nqd + head * HD + half * 64 + d0, operand_word(o0 / l), operand_word(o1 / l));
      }
    }
  }
  DF_STAMP(slot + 1);
  if (bad) *sdead = 1;
  __syncthreads();
  return *sdead != 0;
}

// ------------------------------------------------------------------------------------------------ the kernel
// The launch's arguments, read again from the kernel-argument segment through a pointer the compiler cannot see
// through.  The arguments are some 130 dwords; held in scalar registers across the layer loop they do not fit, and
// the compiler parks them in vector-register lanes (a readlane per use).  Every phase asks for the arguments anew,
// so only what that phase uses is live, and the loads hit the scalar cache.
__device__ __forceinline__ const DArgs& df_args() {
  auto p = __builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return *(const DArgs*)p;
}

// SB = 2, 4, 10, 16, 18: 2, 4, 6, 8, 10 rows in flight while it stages GEMM operands -- every slot costs instructions whether it is used or not, and a second
// flight costs a round trip, so the host picks the smallest SB whose single flight holds the launch's rows.
template <int SB>
__global__ void __launch_bounds__(PBLOCK) k_forward_dataflow(DArgs) {
  using S = DfNarrow;
#include "dataflow_body.h"
}
template <int SB>
__global__ void __launch_bounds__(PBLOCK) k_forward_wide(DArgs) {
  using S = DfWide;
#include "dataflow_body.h"
}

}  // namespace ssd
