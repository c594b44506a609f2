// Device-side helpers shared by the kernels of libssd (gfx950, wave64).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <utility>

namespace ssd {

constexpr int WAVE = 64;
constexpr int BLOCK = 256;            // threads per workgroup of every kernel here (4 waves)
constexpr int ATT_CHUNK = 64;         // keys per attention work item; chunk c covers positions [64c, 64c+64)

typedef uint16_t bf16_t;              // raw bf16 bits
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

__device__ __forceinline__ float bf16_to_f(bf16_t v) { return __uint_as_float(((uint32_t)v) << 16); }
// Round to nearest even with the gfx950 conversion instruction (two values per instruction).
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
typedef __attribute__((ext_vector_type(2))) float f32x2_t;
__device__ __forceinline__ uint32_t f2_to_bf16x2(float lo, float hi) {      // bits [15:0] = bf16(lo), [31:16] = bf16(hi)
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2_t{lo, hi}, bf16x2_t));
}
__device__ __forceinline__ bf16_t f_to_bf16(float f) { return (bf16_t)(f2_to_bf16x2(f, 0.f) & 0xFFFFu); }

// Storage types of activations / weights / KV: load as float, store from float.
struct F32 {
  typedef float T;
  static __device__ __forceinline__ float ld(const T* p) { return *p; }
  static __device__ __forceinline__ void st(T* p, float v) { *p = v; }
};
struct BF16 {
  typedef bf16_t T;
  static __device__ __forceinline__ float ld(const T* p) { return bf16_to_f(*p); }
  static __device__ __forceinline__ void st(T* p, float v) { *p = f_to_bf16(v); }
};

// Philox-4x32-10 (Salmon et al., SC'11).  Counter (slot, seq, step_lo, step_hi), key (seed_lo, seed_hi).
// Returns output word 0; the uniform of a slot is its top 24 bits times 2^-24.
__device__ __forceinline__ uint32_t philox_word0(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                                 uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const uint32_t hi0 = __umulhi(0xD2511F53u, c0), lo0 = 0xD2511F53u * c0;
    const uint32_t hi1 = __umulhi(0xCD9E8D57u, c2), lo1 = 0xCD9E8D57u * c2;
    c0 = hi1 ^ c1 ^ k0;
    c1 = lo1;
    c2 = hi0 ^ c3 ^ k1;
    c3 = lo0;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  return c0;
}
__device__ __forceinline__ float philox_uniform(uint64_t seed, uint32_t seq, uint64_t step, uint32_t slot) {
  const uint32_t w = philox_word0(slot, seq, (uint32_t)step, (uint32_t)(step >> 32), (uint32_t)seed,
                                  (uint32_t)(seed >> 32));
  return (float)(w >> 8) * 5.9604644775390625e-08f;   // exact: 24-bit integer times 2^-24
}

// ---------------------------------------------------------------------------------------------------
// Device-resident state of a paged KV cache (all pointers into caller-provided device memory).
struct KvView {
  int32_t* len;        // [max_seqs] cached positions
  int32_t* n_pend;     // [max_seqs] pending tokens not yet in the cache (1, or 2 for a draft that owes x_K)
  int32_t* pend;       // [max_seqs][2]
  int32_t* owned;      // [max_seqs] blocks owned
  int32_t* table;      // [max_seqs][mbps] block ids
  int32_t* free_stack; // [n_blocks]
  int32_t* ctl;        // [0] free_top  [1] state error bits (KV_ERR_*)  [2] arrival counter of the accept kernel
                       // [3] number of the next forward launch on this cache (the tag of its hand-over words)
                       // [4],[5] cycle counter of a captured cycle (low, high word of the random counter's step)
                       // [6] captured cycles that have been replayed (a draft's cache)
  uint32_t* err;       // sticky error word of the persistent forward kernels: DEV_ERR_* bits
  int32_t* mirror;     // host-mapped copy: [max_seqs][2] = (len, n_pend), then [2*max_seqs] = ctl[1], [2*max_seqs+1] = *err and the MIRROR_* words
  void* pool;
  int n_blocks, bt, mbps, max_seqs, pcap;
  int n_layers, nkv, hd;
};

// Words of the mirror behind the sequences' that say which launches are over: the number of the last forward that was given one, captured cycles.
constexpr int MIRROR_FORWARD = 2, MIRROR_CYCLE = 3, MIRROR_WORDS = 4;

constexpr int KV_ERR_POOL = 1;        // the device allocator ran out of blocks
constexpr int KV_ERR_ROLLBACK = 4;    // a rollback asked for more positions than the sequence holds (refused)
constexpr uint32_t DEV_ERR_TIMEOUT = 1u;   // a bounded wait inside a persistent forward gave up
constexpr uint32_t DEV_ERR_TAGS = 2u;      // the launch counter reached its limit: the workspace must be cleared
// Launch numbers tag the attention's partial results and the new keys' blocks of the barrier-free forward, in 32 bits.  The numbers that a
// cache takes end at 2^25, as ssd.h says: the host clears the workspace and restarts the numbering before that; a forward that
// still finds the limit reached does nothing and raises DEV_ERR_TAGS.
constexpr uint32_t TAG_LIMIT = (1u << 25) - 1u;

// Element offset of (layer, which(0=K,1=V), block, kv head, token in block, 0) in the pool.  Keys are stored
// [token][dim]; values [dim][token], so for values only tok == 0 (the head's base) is meaningful here.
__device__ __forceinline__ size_t kv_offset(const KvView& kv, int layer, int which, int blk, int head, int tok) {
  return ((((size_t)(layer * 2 + which) * kv.n_blocks + blk) * kv.nkv + head) * kv.bt + tok) * (size_t)kv.hd;
}

// All-reduce over the 16 lanes of a DPP row (lanes 16k .. 16k+15) with data-parallel primitives instead of LDS
// shuffles: pairs, quads (quad_perm), half rows (row_half_mirror), rows (row_mirror).  Every step combines a lane's
// value with the value of a lane of the complementary group, so all 16 lanes end with bit-identical results.
template <int CTRL>
__device__ __forceinline__ float dpp_f(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}
__device__ __forceinline__ float row16_sum(float v) {
  v += dpp_f<0xB1>(v);       // quad_perm [1,0,3,2]
  v += dpp_f<0x4E>(v);       // quad_perm [2,3,0,1]
  v += dpp_f<0x141>(v);      // row_half_mirror
  v += dpp_f<0x140>(v);      // row_mirror
  return v;
}

// Butterfly reductions over the 64 lanes of a wave: every lane ends with the same value, and the association order is fixed (lanes
// l ^ 32, l ^ 16, l ^ 8, l ^ 4, l ^ 2, l ^ 1), so results do not depend on anything but the inputs.  Without LDS shuffles, whose
// latency of more than a hundred cycles a step was most of a reduction.  (A rotation by 8 within 16 lanes is l ^ 8; one by 4 brings the
// value of l ^ 4 or of l ^ 12, which are the same after that step.)
template <typename OP>
__device__ __forceinline__ float wave_reduce(float v, OP op) {
  auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = op(__uint_as_float(a[0]), __uint_as_float(a[1]));
  a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = op(__uint_as_float(a[0]), __uint_as_float(a[1]));
  v = op(v, dpp_f<0x128>(v));          // row_ror:8
  v = op(v, dpp_f<0x124>(v));          // row_ror:4
  v = op(v, dpp_f<0x4E>(v));           // quad_perm [2,3,0,1]
  return op(v, dpp_f<0xB1>(v));        // quad_perm [1,0,3,2]
}
__device__ __forceinline__ float wave_sum(float v) { return wave_reduce(v, [](float x, float y) { return x + y; }); }
__device__ __forceinline__ float wave_max(float v) { return wave_reduce(v, [](float x, float y) { return fmaxf(x, y); }); }

// Inclusive prefix sum over the 64 lanes of a wave (integers: exact in any order): within rows of 16 lanes by row_shr, then the
// totals of the rows before.
template <int CTRL>
__device__ __forceinline__ unsigned long long dpp_u64(unsigned long long v) {
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, CTRL, 0xF, 0xF, true), hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(v >> 32), CTRL, 0xF, 0xF, true);
  return ((unsigned long long)(uint32_t)hi << 32) | (uint32_t)lo;
}
__device__ __forceinline__ unsigned long long lane_u64(unsigned long long v, int lane) {
  return ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), lane) << 32) | (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, lane);
}
__device__ __forceinline__ unsigned long long wave_inclusive_scan(unsigned long long v) {
  v += dpp_u64<0x111>(v);              // row_shr:1
  v += dpp_u64<0x112>(v);
  v += dpp_u64<0x114>(v);
  v += dpp_u64<0x118>(v);
  const unsigned long long r0 = lane_u64(v, 15), r1 = r0 + lane_u64(v, 31), r2 = r1 + lane_u64(v, 47);
  const int row = (threadIdx.x & 63) >> 4;
  return v + (row == 0 ? 0ull : row == 1 ? r0 : row == 2 ? r1 : r2);
}

// All-reduce over the four lanes l, l ^ 16, l ^ 32, l ^ 48 (the lanes of a matrix-core tile that hold one row).
__device__ __forceinline__ float max_over_groups(float v) {
  auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
}
__device__ __forceinline__ float sum_over_groups(float v) {
  auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(a[0]) + __uint_as_float(a[1]);
}

// --------------------------------------------------------------------------------------- bf16 / MFMA
// Activations are kept in fp32 and fed to the matrix core as a sum of two bf16 values, x = hi + lo with
// hi = the upper 16 bits of x and lo = bf16(x - hi): two MFMAs per weight fragment instead of one, which
// the weight-streaming regime does not notice, and activation rounding (2^-17 instead of 2^-9 relative)
// stops being the largest error of the bf16 path.  Weights are bf16 as stored.
struct SplitA {
  bf16x8 hi, lo;
};
__device__ __forceinline__ SplitA split_bf16(const u32x4 a, const u32x4 b) {
  const uint32_t x[8] = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
  uint32_t h[4], l[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint32_t u0 = x[2 * i], u1 = x[2 * i + 1];
    const uint32_t h0 = u0 & 0xFFFF0000u, h1 = u1 & 0xFFFF0000u;
    const float r0 = __uint_as_float(u0) - __uint_as_float(h0);       // exact
    const float r1 = __uint_as_float(u1) - __uint_as_float(h1);
    h[i] = (h0 >> 16) | h1;
    l[i] = f2_to_bf16x2(r0, r1);
  }
  SplitA s;
  s.hi = __builtin_bit_cast(bf16x8, u32x4{h[0], h[1], h[2], h[3]});
  s.lo = __builtin_bit_cast(bf16x8, u32x4{l[0], l[1], l[2], l[3]});
  return s;
}

// The same with hi rounded to nearest: lo is half as large, and so is what its own rounding leaves (2^-18 relative).  As many
// instructions; for operands that never leave the registers.
__device__ __forceinline__ SplitA split_bf16_near(const f32x4 a, const f32x4 b) {
  const float x[8] = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
  uint32_t h[4], l[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    h[i] = f2_to_bf16x2(x[2 * i], x[2 * i + 1]);
    l[i] = f2_to_bf16x2(x[2 * i] - __uint_as_float(h[i] << 16), x[2 * i + 1] - __uint_as_float(h[i] & 0xFFFF0000u));       // exact differences
  }
  SplitA s;
  s.hi = __builtin_bit_cast(bf16x8, u32x4{h[0], h[1], h[2], h[3]});
  s.lo = __builtin_bit_cast(bf16x8, u32x4{l[0], l[1], l[2], l[3]});
  return s;
}

// "Split rows": GEMM operand rows [M][K] kept as the matrix core takes them, for the kernels that serve many rows
// (gemm_tile.h).  Value x of (row, k) is stored as hi = upper 16 bits of x and lo = bf16(x - hi); the fragment of row
// tile mt = row / 16 and k-tile kt = k / 32 is 64 lanes x 8 bf16 with lane = row % 16 + 16 * ((k % 32) / 8), element k % 8:
// 1 KB of hi followed by 1 KB of lo, fragments ordered [mt][kt].  A wave loads a fragment with one contiguous 16-byte
// load per lane.  Index (in bf16 elements) of the hi value; the lo value is 512 elements further.
__device__ __forceinline__ size_t split_index(int row, int k, int KT) {
  return ((size_t)((row >> 4) * KT + (k >> 5)) * 2) * 512 + (size_t)(((row & 15) + 16 * ((k & 31) >> 3)) * 8 + (k & 7));
}
__device__ __forceinline__ void st_split_value(bf16_t* base, int KT, int row, int k, float x) {
  const uint32_t u = __float_as_uint(x), h = u & 0xFFFF0000u;
  const size_t i = split_index(row, k, KT);
  base[i] = (bf16_t)(h >> 16);
  base[i + 512] = f_to_bf16(x - __uint_as_float(h));
}

// Four consecutive values of a split row: the hi halves and the lo halves as 8 bytes each.
__device__ __forceinline__ uint2 hi_pairs(const f32x4 v) {             // upper 16 bits of four floats
  const uint32_t a = __float_as_uint(v[0]), b = __float_as_uint(v[1]), c = __float_as_uint(v[2]), d = __float_as_uint(v[3]);
  return make_uint2((a >> 16) | (b & 0xFFFF0000u), (c >> 16) | (d & 0xFFFF0000u));
}
__device__ __forceinline__ uint2 lo_pairs(const f32x4 v) {             // bf16 of what the upper halves leave over
  float r[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) r[i] = v[i] - __uint_as_float(__float_as_uint(v[i]) & 0xFFFF0000u);
  return make_uint2(f2_to_bf16x2(r[0], r[1]), f2_to_bf16x2(r[2], r[3]));
}

// Direct loads to LDS, 16 bytes a lane.  Through a buffer descriptor: after global_load_lds, which the compiler counts as a flat access to both
// memories, every wait that it places for a load or an LDS read is one for all of them, and the loads in flight ahead were waited for
// once per round of a loop.
typedef __amdgpu_buffer_rsrc_t rsrc_t;
__device__ __forceinline__ rsrc_t load_rsrc(const void* base) { return __builtin_amdgcn_make_buffer_rsrc((void*)base, (short)0, 0x7FFFFFF0, 0x00027000); }
__device__ __forceinline__ void load_to_lds(rsrc_t r, void* lds, int lane_off, int off) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)lds, 16, lane_off, off, 0, 0);
}

// f of the constants 0, 1, ..
template <typename F, int... I>
__device__ __forceinline__ void for_each_index(F f, std::integer_sequence<int, I...>) { (f(std::integral_constant<int, I>()), ...); }

__device__ __forceinline__ int ceil_div(int a, int b) { return (a + b - 1) / b; }

// Exclusive prefix sum of one int per thread over a workgroup of up to 1024 threads; w16: 16 entries of LDS.  Callers that
// use it twice put a barrier in between.
__device__ __forceinline__ int block_excl_scan(int v, int* w16, int* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  int inc = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int t = __shfl_up(inc, o, WAVE);
    if (lane >= o) inc += t;
  }
  if (lane == 63) w16[wave] = inc;
  __syncthreads();
  int base = 0, tot = 0;
  for (int i = 0; i < nw; ++i) {
    if (i < wave) base += w16[i];
    tot += w16[i];
  }
  *total = tot;
  return base + inc - v;
}

// The block bookkeeping of many sequences at once, one thread per sequence (whole workgroup calls; `in`: the thread has a
// sequence).  Sequences take from and give back to the free stack in ascending order of their thread, exactly as a serial
// walk over them would: a prefix sum of what the earlier ones take (give) says where on the stack a thread's blocks are.
// (One thread walking 64 sequences costs a chain of dependent memory round trips per sequence: 50 us and more.)
//
// kv_reserve_all: make `seq` own the blocks that cover `tokens` positions.  The blocks are handed out by all threads together
// (a prefill chunk of one sequence takes 64); scan: blockDim + 16 entries of LDS, slot: blockDim entries.
__device__ inline void kv_reserve_all(const KvView& kv, bool in, int seq, int tokens, int* scan, int* slot) {
  const int nt = blockDim.x, own = in ? kv.owned[seq] : 0;
  const int top = kv.ctl[0];
  const int need = in ? max(0, ceil_div(tokens, kv.bt) - own) : 0;
  const int want = min(need, max(0, kv.mbps - own));
  int total;
  const int before = block_excl_scan(want, scan + nt, &total);
  const int take = max(0, min(want, top - before));
  if (take < need) kv.ctl[1] = KV_ERR_POOL;
  if (take > 0) kv.owned[seq] = own + take;
  scan[threadIdx.x] = before + want;
  slot[threadIdx.x] = seq * kv.mbps + own - before;
  __syncthreads();                                         // every thread has read the stack's height
  for (int i = threadIdx.x; i < min(total, top); i += nt) {
    int lo = 0, hi = nt - 1;                               // the thread whose blocks include the i-th one
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (scan[mid] > i) hi = mid; else lo = mid + 1;
    }
    kv.table[slot[lo] + i] = kv.free_stack[top - 1 - i];
  }
  if (threadIdx.x == 0) kv.ctl[0] = max(0, top - total);
  __syncthreads();
}

// kv_truncate_all: truncate `seq` to new_len positions, returning whole blocks past it, highest table index first.
__device__ inline void kv_truncate_all(const KvView& kv, bool in, int seq, int new_len, int* w16) {
  const int own = in ? kv.owned[seq] : 0;
  const int top = kv.ctl[0];
  const int give = in ? max(0, own - ceil_div(new_len, kv.bt)) : 0;
  int total;
  const int before = block_excl_scan(give, w16, &total);
  for (int t = 0; t < give; ++t) {
    int32_t* slot = kv.table + seq * kv.mbps + own - 1 - t;
    kv.free_stack[top + before + t] = *slot;
    *slot = -1;
  }
  if (in) {
    if (give > 0) kv.owned[seq] = own - give;
    kv.len[seq] = new_len;
  }
  __syncthreads();
  if (threadIdx.x == 0) kv.ctl[0] = top + total;
  __syncthreads();
}

__device__ inline void kv_publish_flags(const KvView& kv) {
  kv.mirror[2 * kv.max_seqs] = kv.ctl[1];
  kv.mirror[2 * kv.max_seqs + 1] = (int32_t)*kv.err;
}
__device__ inline void kv_publish_seq(const KvView& kv, int seq) {
  kv.mirror[2 * seq] = kv.len[seq];
  kv.mirror[2 * seq + 1] = kv.n_pend[seq];
}
__device__ inline void kv_publish(const KvView& kv, int seq) {
  kv_publish_seq(kv, seq);
  kv_publish_flags(kv);
}
// After a forward: the next launch on this cache gets the next number (one thread, the kernel that follows the forward), and the host learns that this one is over.
// `launch`: 0 where no forward came before, else 2 p + 1 with the number p that goes into the mirror, 0 for none.  (One argument: another one costs a load of its own, 0.2
// us of each sampling kernel.)
__device__ inline void kv_publish_forward(const KvView& kv, uint32_t launch) {
  if (launch > 1u) kv.mirror[2 * kv.max_seqs + MIRROR_FORWARD] = (int32_t)(launch >> 1);
}
__device__ inline void kv_bump_launch(const KvView& kv, uint32_t launch) {
  const uint32_t t = (uint32_t)kv.ctl[3] + 1u;
  kv.ctl[3] = (int32_t)t;
  kv_publish_forward(kv, launch);
}

// Rows of one forward: row m belongs to sequence seq0 + m / R at offset j = m % R.
struct Rows {
  int32_t* pos;      // [M] position of the row
  int32_t* active;   // [M] 1 if the row's key/value is to be written
  int M, R, seq0;
};

}  // namespace ssd
