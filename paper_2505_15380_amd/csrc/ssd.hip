// libssd: host side of the C ABI declared in include/ssd.h.  Validates arguments, carves the caller's
// workspaces, and enqueues the kernels of one forward / acceptance step on the caller's stream.
#include "../../include/ssd.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <array>
#include <atomic>
#include <chrono>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>
#include <string>
#include <thread>
#include <type_traits>
#include <vector>

#include "attention.h"
#include "common.h"
#include "gemm.h"
#include "gemm_tile.h"
#include "persistent.h"
#include "resident.h"
#include "dataflow.h"
#include "small.h"
#include "sample.h"

using namespace ssd;

// ------------------------------------------------------------------------------------------------ errors
static thread_local std::string g_err;
static int fail(int code, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_err = buf;
  return code;
}
#define HIP_TRY(expr)                                                                      \
  do {                                                                                     \
    hipError_t e_ = (expr);                                                                \
    if (e_ != hipSuccess) return fail(SSD_EHIP, "%s: %s", #expr, hipGetErrorString(e_));   \
  } while (0)
#define LAUNCH_CHECK() HIP_TRY(hipGetLastError())

extern "C" const char* ssd_strerror(int code) {
  switch (code) {
    case SSD_OK: return "ok";
    case SSD_EINVAL: return "invalid argument";
    case SSD_ENOMEM: return "out of pool or buffer space";
    case SSD_EHIP: return "HIP error";
    case SSD_ENOSUP: return "unsupported shape";
    default: return "unknown error";
  }
}
extern "C" const char* ssd_last_error(void) { return g_err.c_str(); }

// ------------------------------------------------------------------------------------------------ profiling
static int g_prof_kind = -1;
static std::vector<std::pair<hipEvent_t, hipEvent_t>> g_prof_events;
struct ProfScope {                   // brackets the launches of one kernel family with a pair of events
  hipEvent_t stop = nullptr;
  hipStream_t st;
  ProfScope(int kind, hipStream_t s) : st(s) {
    if (kind != g_prof_kind) return;
    hipEvent_t a, b;
    if (hipEventCreate(&a) != hipSuccess) return;
    if (hipEventCreate(&b) != hipSuccess) { (void)hipEventDestroy(a); return; }
    (void)hipEventRecord(a, st);
    g_prof_events.emplace_back(a, b);
    stop = b;
  }
  ~ProfScope() { if (stop) (void)hipEventRecord(stop, st); }
};
enum { PROF_QKV = 0, PROF_ATTN = 1, PROF_O = 2, PROF_GATEUP = 3, PROF_DOWN = 4, PROF_HEAD = 5, PROF_PERSISTENT = 6 };

extern "C" int ssd_profile_begin(int kind) {
  if (kind < 0 || kind > 6) return fail(SSD_EINVAL, "profile kind %d out of range", kind);
  if (g_prof_kind >= 0) return fail(SSD_EINVAL, "a profile is already running");
  g_prof_kind = kind;
  return SSD_OK;
}
extern "C" int ssd_profile_end(double* total_ms, int* launches) {
  if (g_prof_kind < 0) return fail(SSD_EINVAL, "no profile is running");
  g_prof_kind = -1;
  double sum = 0;
  int n = 0;
  int rc = SSD_OK;
  for (auto& ev : g_prof_events) {
    float ms = 0;
    hipError_t e = hipEventSynchronize(ev.second);
    if (e == hipSuccess) e = hipEventElapsedTime(&ms, ev.first, ev.second);
    if (e != hipSuccess) rc = fail(SSD_EHIP, "profile events: %s", hipGetErrorString(e));
    else { sum += ms; ++n; }
    (void)hipEventDestroy(ev.first);
    (void)hipEventDestroy(ev.second);
  }
  g_prof_events.clear();
  if (total_ms) *total_ms = sum;
  if (launches) *launches = n;
  return rc;
}

// ------------------------------------------------------------------------------------------------ carving
struct Carver {
  char* base;
  size_t off = 0;
  explicit Carver(void* b) : base((char*)b) {}
  template <typename T>
  T* take(size_t n) {
    off = (off + 255) & ~(size_t)255;
    T* p = base ? (T*)(base + off) : nullptr;
    off += n * sizeof(T);
    return p;
  }
  size_t size() const { return (off + 255) & ~(size_t)255; }
};

static inline int cdiv(int a, int b) { return (a + b - 1) / b; }

// ------------------------------------------------------------------------------------------------ model
struct LayerW {
  const float *ln1, *bqkv, *ln2;
  const void *wqkv, *wo, *wgate, *wup, *wdown;
};
struct ssd_model {
  ssd_model_config c;
  int max_positions;
  const void* embed;
  const float* final_norm;
  const void* head;
  std::vector<LayerW> layers;
  const float2* rope;
  PLayer* dev_layers;
  std::vector<PLayer> host_layers;    // per-layer pointers; the persistent kernel needs them equally spaced
  size_t layer_stride = 0;            // bytes between consecutive layers' tensors (0: not equally spaced)
  size_t esize() const { return c.dtype == SSD_DTYPE_BF16 ? 2 : 4; }
  int n_qkv() const { return (c.n_q_heads + 2 * c.n_kv_heads) * c.head_dim; }
};

static size_t mat_elems(const ssd_model_config& c, int N, int K) {   // elements a matrix takes in the model workspace
  return c.dtype == SSD_DTYPE_BF16 ? (size_t)cdiv(N, 16) * 16 * K : (size_t)N * K;
}

static int check_config(const ssd_model_config* c, int max_positions) {
  if (!c) return fail(SSD_EINVAL, "null config");
  if (c->n_layers < 1 || c->d_model < 1 || c->n_q_heads < 1 || c->n_kv_heads < 1 || c->d_ffn < 1 || c->vocab < 1 ||
      c->n_embed < c->vocab || max_positions < 1 || !(c->rope_base > 1.0f) || !(c->rms_eps >= 0.0f))
    return fail(SSD_EINVAL, "bad model dimensions");
  if (c->dtype != SSD_DTYPE_FP32 && c->dtype != SSD_DTYPE_BF16) return fail(SSD_EINVAL, "bad dtype %d", c->dtype);
  if (c->head_dim != 32 && c->head_dim != 64 && c->head_dim != 128) return fail(SSD_ENOSUP, "head_dim must be 32, 64 or 128");
  if (c->n_q_heads % c->n_kv_heads) return fail(SSD_ENOSUP, "n_q_heads must be a multiple of n_kv_heads");
  if (c->d_model % 32 || (c->n_q_heads * c->head_dim) % 32 || c->d_ffn % 32)
    return fail(SSD_ENOSUP, "d_model, n_q_heads*head_dim and d_ffn must be multiples of 32");
  if (c->vocab > 16384) return fail(SSD_ENOSUP, "vocab > 16384");
  return SSD_OK;
}

// Lays the model workspace out; with base == nullptr only measures it.
static size_t model_layout(const ssd_model_config& c, int max_positions, void* base, ssd_model* m) {
  Carver cv(base);
  const size_t es = c.dtype == SSD_DTYPE_BF16 ? 2 : 4;
  const int d = c.d_model, nqkv = (c.n_q_heads + 2 * c.n_kv_heads) * c.head_dim, nqd = c.n_q_heads * c.head_dim;
  auto mat = [&](int N, int K) { return (const void*)cv.take<char>(mat_elems(c, N, K) * es); };
  const void* embed = cv.take<char>((size_t)c.n_embed * d * es);
  const float* fn = cv.take<float>(d);
  const void* head = mat(c.vocab, d);
  const float2* rope = cv.take<float2>((size_t)max_positions * (c.head_dim / 2));
  PLayer* dev_layers = cv.take<PLayer>(c.n_layers);
  if (m) { m->embed = embed; m->final_norm = fn; m->head = head; m->rope = rope; m->dev_layers = dev_layers; m->layers.resize(c.n_layers); }
  for (int l = 0; l < c.n_layers; ++l) {
    LayerW w;
    w.ln1 = cv.take<float>(d);
    w.wqkv = mat(nqkv, d);
    w.bqkv = cv.take<float>(nqkv);
    w.wo = mat(d, nqd);
    w.ln2 = cv.take<float>(d);
    w.wgate = mat(c.d_ffn, d);
    w.wup = mat(c.d_ffn, d);
    w.wdown = mat(d, c.d_ffn);
    if (!c.qkv_bias) w.bqkv = nullptr;
    if (m) m->layers[l] = w;
  }
  return cv.size();
}

extern "C" size_t ssd_model_workspace_bytes(const ssd_model_config* cfg, int max_positions) {
  if (check_config(cfg, max_positions) != SSD_OK) return 0;
  return model_layout(*cfg, max_positions, nullptr, nullptr);
}

static int put_matrix(const ssd_model_config& c, const void* src, const void* dst, int N, int K, hipStream_t st) {
  if (c.dtype == SSD_DTYPE_BF16) {
    const int ntiles = cdiv(N, 16);
    const size_t pieces = (size_t)ntiles * (K / 32) * 64;
    const int blocks = (int)std::min<size_t>((pieces + 255) / 256, 65535);
    hipLaunchKernelGGL(k_pack_bf16, dim3(blocks), dim3(256), 0, st, (const bf16_t*)src, (uint4*)dst, N, K, ntiles);
    LAUNCH_CHECK();
  } else {
    HIP_TRY(hipMemcpyAsync((void*)dst, src, (size_t)N * K * 4, hipMemcpyDeviceToDevice, st));
  }
  return SSD_OK;
}

extern "C" int ssd_model_create(const ssd_model_config* cfg, const void* const* dev_weights, int n_weights,
                                int max_positions, void* dev_model_ws, size_t ws_bytes, void* stream, ssd_model** out) {
  int rc = check_config(cfg, max_positions);
  if (rc) return rc;
  if (!dev_weights || !dev_model_ws || !out) return fail(SSD_EINVAL, "null argument");
  if (n_weights != 3 + 8 * cfg->n_layers) return fail(SSD_EINVAL, "expected %d weight pointers, got %d", 3 + 8 * cfg->n_layers, n_weights);
  for (int i = 0; i < n_weights; ++i) {
    const bool is_bias = i >= 3 && (i - 3) % 8 == 2;
    if (!dev_weights[i] && !(is_bias && !cfg->qkv_bias)) return fail(SSD_EINVAL, "weight pointer %d is null", i);
  }
  if ((uintptr_t)dev_model_ws & 255) return fail(SSD_EINVAL, "model workspace must be 256-byte aligned");
  const size_t need = model_layout(*cfg, max_positions, nullptr, nullptr);
  if (ws_bytes < need) return fail(SSD_ENOMEM, "model workspace: need %zu bytes, got %zu", need, ws_bytes);
  ssd_model* m = new (std::nothrow) ssd_model();
  if (!m) return fail(SSD_ENOMEM, "host allocation failed");
  m->c = *cfg;
  m->max_positions = max_positions;
  model_layout(*cfg, max_positions, dev_model_ws, m);
  hipStream_t st = (hipStream_t)stream;
  const ssd_model_config& c = *cfg;
  const size_t es = m->esize();
  const int d = c.d_model, nqkv = m->n_qkv(), nqd = c.n_q_heads * c.head_dim;
#define TRY_RC(x) do { rc = (x); if (rc) { delete m; return rc; } } while (0)
#define COPY(dst, src, bytes) do { hipError_t e_ = hipMemcpyAsync((void*)(dst), (src), (bytes), hipMemcpyDeviceToDevice, st); \
    if (e_ != hipSuccess) { delete m; return fail(SSD_EHIP, "copy of weights: %s", hipGetErrorString(e_)); } } while (0)
  COPY(m->embed, dev_weights[0], (size_t)c.n_embed * d * es);
  COPY(m->final_norm, dev_weights[1], (size_t)d * 4);
  TRY_RC(put_matrix(c, dev_weights[2], m->head, c.vocab, d, st));
  for (int l = 0; l < c.n_layers; ++l) {
    const void* const* w = dev_weights + 3 + 8 * l;
    const LayerW& L = m->layers[l];
    COPY(L.ln1, w[0], (size_t)d * 4);
    TRY_RC(put_matrix(c, w[1], L.wqkv, nqkv, d, st));
    if (c.qkv_bias) COPY(L.bqkv, w[2], (size_t)nqkv * 4);
    TRY_RC(put_matrix(c, w[3], L.wo, d, nqd, st));
    COPY(L.ln2, w[4], (size_t)d * 4);
    TRY_RC(put_matrix(c, w[5], L.wgate, c.d_ffn, d, st));
    TRY_RC(put_matrix(c, w[6], L.wup, c.d_ffn, d, st));
    TRY_RC(put_matrix(c, w[7], L.wdown, d, c.d_ffn, st));
  }
  {
    const int half = c.head_dim / 2, total = max_positions * half;
    hipLaunchKernelGGL(k_rope_table, dim3(cdiv(total, 256)), dim3(256), 0, st, (float2*)m->rope, max_positions, half,
                       (double)c.rope_base);
    hipError_t e_ = hipGetLastError();
    if (e_ != hipSuccess) { delete m; return fail(SSD_EHIP, "rope table: %s", hipGetErrorString(e_)); }
  }
  m->host_layers.resize(c.n_layers);
  for (int l = 0; l < c.n_layers; ++l) {
    const LayerW& L = m->layers[l];
    m->host_layers[l] = PLayer{L.wqkv, L.wo, L.wgate, L.wup, L.wdown, L.ln1, L.ln2, L.bqkv};
  }
  m->layer_stride = 1;
  if (c.n_layers > 1) {
    const size_t st = (const char*)m->host_layers[1].wqkv - (const char*)m->host_layers[0].wqkv;
    bool uniform = true;
    for (int l = 1; l < c.n_layers; ++l) {
      const PLayer &x = m->host_layers[l - 1], &y = m->host_layers[l];
      auto gap = [&](const void* p, const void* q) { return (size_t)((const char*)q - (const char*)p); };
      uniform = uniform && gap(x.wqkv, y.wqkv) == st && gap(x.wo, y.wo) == st && gap(x.wgate, y.wgate) == st &&
                gap(x.wup, y.wup) == st && gap(x.wdown, y.wdown) == st && gap(x.ln1, y.ln1) == st && gap(x.ln2, y.ln2) == st &&
                (!c.qkv_bias || gap(x.bqkv, y.bqkv) == st);
    }
    m->layer_stride = uniform ? st : 0;
  }
  {
    hipError_t e_ = hipMemcpyAsync(m->dev_layers, m->host_layers.data(), sizeof(PLayer) * c.n_layers, hipMemcpyHostToDevice, st);
    if (e_ == hipSuccess) e_ = hipStreamSynchronize(st);
    if (e_ != hipSuccess) { delete m; return fail(SSD_EHIP, "layer table: %s", hipGetErrorString(e_)); }
  }
#undef COPY
#undef TRY_RC
  *out = m;
  return SSD_OK;
}

extern "C" int ssd_model_destroy(ssd_model* m) {
  delete m;
  return SSD_OK;
}

// ------------------------------------------------------------------------------------------------ kv
constexpr int MAX_SPLITS = 16;   // capacity of the k-split partial buffer
constexpr int MAX_ROWS = 1024;
constexpr int MAX_PROMPT_ROWS = 4096;

struct ssd_kv {
  const ssd_model* m;
  KvView v;
  int max_seqs, max_rows, NC;
  int prompt_rows;                 // rows that the per-operator buffers have room for (at least max_seqs * max_rows)
  // workspace
  Rows rows;
  float *h, *q, *o_part, *ml_part, *part, *logits, *probs;
  void *xn, *attn, *act;
  int32_t* scratch_i;              // [2 * max_seqs]: n_accepted / next_token when the caller passes none
  // persistent-kernel buffers (one instance per layer, see persistent.h)
  float *p_h, *p_sumsq, *p_part, *p_att_o, *p_att_ml;
  bf16_t *p_hg, *p_q, *p_attn, *p_act;        // split operand rows: 2 bf16 per value
  int32_t* tickets;
  uint32_t* bar;
  unsigned long long* trace;       // [256][512] clock samples of the persistent kernel's barriers
  bool trace_on = false;
  int NP, p_rows;
  uint32_t bar_epoch = 0;          // grid barriers executed so far by the kernel with barriers (compared wrap-safe)
  uint32_t launch_no = 1;          // host's copy of ctl[3]: the number the next forward on this cache will read
  int persistent_wgs = 0;          // 0: the persistent kernel is not usable for this cache
  int cus = 0;                     // compute units of the device
  // workspace of the barrier-free forward (see dataflow.h); null when that kernel is not usable
  u64 *t_base = nullptr, *t_att_p, *t_part, *t_rowblk;
  uint32_t *t_h, *t_hg, *t_sq, *t_q, *t_kvn, *t_attn;
  size_t t_words = 0, t_attp_at = 0;     // words of it; words ahead of the attention's partials (GEMM operands are among them)
  int t_rows = 0, t_NP = 0;        // rows and attention parts that it has room for
  bool dataflow = false;
  bool small = false;              // fp32: a few rows as one launch, else one per operator
  bool wide = false;               // head size 128: the same forward in its wide form, else one launch per operator
  int mlp_tiles = 1;               // wide: k-tiles of the down projection that an MLP workgroup takes
  bool attn_whole = false;   // ssd_kv_last_forward_path tells launches whose attention is one part (4) from others (3) on this cache
  bool attn_mfma = true;     // per-operator path: matrix-core attention where it applies (SSD_ATTN=valu: the scalar kernel)
  int32_t* ticket_alt = nullptr;   // ssd_verify_noalloc: the commit's arrival counter in the library's static scratch
  // what of its launches other streams' may have to be kept from (resident.h); under g_resident_mutex but for the words that device code leaves in the mirror
  struct { ssd_kv* next = nullptr; bool listed = false, slow = false; int device = -1, wgs = 0; const void* stream = nullptr; uint32_t forward = 0, cycle = 0; } run;
  uint32_t forwards = 0, cycles = 0;      // such launches given a number so far: forwards by themselves, captured cycles (on the draft's cache)
  uint32_t publish = 0;            // the number that the kernel behind this forward leaves in the mirror, 0: none
  bool capturing = false;          // a cycle is being captured on this cache: no synchronisation, no fallback kernels
  int last_path = 0;               // 1 per-operator launches, 2 barrier kernel, 3 barrier-free kernel, 4 the same with attention without parts, 5 fp32 in one launch
  bool last_whole = false;
  int last_wgs = 0;                // workgroups of the last barrier-free forward; of the largest one of a cycle that is being captured
  int df_sb = 0;             // SSD_DF_FLIGHT=2|4|10|16|18: instantiation of the barrier-free forward up to 8 rows (0: chosen per launch)
  // host
  int32_t* mirror_host;
  std::vector<int> len_ub, npend_ub;
};

// Launches whose workgroups wait for each other, of all caches (resident.h).  One that does not fit beside what other streams still run is held back here, on the host,
// until they are over, which the kernels behind them leave in the caches' mirrors.  Nothing is asked of the other streams themselves, which may be being captured, be
// another thread's (hipStreamPerThread) or be gone: HIP (7.2) ends the process when it is asked about a stream that was destroyed, refuses to wait for an event of one that is
// being captured, and breaks off every capture when the device is waited for.  And a program with one stream pays nothing, where an event behind each launch
// takes 1.0 to 1.4 us of its stream's time (of 22 for the smallest forward).  us for a step of each of two streams in turn, with events and stream waits -> held back here:
// two 0.5B targets 669 -> 659 (one after the other 647), two drafts 166 -> 156 (144), a 0.5B target and the smallest one, which fit, 393 -> 323.  A launch that has been held back for RESIDENT_WAIT_MS, behind whatever else these streams
// have before theirs, is not admitted, nor are others while that lasts: the caller takes launches that do not wait.
// The mutex is held until the launch is enqueued, so that no other thread's comes in between.  Where a caller captures the calls, replays are not seen: there head size
// 128 and fp32, whose launches per operator can be replayed on any streams at once and any number of times, keep those; with head size 64 the graphs are the caller's to order.
static std::mutex g_resident_mutex;
static ssd_kv* g_resident = nullptr;                       // caches that have had such a launch
constexpr int RESIDENT_WAIT_MS = 1000;

// What tells streams apart: hipStreamPerThread is another one in each thread, hipStreamLegacy the default one.  (A handle that is used again after its stream was destroyed
// does no harm: hipStreamDestroy waits for the stream's work.)
static const void* resident_key(hipStream_t st) {
  static std::atomic<size_t> threads{0};
  thread_local const size_t thread = threads++;
  return st == hipStreamPerThread ? (const void*)(2 * thread + 1) : st == hipStreamLegacy ? nullptr : (const void*)st;
}

static bool resident_running(const ssd_kv* kv) {
  const volatile int32_t* w = kv->mirror_host + 2 * kv->max_seqs;
  return (((uint32_t)w[MIRROR_FORWARD] - kv->run.forward) & 0x40000000u) != 0 || (int32_t)((uint32_t)w[MIRROR_CYCLE] - kv->run.cycle) < 0;
}

struct ResidentLaunch {
  std::unique_lock<std::mutex> lock;
  bool admitted = true;                                    // false: launches that do not wait must do
  ResidentLaunch(ssd_kv* kv, hipStream_t st, int wgs, bool cycle = false) : lock(g_resident_mutex) {
    int device = -1;
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    if (hipGetDevice(&device) != hipSuccess) return;
    if (hipStreamIsCapturing(st, &cs) != hipSuccess) { (void)hipGetLastError(); return; }      // (the default stream beside a capture: the launch will say so)
    if (cs != hipStreamCaptureStatusNone) {                // replays in a caller's graph are not seen: only the forms that have always been captured there
      admitted = kv->capturing || !(kv->wide || kv->small);
      return;
    }
    const void* key = resident_key(st);
    std::chrono::steady_clock::time_point until{};
    while (!fits(kv, device, key, wgs)) {
      bool slow = false;
      for (ssd_kv* o = g_resident; o; o = o->run.next) slow = slow || (o->run.slow && other(o, kv, device, key));
      const auto now = std::chrono::steady_clock::now();
      if (until.time_since_epoch().count() == 0) until = now + std::chrono::milliseconds(RESIDENT_WAIT_MS);
      if (slow || now >= until) {
        for (ssd_kv* o = g_resident; o; o = o->run.next)
          if (other(o, kv, device, key)) o->run.slow = true;
        admitted = false;
        return;
      }
      std::this_thread::yield();
    }
    auto& run = kv->run;
    if (!run.listed) { run.listed = true; run.next = g_resident; g_resident = kv; }
    run.wgs = resident_running(kv) ? std::max(run.wgs, wgs) : wgs;      // (its earlier ones too, whatever stream they are on: the caller orders a cache's calls)
    run.slow = false;
    run.device = device;
    run.stream = key;
    if (cycle) { run.cycle = ++kv->cycles; return; }
    kv->forwards = (kv->forwards + 1) & 0x7FFFFFFFu;       // (31 bits reach the kernels)
    if (kv->forwards == 0) kv->forwards = 1;
    run.forward = kv->publish = kv->forwards;
  }
  // Does `o` run something that a launch on `kv` has to mind?
  static bool other(const ssd_kv* o, const ssd_kv* kv, int device, const void* key) {
    return o != kv && o->run.device == device && o->run.stream != key && resident_running(o);
  }
  static bool fits(const ssd_kv* kv, int device, const void* key, int wgs) {
    Resident running[64];
    int n = 0;
    for (const ssd_kv* o = g_resident; o; o = o->run.next) {
      if (!other(o, kv, device, key)) continue;
      if (n == 64) return false;
      running[n++] = {o->run.stream, o->run.wgs};
    }
    return n == 0 || resident_fits(running, n, key, wgs, kv->cus);
  }
};

static void resident_forget(ssd_kv* kv) {
  std::lock_guard<std::mutex> lock(g_resident_mutex);
  for (ssd_kv** p = &g_resident; *p; p = &(*p)->run.next)
    if (*p == kv) { *p = kv->run.next; return; }
}

// Shapes whose fp32 forward of a few rows is one launch (small.h).  (With head size 64 two chunks of keys and values do not fit the registers.)
// A workgroup of a kv head computes the projections of its G query heads, its key and its value two at a time, and every workgroup of gate / up the whole
// output projection, where the launches per operator have a workgroup for each: with wide rows and many heads the chain of those is the shorter one.  The line is a fit to
// 4 widths x 13 groupings x 2 ffn sizes x 3 launches (1 to 64 rows), time per operator over time in one launch: width 256, 8 heads over 8 / 4 / 2 / 1 kv heads
// 1.01 / 1.02 / 0.93 / 0.80, 6 over 2 1.00, 6 over 1 0.91, 4 over 1 1.03; width 192, 8 over 2 / 1 1.08 / 0.94, 6 over 1 1.02; width 128, 8 over 1 1.12; the
// two configurations 1.35 and 1.6.
static bool small_shape(const ssd_model_config& c) {
  const int group = c.n_q_heads / c.n_kv_heads;
  return c.dtype == SSD_DTYPE_FP32 && c.head_dim == SF_HD && c.d_model <= SF_MAX_D && c.n_q_heads * SF_HD <= SF_MAX_D && c.d_ffn <= SF_MAX_FFN &&
         group <= SF_MAX_GROUP && c.d_model * (c.n_q_heads + 3 * (cdiv(group + 2, 2) - 2)) <= 9 * 256;
}

// Rows of the per-operator buffers.  A cache for one sequence's prompts in the largest launches (max_seqs 1, max_rows 1024) takes launches of up to
// 4096 rows where attention needs no partials for them (prompt_chunk): 136 MB more for the 0.5B shape and 4096 positions.
static int prompt_capacity(const ssd_model* m, int max_seqs, int max_rows) {
  if (max_seqs != 1 || max_rows != MAX_ROWS || m->c.dtype != SSD_DTYPE_BF16 || m->c.head_dim == 32) return max_seqs * max_rows;
  return std::min(std::max(m->max_positions, MAX_ROWS), MAX_PROMPT_ROWS);
}

static size_t kv_layout(const ssd_model* m, int max_seqs, int max_rows, int n_blocks, int mbps, void* base, ssd_kv* kv) {
  const ssd_model_config& c = m->c;
  Carver cv(base);
  const int Mmax = max_seqs * max_rows, Wmax = prompt_capacity(m, max_seqs, max_rows);
  const int NC = cdiv(m->max_positions, ATT_CHUNK);
  const int nqd = c.n_q_heads * c.head_dim;
  int32_t* len = cv.take<int32_t>(max_seqs);
  int32_t* n_pend = cv.take<int32_t>(max_seqs);
  int32_t* pend = cv.take<int32_t>(2 * max_seqs);
  int32_t* owned = cv.take<int32_t>(max_seqs);
  int32_t* table = cv.take<int32_t>((size_t)max_seqs * mbps);
  int32_t* free_stack = cv.take<int32_t>(n_blocks);
  int32_t* ctl = cv.take<int32_t>(8);
  int32_t* rpos = cv.take<int32_t>(Wmax);
  int32_t* ract = cv.take<int32_t>(Wmax);
  int32_t* scratch_i = cv.take<int32_t>(2 * max_seqs);
  const int Mpad = cdiv(Wmax, 16) * 16;                    // operand buffers also serve as split rows: whole row tiles
  float* h = cv.take<float>((size_t)Wmax * c.d_model);
  void* xn = cv.take<float>((size_t)Mpad * c.d_model);
  float* q = cv.take<float>((size_t)Wmax * nqd);
  float* o_part = cv.take<float>((size_t)Mmax * c.n_q_heads * NC * c.head_dim);
  float* ml_part = cv.take<float>((size_t)Mmax * c.n_q_heads * NC * 2);
  void* attn = cv.take<float>((size_t)Mpad * nqd);
  float* part = cv.take<float>((size_t)MAX_SPLITS * Mmax * c.d_model);
  void* act = cv.take<float>((size_t)Mpad * c.d_ffn);
  float* logits = cv.take<float>((size_t)Mmax * c.vocab);
  float* probs = cv.take<float>((size_t)Mmax * c.vocab);
  const int NP = cdiv(m->max_positions, ATT_PART);
  const bool p_ok = c.dtype == SSD_DTYPE_BF16 && c.head_dim == 64;
  const int PR = p_ok ? std::min(Mmax, 16) : 0, L = c.n_layers;      // rows the persistent kernel can take
  float* p_h = cv.take<float>((size_t)(2 * L + 1) * PR * c.d_model);
  bf16_t* p_hg = cv.take<bf16_t>((size_t)(2 * L + 1) * PR * c.d_model * 2);
  float* p_sumsq = cv.take<float>((size_t)(2 * L + 1) * PR * (c.d_model / 32 + 1));
  bf16_t* p_q = cv.take<bf16_t>((size_t)L * PR * nqd * 2);
  bf16_t* p_attn = cv.take<bf16_t>((size_t)L * PR * nqd * 2);
  bf16_t* p_act = cv.take<bf16_t>((size_t)L * PR * c.d_ffn * 2);
  float* p_part = cv.take<float>((size_t)2 * L * P_MAX_SPLITS * PR * c.d_model);
  float* p_att_o = cv.take<float>((size_t)L * PR * c.n_q_heads * NP * 64);
  float* p_att_ml = cv.take<float>((size_t)L * PR * c.n_q_heads * NP * 2);
  int32_t* tickets = cv.take<int32_t>(std::max(c.d_model / 32 + 1, Mmax * c.n_kv_heads));
  uint32_t* bar = cv.take<uint32_t>(128);
  // words of the barrier-free forward: one block, zeroed at creation.  Two sets of 32-bit words, the attention's partials (words of 64 bits
  // from here on), the MLP's
  const bool small_ok = small_shape(c);
  const bool wide_ok = c.dtype == SSD_DTYPE_BF16 && c.head_dim == 128;
  const size_t TR = wide_ok ? std::min(Mmax, 16) : PR, SR = small_ok ? std::min(Mmax, SF_MAX_ROWS) : 0;
  const size_t s_set = (size_t)L * SR * (nqd + 2 * c.d_model + c.d_ffn);      // (32-bit words; two sets)
  const int HD = wide_ok ? 128 : 64, TNP = wide_ok ? df_parts(m->max_positions + 1) : NP;
  unsigned long long* trace = cv.take<unsigned long long>(TR ? 256 * 512 : 0);
  const size_t w_h = (size_t)(2 * L + 1) * TR * c.d_model, w_sq = (size_t)(2 * L + 1) * TR * (c.d_model / 8);
  const size_t w_q = (size_t)L * TR * nqd, w_kvn = (size_t)L * TR * 2 * c.n_kv_heads * HD;
  const size_t w_attp = (size_t)L * TR * c.n_q_heads * TNP * (HD / 64 * 96);
  const size_t w_part = (size_t)2 * (c.d_ffn / 32) * TR * c.d_model;     // (two buffers of fp32, at most twice the rows apart: df_part_pitch)
  const size_t t_words = small_ok ? s_set + SF_MAX_ROWS + 16 : w_h * 2 + w_sq + w_q * 2 + w_kvn + w_attp + w_part + 32;
  u64* t_base = cv.take<u64>(t_words);
  if (kv) {
    kv->t_base = t_base; kv->t_words = t_words; kv->t_rows = (int)TR; kv->t_NP = TNP;
    uint32_t* t = (uint32_t*)t_base;
    kv->t_h = t; t += w_h; kv->t_hg = t; t += w_h; kv->t_sq = t; t += w_sq; kv->t_q = t; t += w_q; kv->t_attn = t; t += w_q; kv->t_kvn = t;
    kv->t_attp_at = w_h * 2 + w_sq + w_q * 2 + w_kvn;      // (words of 64 bits ahead; 32-bit words of a set)
    kv->t_att_p = t_base + kv->t_attp_at;
    kv->t_part = kv->t_att_p + w_attp;
    kv->t_rowblk = kv->t_part + w_part;
    if (small_ok) { kv->t_rows = (int)SR; kv->t_attp_at = s_set; kv->t_rowblk = t_base + s_set; }

    kv->trace = trace;
    kv->p_h = p_h; kv->p_hg = p_hg; kv->p_sumsq = p_sumsq; kv->p_q = p_q; kv->p_attn = p_attn; kv->p_act = p_act; kv->p_part = p_part; kv->p_att_o = p_att_o;
    kv->p_att_ml = p_att_ml; kv->tickets = tickets; kv->bar = bar; kv->NP = NP; kv->p_rows = PR;
    kv->v.len = len; kv->v.n_pend = n_pend; kv->v.pend = pend; kv->v.owned = owned; kv->v.table = table;
    kv->v.free_stack = free_stack; kv->v.ctl = ctl;
    kv->rows.pos = rpos; kv->rows.active = ract;
    kv->scratch_i = scratch_i;
    kv->h = h; kv->xn = xn; kv->q = q; kv->o_part = o_part; kv->ml_part = ml_part; kv->attn = attn; kv->part = part;
    kv->act = act; kv->logits = logits; kv->probs = probs;
    kv->NC = NC;
    kv->prompt_rows = Wmax;
  }
  return cv.size();
}

extern "C" size_t ssd_kv_pool_bytes(const ssd_model* m, int n_blocks, int block_tokens) {
  if (!m || n_blocks < 1 || block_tokens < 1) return 0;
  return (size_t)m->c.n_layers * 2 * n_blocks * m->c.n_kv_heads * block_tokens * m->c.head_dim * m->esize();
}

extern "C" size_t ssd_kv_workspace_bytes(const ssd_model* m, int max_seqs, int max_rows, int n_blocks, int mbps) {
  if (!m || max_seqs < 1 || max_rows < 1 || n_blocks < 1 || mbps < 1) return 0;
  return kv_layout(m, max_seqs, max_rows, n_blocks, mbps, nullptr, nullptr);
}

extern "C" int ssd_kv_create(const ssd_model* m, int max_seqs, int max_rows, int n_blocks, int block_tokens, int mbps,
                             int pending_cap, void* dev_pool, size_t pool_bytes, void* dev_ws, size_t ws_bytes,
                             void* stream, ssd_kv** out) {
  if (!m || !dev_pool || !dev_ws || !out) return fail(SSD_EINVAL, "null argument");
  if (max_seqs < 1 || max_rows < 1 || n_blocks < 1 || block_tokens < 1 || mbps < 1)
    return fail(SSD_EINVAL, "bad cache dimensions");
  if (max_seqs * max_rows > MAX_ROWS) return fail(SSD_ENOSUP, "max_seqs*max_rows = %d exceeds %d", max_seqs * max_rows, MAX_ROWS);
  if (pending_cap != 1 && pending_cap != 2) return fail(SSD_EINVAL, "pending_cap must be 1 or 2");
  if (max_rows < pending_cap) return fail(SSD_EINVAL, "max_rows < pending_cap");
  if (((uintptr_t)dev_pool & 255) || ((uintptr_t)dev_ws & 255)) return fail(SSD_EINVAL, "buffers must be 256-byte aligned");
  const size_t need_pool = ssd_kv_pool_bytes(m, n_blocks, block_tokens);
  if (pool_bytes < need_pool) return fail(SSD_ENOMEM, "KV pool: need %zu bytes, got %zu", need_pool, pool_bytes);
  const size_t need_ws = kv_layout(m, max_seqs, max_rows, n_blocks, mbps, nullptr, nullptr);
  if (ws_bytes < need_ws) return fail(SSD_ENOMEM, "KV workspace: need %zu bytes, got %zu", need_ws, ws_bytes);
  ssd_kv* kv = new (std::nothrow) ssd_kv();
  if (!kv) return fail(SSD_ENOMEM, "host allocation failed");
  kv->m = m;
  kv->max_seqs = max_seqs;
  kv->max_rows = max_rows;
  kv_layout(m, max_seqs, max_rows, n_blocks, mbps, dev_ws, kv);
  KvView& v = kv->v;
  v.pool = dev_pool;
  v.n_blocks = n_blocks; v.bt = block_tokens; v.mbps = mbps; v.max_seqs = max_seqs; v.pcap = pending_cap;
  v.n_layers = m->c.n_layers; v.nkv = m->c.n_kv_heads; v.hd = m->c.head_dim;
  v.err = kv->bar + 64;
  hipError_t e = hipHostMalloc((void**)&kv->mirror_host, (2 * max_seqs + MIRROR_WORDS) * sizeof(int32_t), hipHostMallocMapped);
  if (e != hipSuccess) { delete kv; return fail(SSD_EHIP, "hipHostMalloc: %s", hipGetErrorString(e)); }
  memset(kv->mirror_host, 0, (2 * max_seqs + MIRROR_WORDS) * sizeof(int32_t));
  e = hipHostGetDevicePointer((void**)&v.mirror, kv->mirror_host, 0);
  if (e != hipSuccess) { (void)hipHostFree(kv->mirror_host); delete kv; return fail(SSD_EHIP, "hipHostGetDevicePointer: %s", hipGetErrorString(e)); }
  kv->len_ub.assign(max_seqs, 0);
  kv->npend_ub.assign(max_seqs, 0);
  const int n = std::max(std::max(n_blocks, max_seqs * mbps), max_seqs);
  hipLaunchKernelGGL(k_kv_init, dim3(cdiv(n, 256)), dim3(256), 0, (hipStream_t)stream, v);
  e = hipGetLastError();
  if (e == hipSuccess) e = hipMemsetAsync(kv->bar, 0, 128 * sizeof(uint32_t), (hipStream_t)stream);
  if (e == hipSuccess)
    e = hipMemsetAsync(kv->tickets, 0, sizeof(int32_t) * std::max(m->c.d_model / 32 + 1, max_seqs * max_rows * m->c.n_kv_heads),
                       (hipStream_t)stream);
  {
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) == hipSuccess && hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess)
      kv->cus = cus;                                       // (every path sizes its k-splits by it)
  }
  // The persistent forward needs: bf16 storage, head_dim 64, 16-token blocks, <= 16 query heads per kv head.
  kv->persistent_wgs = 0;
  if (e == hipSuccess && m->c.dtype == SSD_DTYPE_BF16 && m->c.head_dim == 64 && block_tokens == 16 && m->layer_stride &&
      m->c.n_q_heads / m->c.n_kv_heads <= 16 &&
      (size_t)n_blocks * m->c.n_kv_heads * 1024 < ((size_t)1 << 31)) {   // lane offsets into a K/V plane are 32-bit
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && cus >= 16) {
      const int want = std::max(32, cdiv(m->c.d_ffn / 16, 2));      // two gate/up tile pairs per workgroup
      kv->persistent_wgs = std::max(0, std::min(want, cus));        // one workgroup per CU at most: all co-resident
      kv->cus = cus;
    }
  }
  // Its wide form: head size 128, rows that a wave's share of the down projection and the staging area hold, and compute units for the MLP's items beside
  // QKV's and the output projection's, two to a workgroup, and some for attention.  An MLP workgroup takes as few k-tiles as that leaves room for.
  bool wide = false;
  if (e == hipSuccess && m->c.dtype == SSD_DTYPE_BF16 && m->c.head_dim == 128 && block_tokens == 16 && m->layer_stride && m->c.d_model <= DfWide::MAX_K && m->c.n_q_heads * 128 <= DfWide::MAX_K &&
      m->c.n_q_heads / m->c.n_kv_heads <= 16 && (size_t)n_blocks * m->c.n_kv_heads * 2048 < ((size_t)1 << 31)) {
    const int room = kv->cus - cdiv(m->n_qkv() / 32 + m->c.d_model / 32, 2) - 16;
    wide = room > 0 && cdiv(m->c.d_ffn / 32, room) <= 2 && (size_t)m->c.d_ffn * m->c.d_model * 2 < ((size_t)1 << 32) - 32;
    if (wide) kv->mlp_tiles = cdiv(m->c.d_ffn / 32, room);
  }
  const bool small = e == hipSuccess && small_shape(m->c) && block_tokens == 16 && m->layer_stride && kv->t_words < ((size_t)1 << 28) &&
                     (size_t)n_blocks * m->c.n_kv_heads * (64 * SF_HD) < ((size_t)1 << 31);      // (words, and a plane of the pool, are addressed by 32 bits of bytes)
  // The barrier-free forward additionally needs its word offsets to fit 32 bits; its words start as zeros.
  kv->dataflow = false;
  if (e == hipSuccess && (kv->persistent_wgs > 0 || wide || small) && kv->t_words > 0 && kv->t_words < ((size_t)1 << 32) && kv->t_attp_at < ((size_t)1 << 28) &&
      (size_t)kv->t_rows * m->c.n_q_heads * kv->t_NP * (wide ? 192 : 96) < ((size_t)1 << 28)) {      // (pairs of words are addressed by 32 bits of bytes: ahead of the parts, and in a layer's parts)
    e = hipMemsetAsync(kv->t_base, 0, kv->t_words * sizeof(u64), (hipStream_t)stream);
    const char* env = getenv("SSD_FORWARD");
    const bool on = !(env && strcmp(env, "barrier") == 0);
    kv->dataflow = on && !wide && !small;                  // (what a captured cycle needs of both its caches)
    kv->small = on && small;
    kv->wide = on && wide;
  }
  {
    const char* env = getenv("SSD_ATTN");
    kv->attn_mfma = !(env && strcmp(env, "valu") == 0);
    env = getenv("SSD_ATTN_WHOLE");
    kv->attn_whole = env ? (env[0] == '1' || (env[0] == '2' && pending_cap == 2)) : (pending_cap == 2);
    env = getenv("SSD_DF_FLIGHT");
    kv->df_sb = env ? atoi(env) : 0;
    if (kv->df_sb != 2 && kv->df_sb != 4 && kv->df_sb != 10 && kv->df_sb != 16 && kv->df_sb != 18) kv->df_sb = 0;
  }
  if (e != hipSuccess) { (void)hipHostFree(kv->mirror_host); delete kv; return fail(SSD_EHIP, "k_kv_init: %s", hipGetErrorString(e)); }
  *out = kv;
  return SSD_OK;
}

extern "C" int ssd_kv_destroy(ssd_kv* kv) {
  if (!kv) return SSD_OK;
  resident_forget(kv);
  if (kv->mirror_host) (void)hipHostFree(kv->mirror_host);
  delete kv;
  return SSD_OK;
}

// Error words that device code left in the host-mapped mirror (no synchronisation: what has been published so far).
// They are sticky until ssd_kv_clear_error.
static int kv_check_flags(const ssd_kv* kv) {
  const volatile int32_t* mh = kv->mirror_host;
  const int dev_err = mh[2 * kv->max_seqs + 1], st_err = mh[2 * kv->max_seqs];
  if (dev_err & (int)DEV_ERR_TIMEOUT)
    return fail(SSD_EHIP, "a bounded wait inside a persistent forward kernel timed out: results since then are void and "
                          "nothing was committed; call ssd_kv_clear_error before using this cache again");
  if (dev_err & (int)DEV_ERR_TAGS)
    return fail(SSD_EHIP, "the launch numbering of this cache is exhausted; call ssd_kv_clear_error");
  if (st_err & KV_ERR_ROLLBACK)
    return fail(SSD_EINVAL, "a rollback asked for more positions than the sequence held and was refused");
  if (st_err & KV_ERR_POOL) return fail(SSD_ENOMEM, "device allocator reported pool exhaustion");
  return SSD_OK;
}

// Bring the host's length bounds up to date with the device (synchronises the stream).
static int kv_refresh(ssd_kv* kv, hipStream_t st) {
  HIP_TRY(hipStreamSynchronize(st));
  for (int s = 0; s < kv->max_seqs; ++s) {
    kv->len_ub[s] = kv->mirror_host[2 * s];
    kv->npend_ub[s] = kv->mirror_host[2 * s + 1];
  }
  return kv_check_flags(kv);
}

// Re-zero everything the persistent kernels synchronise through and restart the launch numbering (stream-ordered).
static int kv_clear_sync_state(ssd_kv* kv, hipStream_t st) {
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  HIP_TRY(hipStreamIsCapturing(st, &cs));
  if (cs != hipStreamCaptureStatusNone) return fail(SSD_EINVAL, "the cache's launch numbering cannot be cleared inside a stream capture");
  HIP_TRY(hipMemsetAsync(kv->bar, 0, 128 * sizeof(uint32_t), st));
  HIP_TRY(hipMemsetAsync(kv->tickets, 0, sizeof(int32_t) * std::max(kv->m->c.d_model / 32 + 1, kv->max_seqs * kv->max_rows * kv->m->c.n_kv_heads), st));
  if (kv->t_base && kv->t_words) HIP_TRY(hipMemsetAsync(kv->t_base, 0, kv->t_words * sizeof(u64), st));
  hipLaunchKernelGGL(k_kv_clear_error, dim3(1), dim3(1), 0, st, kv->v);
  LAUNCH_CHECK();
  kv->launch_no = 1;
  kv->bar_epoch = 0;
  return SSD_OK;
}

// Before enqueuing `n` more forwards on the cache: the launch numbers they will read must stay below the limit.
static int kv_launch_guard(ssd_kv* kv, hipStream_t st, uint32_t n) {
  if (kv->launch_no + n < TAG_LIMIT) return SSD_OK;
  return kv_clear_sync_state(kv, st);
}

// Can sequences [seq0, seq0+B) each take R more positions?  Uses the host's upper bounds; refreshes once
// from the device before giving up.
static int kv_check_room(ssd_kv* kv, int seq0, int B, int R, hipStream_t st) {
  for (int attempt = 0; attempt < 2; ++attempt) {
    long blocks = 0;
    bool ok = true;
    for (int s = 0; s < kv->max_seqs; ++s) {
      const bool in = s >= seq0 && s < seq0 + B;
      const int tokens = kv->len_ub[s] + (in ? R : 0);
      const int nb = cdiv(tokens, kv->v.bt);
      if (in && (nb > kv->v.mbps || tokens > kv->m->max_positions)) ok = false;
      blocks += nb;
    }
    if (ok && blocks <= kv->v.n_blocks) return SSD_OK;
    if (attempt == 0) {
      int rc = kv_refresh(kv, st);
      if (rc) return rc;
    }
  }
  return fail(SSD_ENOMEM, "KV cache cannot hold %d more positions for sequences %d..%d", R, seq0, seq0 + B - 1);
}

// The sampler kernels are unrolled over a thread's entries of the vocabulary: 1, 8 or 16 (what is not needed is instructions to fetch
// and to pass over: one row of a vocabulary of 512 with its draw 8.1 us with 8, 4.9 with 1).
#define SAMPLER(kernel, V, blocks, st, ...)                                                                              \
  do {                                                                                                                   \
    if ((V) <= SBLOCK) hipLaunchKernelGGL(kernel<1>, dim3(blocks), dim3(SBLOCK), 0, st, __VA_ARGS__);                     \
    else if ((V) <= 8 * SBLOCK) hipLaunchKernelGGL(kernel<8>, dim3(blocks), dim3(SBLOCK), 0, st, __VA_ARGS__);            \
    else hipLaunchKernelGGL(kernel<16>, dim3(blocks), dim3(SBLOCK), 0, st, __VA_ARGS__);                                  \
  } while (0)

// ------------------------------------------------------------------------------------------------ forward
template <int EPI>
static int launch_gemm_f32(const GemmArgs& g, int items, hipStream_t st) {
  const int waves = std::min(GF_MAX_WAVES, std::max(4, cdiv(g.K / 16, 4)));      // the epilogue has 256 threads
  hipLaunchKernelGGL((k_gemm_f32<EPI>), dim3(items, cdiv(g.M, 16)), dim3(waves * WAVE), 0, st, g);
  LAUNCH_CHECK();
  return SSD_OK;
}

// The output of a bf16 GEMM (gemm_tile.h) cut into workgroups of rows x cols tiles and k-slices.
template <int EPI>
static TilePlan gemm_plan(const GemmArgs& g, int rows, int cols, int slices) {
  const int KT = g.K / 32, n_wt = EPI == EPI_SWIGLU ? 2 * cdiv(g.N, 16) : cdiv(g.N, 16);       // weight tiles (gate and up both count)
  TilePlan p;
  p.n_colb = cdiv(n_wt, cols);
  p.n_rowb = cdiv(cdiv(g.M, 16), rows);
  p.slice_kt = cdiv(KT, slices);
  p.n_slices = cdiv(KT, p.slice_kt);
  p.per_xcd = cdiv(p.n_colb * p.n_rowb * p.n_slices, 8);
  p.rows_xcd = p.cols_xcd = p.lg_per = p.lg_colg = 0;
  p.rows_inv = 0;
  return p;
}
// The XCDs' shares of a plan (runs so far): the placement for which their L2s fetch the least, of the runs and of the grids that give no XCD more
// workgroups than the runs do.  (Against the runs because such a grid can fetch twice as much: gate / up of 512 rows of the 0.5B shape, 61 x 4 blocks of
// 10 x 8 tiles, 74 MB in four row groups, the only ones that fit, and 34 in runs.  us a launch in a prompt, that grid -> runs: 200 rows 18.8 -> 17.3, 256
// 19.3 -> 17.9, 448 to 512 1.0 to 2.9 less, 832 and 896 0.4 and 0.7; 1024 rows of this shape and of the 1.5B shape, where the matrix cores are what
// counts, equal.  Grids that give an XCD up to an eighth more workgroups than a run fetch less still, and were from 1.8 us faster to 0.9 slower.)
// `xcd_cus` > 0 (a prompt's launches of more than 1024 rows, whose activations are far larger than the L2s): any grid that takes no more rounds of an XCD's compute
// units than the runs do.
static void place_tiles(TilePlan& p, int rt, int ct, int xcd_cus) {
  const long row = rt * 64, col = ct * 32;                 // bytes per k of a block's activations (hi + lo) and of its weights
  const int per_slice = p.n_colb * p.n_rowb, run = p.per_xcd, most = xcd_cus > 0 ? cdiv(run, xcd_cus) * xcd_cus : run;
  if (8 % p.n_slices) return;
  long best = 0;
  for (int x = 0; x < 8; ++x)
    for (int o = x * run, end = std::min(o + run, per_slice * p.n_slices), next; o < end; o = next) {
      next = std::min(end, (o / per_slice + 1) * per_slice);
      const int first = o % per_slice, last = (next - 1) % per_slice, cols = last / p.n_rowb - first / p.n_rowb + 1;
      best += cols * col + std::min(p.n_rowb, cols == 1 ? last - first + 1 : cols == 2 ? p.n_rowb - first % p.n_rowb + last % p.n_rowb + 1 : p.n_rowb) * row;
    }
  p.lg_per = __builtin_ctz(8 / p.n_slices);
  for (int lc = p.lg_per; lc >= 0; --lc) {
    const int r = cdiv(p.n_rowb, 1 << (p.lg_per - lc)), c = cdiv(p.n_colb, 1 << lc);
    const long bytes = p.n_slices * (cdiv(p.n_colb, c) * (p.n_rowb * row) + cdiv(p.n_rowb, r) * (p.n_colb * col));
    if (r * c > most || most > 4096 || r > 256 || bytes > best || (p.rows_xcd && bytes == best)) continue;      // (4096, 256: TilePlan's rows_inv)
    best = bytes;
    p.rows_xcd = r; p.cols_xcd = c; p.lg_colg = lc; p.rows_inv = (1u << 20) / r + 1;
    p.per_xcd = std::max(run, r * c);
  }
}
static int plan_wgs(const TilePlan& p) { return p.n_colb * p.n_rowb * p.n_slices; }

// More than 64 KB of dynamic LDS is opt-in, once per kernel and device; a static object per kernel.
struct LdsOptIn {
  std::atomic<u64> asked{0};                               // a bit per device
  hipError_t ask(const void* kernel, int bytes) {
    int dev = 0;
    if (hipError_t e = hipGetDevice(&dev); e != hipSuccess) return e;
    const u64 bit = dev < 64 ? 1ull << dev : 0;
    if (asked.load(std::memory_order_relaxed) & bit) return hipSuccess;
    const hipError_t e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e == hipSuccess) asked.fetch_or(bit, std::memory_order_relaxed);
    return e;
  }
};
// The kernel, the tile and the slices of the least estimated time.  A shape's three figures are us, fitted by least squares to the times of the
// layers' launches in prompts of 24 to 1024 rows of both model shapes (29 sizes each): of a launch, per k-tile, and per k-tile for each of a compute
// unit's workgroups.  Partial outputs cost their write at 4.2 TB/s and their read at 5.  The shape that is picked is 0.4 % (gate / up, output
// projection) to 1.4 % (QKV) slower on average than the fastest of 19 to 25 shapes at each size, up to 12 % where two are close; those that
// are left out were nowhere needed for that.  (Other widths of whole 64 columns follow the same figures; none of those was measured.  A kernel launched again and again by
// itself is up to 2 us faster than between the others, and not equally so: figures from such runs picked shapes that were slower in a forward.)
enum GemmKernel { KERNEL_KWAVE, KERNEL_BLOCK, KERNEL_TILE, KERNEL_TILE_DEEP };      // (deep: eight k-tiles in flight instead of four)
struct GemmShape { int rt, ct, w; GemmKernel kernel; float launch, per_kt, per_wg; };       // row tiles x column slots, waves
template <int EPI>
static auto gemm_shapes() {
  constexpr GemmKernel K = KERNEL_KWAVE, B = KERNEL_BLOCK, T = KERNEL_TILE, D = KERNEL_TILE_DEEP;
  if constexpr (EPI == EPI_SWIGLU)
    return std::array<GemmShape, 9>{{{2, 8, 4, B, 3.95f, 0.044f, 0.176f}, {4, 6, 4, B, 5.51f, 0.f, 0.227f}, {4, 8, 8, B, 5.51f, 0.f, 0.250f},
                                     {8, 16, 8, B, 3.87f, 0.f, 0.724f}, {4, 10, 4, T, 5.26f, 0.043f, 0.278f}, {8, 8, 8, T, 3.30f, 0.f, 0.436f},
                                     {8, 10, 8, T, 3.79f, 0.f, 0.532f}, {8, 12, 4, T, 7.84f, 0.f, 0.514f}, {16, 10, 8, T, 5.12f, 0.f, 0.895f}}};
  else if constexpr (EPI == EPI_PARTIAL)
    return std::array<GemmShape, 10>{{{2, 4, 8, K, 3.02f, 0.017f, 0.115f}, {4, 6, 8, B, 3.67f, 0.014f, 0.195f}, {4, 8, 8, B, 3.67f, 0.023f, 0.206f},
                                      {8, 12, 8, B, 4.73f, 0.f, 0.480f}, {8, 6, 8, T, 3.86f, 0.f, 0.289f}, {8, 7, 8, T, 4.20f, 0.f, 0.298f},
                                      {8, 8, 8, T, 4.17f, 0.f, 0.326f}, {2, 2, 2, D, 2.81f, 0.023f, 0.066f}, {4, 3, 4, D, 2.98f, 0.001f, 0.143f},
                                      {4, 4, 4, D, 2.74f, 0.f, 0.155f}}};
  else if constexpr (EPI == EPI_QKV)
    return std::array<GemmShape, 9>{{{1, 2, 8, K, 3.38f, 0.f, 0.066f}, {2, 2, 8, K, 3.86f, 0.f, 0.081f}, {2, 4, 8, K, 5.02f, 0.f, 0.099f},
                                     {3, 4, 8, K, 4.47f, 0.f, 0.147f}, {4, 4, 8, K, 6.19f, 0.f, 0.132f}, {4, 8, 8, B, 6.65f, 0.221f, 0.f},
                                     {4, 4, 4, T, 4.88f, 0.039f, 0.148f}, {4, 6, 4, T, 5.77f, 0.091f, 0.143f}, {3, 2, 3, D, 3.26f, 0.008f, 0.109f}}};
  else
    return std::array<GemmShape, 8>{{{1, 2, 8, K, 3.18f, 0.f, 0.063f}, {2, 2, 2, D, 3.35f, 0.f, 0.083f}, {2, 3, 2, D, 3.36f, 0.011f, 0.102f},
                                     {2, 4, 2, D, 4.31f, 0.004f, 0.103f}, {3, 2, 3, D, 2.85f, 0.f, 0.117f}, {4, 3, 4, D, 3.67f, 0.f, 0.157f},
                                     {4, 4, 4, D, 4.94f, 0.f, 0.144f}, {4, 6, 4, D, 4.59f, 0.221f, 0.f}}};
}
// Launches of more than 1024 rows, which only prompts have: a compute unit then has several workgroups whatever the tile, so the tiles are those of four
// waves that leave room for a second workgroup, whose matrix instructions hide the first one's operands and epilogue (gate / up, down), and wider
// ones than a single round wants (QKV, output projection).  Figures as above, fitted to 1100 to 4096 rows of the 0.5B shape and 1100 to 3000 of the
// 1.5B shape (14 sizes, 9 to 25 shapes each): the shape picked is 0.4 to 0.7 us a launch slower on average than the fastest, 3 at most.  us a layer against
// what the figures above pick, at 4096 rows of width 896 and at 3000 of 1536: gate / up -11.4 and -6.8, down 0.5 and -13.4, QKV -6.0 and -7.6, output projection
// -10.3 and -7.4.  (At 65 to 1024 rows these shapes are within 1 us of those picked above, mostly slower.)
template <int EPI>
static auto gemm_shapes_prompt() {
  constexpr GemmKernel B = KERNEL_BLOCK, T = KERNEL_TILE, D = KERNEL_TILE_DEEP;
  if constexpr (EPI == EPI_SWIGLU)
    return std::array<GemmShape, 3>{{{8, 10, 4, T, 13.82f, 0.f, 0.265f}, {8, 12, 4, T, 6.78f, 0.055f, 0.325f}, {12, 8, 4, T, 0.f, 0.542f, 0.266f}}};
  else if constexpr (EPI == EPI_PARTIAL)
    return std::array<GemmShape, 5>{{{8, 7, 8, T, 7.06f, 0.f, 0.259f}, {8, 8, 8, T, 8.74f, 0.f, 0.264f}, {8, 10, 4, T, 2.09f, 0.105f, 0.306f},
                                     {8, 12, 4, T, 3.85f, 0.105f, 0.326f}, {12, 8, 4, T, 3.27f, 0.095f, 0.351f}}};
  else if constexpr (EPI == EPI_QKV)
    return std::array<GemmShape, 6>{{{4, 6, 4, T, 3.27f, 0.001f, 0.218f}, {4, 8, 8, B, 4.68f, 0.f, 0.228f}, {8, 6, 8, T, 5.44f, 0.142f, 0.192f},
                                     {8, 8, 8, T, 5.95f, 0.016f, 0.323f}, {8, 10, 8, T, 5.66f, 0.214f, 0.227f}, {16, 8, 8, T, 6.9f, 0.f, 0.605f}}};
  else
    return std::array<GemmShape, 5>{{{4, 4, 4, D, 3.49f, 0.007f, 0.212f}, {4, 6, 4, D, 6.01f, 0.f, 0.215f}, {4, 8, 4, T, 1.62f, 0.244f, 0.139f},
                                     {8, 6, 8, T, 8.9f, 0.089f, 0.184f}, {8, 7, 8, T, 4.99f, 0.24f, 0.139f}}};
}
// Sizes whose k range is shorter than eight k-tiles, and k-split outputs of a width that is no multiple of 64, keep the shapes that they had
// before: no such size was in the fit, no configuration has one, and the tests of ragged tiles hold each of them to its shape here.  (This costs a user of such
// a width time: at 23 of the tests' sizes the shapes above were mostly the faster ones, by 0 to 30 %.)
template <int EPI>
static auto gemm_shapes_ragged() {
  constexpr GemmKernel B = KERNEL_BLOCK, T = KERNEL_TILE;
  if constexpr (EPI == EPI_SWIGLU)
    return std::array<GemmShape, 9>{{{4, 8, 8, B, 0.f, 0.074f, 0.262f}, {4, 10, 4, B, 0.f, 0.032f, 0.448f}, {5, 6, 5, B, 0.f, 0.117f, 0.272f},
                                     {7, 6, 7, B, 0.f, 0.013f, 0.397f}, {4, 8, 4, T, 0.f, 0.179f, 0.215f}, {8, 8, 8, T, 0.f, 0.153f, 0.377f},
                                     {8, 10, 8, T, 0.f, 0.196f, 0.455f}, {8, 12, 4, T, 0.f, 0.274f, 0.482f}, {16, 10, 8, T, 0.f, 0.088f, 0.960f}}};
  else if constexpr (EPI == EPI_PARTIAL)
    return std::array<GemmShape, 6>{{{4, 4, 4, B, 0.f, 0.027f, 0.145f}, {4, 8, 8, B, 0.f, 0.024f, 0.223f}, {8, 7, 8, B, 0.f, 0.f, 0.369f},
                                     {8, 8, 8, T, 0.f, 0.031f, 0.368f}, {16, 6, 8, T, 0.f, 0.f, 0.586f}, {16, 8, 8, T, 0.f, 0.f, 0.682f}}};
  else
    return std::array<GemmShape, 3>{{{4, 4, 4, T, 0.f, 0.f, 0.200f}, {4, 6, 4, T, 0.f, 0.f, 0.233f}, {4, 8, 4, T, 0.f, 0.f, 0.267f}}};
}
template <int EPI, int RT, int CT, int WR, int WC, int NBUF>
static int launch_gemm_block(const GemmArgs& g, const TilePlan& p, hipStream_t st) {
  constexpr int LDS = NBUF * (2 * RT + CT) * 1024;
  static LdsOptIn lds;
  if (hipError_t e = lds.ask((const void*)k_gemm_block<EPI, RT, CT, WR, WC, NBUF>, LDS); e != hipSuccess)
    return fail(SSD_EHIP, "hipFuncSetAttribute: %s", hipGetErrorString(e));
  hipLaunchKernelGGL((k_gemm_block<EPI, RT, CT, WR, WC, NBUF>), dim3(8 * p.per_xcd), dim3(WR * WC * 64), LDS, st, g, p);
  LAUNCH_CHECK();
  return p.n_slices;
}
struct GemmPick {
  GemmKernel kernel;
  int rt, ct, w;                                           // row tiles x column slots of a workgroup; its waves (k_gemm_tile)
  TilePlan p;
  double us = 0;                                           // the estimate, where the pick is by estimate
};
template <int EPI, typename SHAPES>
static GemmPick pick_gemm_shape(const GemmArgs& g, int cus, int max_slices, const SHAPES& shapes) {
  const int KT = g.K / 32;
  GemmShape c{};
  double best_us = 0;
  TilePlan p{};
  for (const GemmShape& s : shapes)
    for (int ns = 1; ns <= std::min(8, max_slices) && (ns == 1 || KT / ns >= 7); ns *= 2) {
      const TilePlan q = gemm_plan<EPI>(g, s.rt, s.ct, ns);
      const double us = s.launch + q.slice_kt * (s.per_kt + s.per_wg * cdiv(plan_wgs(q), cus)) + (EPI == EPI_PARTIAL ? (double)q.n_slices * g.M * g.N * 4 * 0.44e-6 : 0.0);
      if (!c.w || us < best_us) { c = s; best_us = us; p = q; }
    }
  return {c.kernel, c.rt, c.ct, c.w, p, best_us};
}
template <int EPI>
static GemmPick pick_gemm_ragged(const GemmArgs& g, int cus, int max_slices) {
  if constexpr (EPI == EPI_QKV) {
    const TilePlan small = gemm_plan<EPI>(g, 4, 4, 1);
    if (plan_wgs(small) <= cus + cus / 4) return {KERNEL_BLOCK, 4, 4, 4, small};
    return {KERNEL_BLOCK, 4, 8, 8, gemm_plan<EPI>(g, 4, 8, 1)};
  } else {
    GemmPick c = pick_gemm_shape<EPI>(g, cus, max_slices, gemm_shapes_ragged<EPI>());
    if (EPI == EPI_RESID && plan_wgs(c.p) <= cus) c.kernel = KERNEL_TILE_DEEP;
    return c;
  }
}
template <int EPI>
static int launch_gemm_tile(const GemmArgs& g, const GemmPick& c, hipStream_t st) {
  const TilePlan& p = c.p;
#define BLOCK(RT, CT, WR, WC, NBUF) \
  if (c.kernel == KERNEL_BLOCK && c.rt == RT && c.ct == CT) return launch_gemm_block<EPI, RT, CT, WR, WC, NBUF>(g, p, st)
#define TILE_OF(KERNEL, RT, CT, W, NBUF, UA, MINB)                                                                         \
  if (c.kernel == KERNEL && c.rt == RT && c.ct == CT && c.w == W) {                                                        \
    hipLaunchKernelGGL((k_gemm_tile<EPI, RT / W, CT, W, NBUF, UA, MINB>), dim3(8 * p.per_xcd), dim3(W * 64), 0, st, g, p); \
    LAUNCH_CHECK();                                                                                                        \
    return EPI == EPI_RESID ? p.n_colb : p.n_slices;                                                                       \
  }
#define TILE(RT, CT, W) TILE_OF(KERNEL_TILE, RT, CT, W, 4, 4, RT == 16 ? 1 : 2)
#define TILE_DEEP(RT, CT, W) TILE_OF(KERNEL_TILE_DEEP, RT, CT, W, 8, 8, 1)
#define TILE_PAIR(RT, CT, W) TILE_OF(KERNEL_TILE, RT, CT, W, 3, 2, 2)       // (two k-tiles of activations in flight: more do not fit the registers beside a second workgroup's)
  if constexpr (EPI == EPI_QKV) {
    BLOCK(4, 4, 4, 1, 5); BLOCK(4, 8, 4, 2, 5);
    TILE(4, 4, 4) TILE(4, 6, 4) TILE_DEEP(3, 2, 3) TILE(8, 6, 8) TILE(8, 8, 8) TILE(8, 10, 8) TILE(16, 8, 8)
  } else if constexpr (EPI == EPI_SWIGLU) {
    BLOCK(2, 8, 2, 2, 5); BLOCK(4, 6, 4, 1, 5); BLOCK(4, 8, 4, 2, 5); BLOCK(4, 10, 4, 1, 5); BLOCK(5, 6, 5, 1, 5); BLOCK(7, 6, 7, 1, 5); BLOCK(8, 16, 4, 2, 4);
    TILE(4, 8, 4) TILE(4, 10, 4) TILE(8, 8, 8) TILE(8, 10, 8) TILE(16, 10, 8)
    TILE_PAIR(8, 10, 4) TILE_PAIR(8, 12, 4) TILE_PAIR(12, 8, 4)
  } else if constexpr (EPI == EPI_PARTIAL) {
    BLOCK(4, 4, 4, 1, 5); BLOCK(4, 6, 4, 2, 5); BLOCK(4, 8, 4, 2, 5); BLOCK(8, 7, 8, 1, 4); BLOCK(8, 12, 4, 2, 4);
    TILE(8, 6, 8) TILE(8, 7, 8) TILE(8, 8, 8) TILE(16, 6, 8) TILE(16, 8, 8)
    TILE_PAIR(8, 10, 4) TILE_PAIR(8, 12, 4) TILE_PAIR(12, 8, 4)
    TILE_DEEP(2, 2, 2) TILE_DEEP(4, 3, 4) TILE_DEEP(4, 4, 4)
  } else if constexpr (EPI == EPI_RESID) {
    TILE(4, 4, 4) TILE(4, 6, 4) TILE(4, 8, 4) TILE(8, 6, 8) TILE(8, 7, 8)
    TILE_DEEP(2, 2, 2) TILE_DEEP(2, 3, 2) TILE_DEEP(2, 4, 2) TILE_DEEP(3, 2, 3) TILE_DEEP(4, 3, 4) TILE_DEEP(4, 4, 4) TILE_DEEP(4, 6, 4) TILE_DEEP(4, 8, 4)
  }
#undef BLOCK
#undef TILE_OF
#undef TILE
#undef TILE_DEEP
#undef TILE_PAIR
  return fail(SSD_EHIP, "no GEMM kernel of %d x %d tiles and %d waves", c.rt, c.ct, c.w);
}

// What a bf16 GEMM runs, from the sizes alone.
// By the estimate above from 17 rows on (gate / up, whose few-row kernel reads sums of squares over 16 columns: from 65 on).
// Fewer rows: k_gemm_kwave with the smallest tile that leaves no more workgroups than compute units, or else the largest usable one.  What bounds it
// is how long a workgroup's operand stream takes, so the work is spread as far as one round of workgroups allows; k-split outputs get 8 slices
// (4 where k is short) while that round lasts.
// (Sizes outside the fit: gate / up and k-split outputs of up to 64 rows, QKV and output projection up to 512, and the output projection as long
// as tiles of 4 x 4 fill one round.)
template <int EPI>
static GemmPick pick_gemm_cut(const GemmArgs& g, int cus, int max_slices) {
  const int KT = g.K / 32, MT = cdiv(g.M, 16);
  constexpr bool whole_k = EPI == EPI_QKV || EPI == EPI_RESID;
  if (g.M > MAX_ROWS) return pick_gemm_shape<EPI>(g, cus, max_slices, gemm_shapes_prompt<EPI>());
  if (KT >= 8 && (max_slices == 1 || g.N % 64 == 0)) {
    if (MT > (EPI == EPI_SWIGLU ? 4 : 1)) return pick_gemm_shape<EPI>(g, cus, max_slices, gemm_shapes<EPI>());
  } else if (MT > (whole_k ? 32 : 4) && !(EPI == EPI_RESID && plan_wgs(gemm_plan<EPI>(g, 4, 4, 1)) <= cus)) {
    return pick_gemm_ragged<EPI>(g, cus, max_slices);
  }
  static const int shapes[][2] = {{1, 2}, {2, 2}, {1, 4}, {3, 2}, {1, 6}, {2, 4}, {2, 6}, {3, 4}, {4, 4}, {3, 6}, {4, 6}};   // by area
  auto usable = [&](const int* c) {
    return c[0] <= MT && (EPI == EPI_SWIGLU ? c[0] < 4 || c[1] == 6 : c[1] <= 4);
  };
  GemmPick c{KERNEL_KWAVE, 0, 0, 8, {}};
  for (int ns = max_slices >= 8 && KT >= 64 ? 8 : max_slices >= 4 && KT >= 16 ? 4 : 1; ns >= 1 && !c.rt; ns /= 2)
    for (const auto& t : shapes) {
      if (!usable(t)) continue;
      const TilePlan q = gemm_plan<EPI>(g, t[0], t[1], ns);
      if (plan_wgs(q) <= cus) { c.rt = t[0]; c.ct = t[1]; c.p = q; break; }
    }
  if (!c.rt)                                             // more than one round whatever the tile: the largest usable one
    for (const auto& t : shapes)
      if (usable(t)) { c.rt = t[0]; c.ct = t[1]; c.p = gemm_plan<EPI>(g, c.rt, c.ct, 1); }
  return c;
}
template <int EPI>
static GemmPick pick_gemm(const GemmArgs& g, int cus, int max_slices) {
  GemmPick c = pick_gemm_cut<EPI>(g, cus, max_slices);
  place_tiles(c.p, c.rt, c.ct, g.M > MAX_ROWS ? cus / 8 : 0);
  return c;
}
// Slices of k-split outputs of `rows` rows in the buffer of partials, which has room for MAX_SPLITS of `capacity` rows.
static int partial_slices(int capacity, int rows) { return std::min(MAX_SPLITS, std::max(1, MAX_SPLITS * capacity / rows)); }
// Does a prompt's down projection add the residual and leave the sums of squares itself, as the output projection does, so that no add + norm kernel runs ahead of the
// next layer's QKV projection, which then divides by the r.m.s.?  For that it cannot be k-split.  Where the estimates say so, with what the add + norm kernel takes.
// Prompts of 4096, 3400 and 3000 positions of width 896 -4.9, -1.8 and -3.4 %, of 2500 -0.3; by hand where the estimate says no, 2048 +7.4, 1501 of width 1536 +2.1.
static bool down_adds_residual(const GemmArgs& g, int cus, int max_slices) {
  if (g.M <= MAX_ROWS) return false;
  return pick_gemm<EPI_RESID>(g, cus, 1).us < pick_gemm<EPI_PARTIAL>(g, cus, max_slices).us + 3.0 + 4.2e-6 * g.M * g.N;
}
// Returns the number of k-slices (1 unless `max_slices` allows more: outputs that are k-split partials); EPI_RESID: of the pieces of a
// row's sum of squares.
template <int EPI>
static int launch_gemm(const GemmArgs& g, int cus, int max_slices, hipStream_t st) {
  const GemmPick c = pick_gemm<EPI>(g, cus, max_slices);
  if (c.kernel != KERNEL_KWAVE) return launch_gemm_tile<EPI>(g, c, st);
  const TilePlan& p = c.p;
#define KWAVE(TM, TN, U)                                                                             \
  if (c.rt == TM && c.ct == TN) hipLaunchKernelGGL((k_gemm_kwave<EPI, TM, TN, 8, U>), dim3(8 * p.per_xcd), dim3(512), 0, st, g, p)
  KWAVE(1, 2, 4);
  else KWAVE(2, 2, 4);
  else KWAVE(1, 4, 4);
  else KWAVE(3, 2, 4);
  else KWAVE(2, 4, 2);
  else KWAVE(3, 4, 2);
  else if constexpr (EPI == EPI_SWIGLU) { KWAVE(1, 6, 4); else KWAVE(2, 6, 2); else KWAVE(3, 6, 1); else KWAVE(4, 6, 1); }
  else { KWAVE(4, 4, 2); }
  LAUNCH_CHECK();
  return EPI == EPI_RESID ? p.n_colb * (c.ct / 2) : p.n_slices;
#undef KWAVE
}

// Matrix-core attention: parts so that a launch has about a workgroup per CU and a key group at least one chunk; one part, and no
// merge kernel, where the tiles alone fill half the device or the keys are few.  `plan_chunks`: the chunks of a sequence that the
// parts are cut for.  A prompt's launch gives its own (the host knows them: they follow from the call).  Any other gives
// ATT_PLAN_CHUNKS, so that the cut, and with it the bits of a row, depends on the launch's shape and not on the lengths of
// other sequences or on the host's bound of its own.  64 (4096 positions) was as fast as cutting for the longest sequence of the
// launch on every batch measured (16 x 7 rows at 256 to 4096 positions 2521 us a cycle either way, 64 x 8 at 128 to 1024 3536,
// 8 x 9 of the 1.5B shape 3850); 48, 32 and 16 were up to 2, 5 and 8 % slower.
constexpr int ATT_PLAN_CHUNKS = 64;
template <int HD, int WQ, int WK, bool LAZY>
static int launch_attn_mfma_parts(const AttnArgs& a, int n_tg, int nkv, int B, hipStream_t st) {
  constexpr int LDS = WK * 2 * 2 * HD * 128;              // two buffers of 64 keys and 64 values per key group
  static LdsOptIn lds;
  if (hipError_t e = lds.ask((const void*)k_attn_mfma<HD, WQ, WK, LAZY>, LDS); e != hipSuccess)
    return fail(SSD_EHIP, "hipFuncSetAttribute: %s", hipGetErrorString(e));
  hipLaunchKernelGGL((k_attn_mfma<HD, WQ, WK, LAZY>), dim3(a.nparts * n_tg, nkv, B), dim3(WQ * WK * 64), LDS, st, a);
  LAUNCH_CHECK();
  return SSD_OK;
}
struct AttnPick { int wq, wk, n_tg, part_chunks; bool lazy; };        // row tiles x key groups of a workgroup, groups of tiles, chunks of a part; the loop whose reference rarely moves
static AttnPick pick_attn_mfma(int hd, int rows, int group, int plan_chunks, bool prompt, int nkv, int B, int cus) {
  const int tiles = cdiv(rows * group, 16);
  // Two tiles x four key groups (head size 64) where workgroups of four tiles would be for a quarter to half of the device: a chain
  // of half as many chunks, on twice the compute units where there are tiles for them (64 sequences x 8 rows at 128 to 1024 positions
  // 15.7 -> 13.6 us a launch; a prompt of 293 to 585 rows of the 0.5B shape, with the merge and between events, 12.4 -> 10.2 at 300 rows,
  // 14.5 -> 10.7 at 512, 15.8 -> 11.9 at 576).  With fewer workgroups than that the parts fill the device, and four tiles x two groups take
  // 11.7 us for 16 sequences x 7 rows where two x four take 13.0.
  // Four x four for prompts whose parts have more than 16 chunks, all of which gain (attention.h).  From 11 chunks on some do: a
  // prompt's first launch of the 0.5B shape, us between events with 4 x 2 and with 4 x 4: 592 rows (10 chunks) 13.6 and 14.1, 700 (11)
  // 14.9 and 14.6, 832 (13) 16.6 and 15.9, 1024 (16) 18.3 and 17.1.
  const int four = B * nkv * cdiv(tiles, 4);
  const bool narrow = hd == 64 && four <= cus / 2 && four >= cus / 4;
  AttnPick c{narrow ? 2 : 4, narrow ? 4 : 2, 0, 0, false};
  c.n_tg = cdiv(tiles, c.wq);
  const int want = std::min(std::max(1, cus / (c.n_tg * nkv * B)), cdiv(plan_chunks, c.wk));
  c.part_chunks = cdiv(cdiv(plan_chunks, want), c.wk) * c.wk;
  // With more workgroups than compute units 4 x 2 instead, two on a compute unit, whose ends and beginnings overlap, and from three times as many 8 x 2, which reads
  // the keys half as often (one launch for the whole prompt, 1100 / 1501 / 2500 / 4096 rows: 4 x 4 19.0 / 25.3 / 45.6 / 89, 4 x 2 18.8 / 24.7 / 44.8 / 78, 8 x 2
  // 24.9 / 30.2 / 44.6 / 73 to 78).  Head size 128 has the room for 4 x 2 alone (1100 and 1501 rows of the 1.5B shape 29.1 -> 27.2 and 36.2 -> 33.1).
  if (!narrow && prompt && c.part_chunks > 16) {
    c.lazy = true;
    if (hd == 64 && four <= cus) c.wk = 4;
    if (hd == 64 && four > 3 * cus) { c.wq = 8; c.n_tg = cdiv(tiles, c.wq); }
    c.part_chunks = cdiv(c.part_chunks, c.wk) * c.wk;      // (a part is whole rounds of the key groups: they would walk into the next one)
  }
  return c;
}
template <int HD>
static int launch_attn_mfma(AttnArgs a, int nchunks, int plan_chunks, bool prompt, int nkv, int B, int M, int cus, hipStream_t st) {
  const AttnPick c = pick_attn_mfma(HD, a.rows.R, a.nq / nkv, plan_chunks, prompt, nkv, B, cus);
  a.part_keys = c.part_chunks * 64;
  a.nparts = cdiv(nchunks, c.part_chunks);
  a.n_tg = c.n_tg;
  int rc;
  if constexpr (HD == 64)
    rc = c.wq == 2 ? launch_attn_mfma_parts<HD, 2, 4, false>(a, c.n_tg, nkv, B, st)
         : c.wq == 8 ? launch_attn_mfma_parts<HD, 8, 2, true>(a, c.n_tg, nkv, B, st)
         : c.wk == 4 ? launch_attn_mfma_parts<HD, 4, 4, true>(a, c.n_tg, nkv, B, st)
         : c.lazy ? launch_attn_mfma_parts<HD, 4, 2, true>(a, c.n_tg, nkv, B, st) : launch_attn_mfma_parts<HD, 4, 2, false>(a, c.n_tg, nkv, B, st);
  else rc = c.lazy ? launch_attn_mfma_parts<HD, 4, 2, true>(a, c.n_tg, nkv, B, st) : launch_attn_mfma_parts<HD, 4, 2, false>(a, c.n_tg, nkv, B, st);
  if (rc) return rc;
  if (a.nparts > 1) {
    hipLaunchKernelGGL((k_attn_combine_parts<HD>), dim3(cdiv(M * a.nq, BLOCK / (HD / 4))), dim3(BLOCK), 0, st, a);
    LAUNCH_CHECK();
  }
  return SSD_OK;
}

template <typename DT, int HD>
static int launch_attn(AttnArgs a, int nchunks, int plan_chunks, bool prompt, int nkv, int B, int M, bool mfma, int cus, hipStream_t st) {
  if constexpr (std::is_same<DT, BF16>::value && (HD == 64 || HD == 128)) {
    if (mfma && a.kv.bt == 16) return launch_attn_mfma<HD>(a, nchunks, plan_chunks, prompt, nkv, B, M, cus, st);
  }
  if constexpr (std::is_same<DT, F32>::value) {
    const int tiles = cdiv(a.rows.R * (a.nq / nkv), 16);
    if (a.kv.bt == 16) {                                   // (a tile of keys is a block)
      a.nchunks = nchunks;
      a.nparts = cdiv(nchunks, att_f32_part<HD>());
      a.part_keys = att_f32_part<HD>() * ATT_CHUNK;
      hipLaunchKernelGGL((k_attn_f32<HD>), dim3(a.nparts * tiles, nkv, B), dim3(att_f32_waves<HD>() * WAVE), 0, st, a);
      LAUNCH_CHECK();
      if (a.nparts > 1) {
        hipLaunchKernelGGL((k_attn_combine<HD, F32>), dim3(M * a.nq), dim3(WAVE), 0, st, a);
        LAUNCH_CHECK();
      }
      return SSD_OK;
    }
  }
  a.part_keys = ATT_CHUNK;
  hipLaunchKernelGGL((k_attn_chunk<HD, DT>), dim3(nchunks, nkv, B), dim3(BLOCK), 0, st, a);
  LAUNCH_CHECK();
  hipLaunchKernelGGL((k_attn_combine<HD, F32>), dim3(M * a.nq), dim3(WAVE), 0, st, a);
  LAUNCH_CHECK();
  return SSD_OK;
}

// The same forward as one persistent kernel (see persistent.h).  Returns -1 when it is not admitted beside what other streams run.
static int forward_persistent(const ssd_model* m, ssd_kv* kv, Rows rows, int B, int pcap, const int32_t* dev_tokens,
                              int tok_stride, bool with_head, hipStream_t st) {
  const ssd_model_config& c = m->c;
  PArgs a;
  memset(&a, 0, sizeof a);
  a.n_layers = c.n_layers; a.d = c.d_model; a.nq = c.n_q_heads; a.nkv = c.n_kv_heads; a.ffn = c.d_ffn; a.vocab = c.vocab;
  a.n_embed = c.n_embed; a.eps = c.rms_eps; a.scale = 1.0f / sqrtf((float)c.head_dim);
  a.embed = (const bf16_t*)m->embed; a.final_norm = m->final_norm; a.head = m->head; a.rope = m->rope;
  a.layer0 = m->host_layers[0];
  a.layer_stride = m->layer_stride;
  a.kv = kv->v; a.rows = rows; a.pcap = pcap; a.n_seqs = B; a.tok_stride = tok_stride; a.with_head = with_head ? 1 : 0;
  a.tokens = dev_tokens;
  const size_t PR = kv->p_rows;
  a.h = kv->p_h; a.hg = kv->p_hg; a.sumsq = kv->p_sumsq; a.q = kv->p_q; a.attn = kv->p_attn; a.act = kv->p_act;
  a.part = kv->p_part; a.att_o = kv->p_att_o; a.att_ml = kv->p_att_ml; a.logits = kv->logits; a.NP = kv->NP;
  a.st_h = PR * c.d_model; a.st_hg = 2 * PR * c.d_model; a.st_sq = PR * (c.d_model / 32);
  a.st_q = 2 * PR * c.n_q_heads * c.head_dim; a.st_act = 2 * PR * c.d_ffn;
  a.st_part = (size_t)P_MAX_SPLITS * PR * c.d_model; a.part_stride = PR * c.d_model;
  a.st_att_o = PR * c.n_q_heads * kv->NP * 64; a.st_att_ml = PR * c.n_q_heads * kv->NP * 2;
  int max_len = 0;
  for (int s = rows.seq0; s < rows.seq0 + B; ++s) max_len = std::max(max_len, kv->len_ub[s]);
  a.n_parts = std::min(kv->NP, cdiv(max_len + rows.R, ATT_PART));
  a.tickets = kv->tickets; a.bar = kv->bar; a.epoch_base = kv->bar_epoch;
  a.trace = (kv->trace_on && 2 * (1 + 5 * c.n_layers) <= 512) ? kv->trace : nullptr;
  const int G = kv->persistent_wgs, NU = 2 * G, npairs = c.d_model / 32;
  auto splits = [&](int K) { return std::max(1, std::min(std::min(NU / npairs, (K / 32) / 4), P_MAX_SPLITS)); };
  a.gs_o = (c.n_q_heads * c.head_dim) / 32 <= 4 * PF_K ? 1 : splits(c.n_q_heads * c.head_dim);   // <= PF_K k-tiles per wave: all prefetched
  a.gs_d = splits(c.d_ffn);
  const ResidentLaunch order(kv, st, G);
  if (!order.admitted) return -1;
  kv->bar_epoch += (with_head ? 1u : 0u) + 5u * (uint32_t)c.n_layers;  // barriers this launch executes
  ProfScope ps(PROF_PERSISTENT, st);
  hipLaunchKernelGGL(k_forward_persistent, dim3(G), dim3(PBLOCK), 0, st, a);
  LAUNCH_CHECK();
  return SSD_OK;
}

// The same forward without grid barriers between phases (see dataflow.h).  Returns -1 when the launch does not
// fit that kernel's limits or is not admitted beside what other streams run, so that the caller takes another one instead.
static int forward_dataflow(const ssd_model* m, ssd_kv* kv, Rows rows, int B, int pcap, const int32_t* dev_tokens,
                            int tok_stride, bool with_head, hipStream_t st) {
  const ssd_model_config& c = m->c;
  const int npairs = c.d_model / 32, M = rows.M;
  const int nqd = c.n_q_heads * c.head_dim, grp = c.n_q_heads / c.n_kv_heads;
  int max_len = 0;
  for (int s = rows.seq0; s < rows.seq0 + B; ++s) max_len = std::max(max_len, kv->len_ub[s]);
  // Workgroups for the attention's parts: as many as the host's bound of the lengths allows for (the cut of a row's keys follows
  // from its position, see dataflow.h).
  const int n_parts = df_parts(max_len + rows.R);
  // Workgroups [0, g_mlp) take the MLP items (two 16-column items each); the phases with few items (QKV, attention,
  // output projection) get workgroups of their own after them, as far as the device has compute units.
  const bool wide = kv->wide;
  const int g_mlp = wide ? cdiv(c.d_ffn / 32, kv->mlp_tiles) : std::min(kv->persistent_wgs, cdiv(c.d_ffn / 16, 2));
  const int n_att = B * c.n_kv_heads * cdiv(rows.R * grp, 16) * n_parts * (wide ? DfWide::NH : DfNarrow::NH), n_qkv = m->n_qkv() / 32, n_other = n_qkv + npairs;
  // with compute units to spare every item of the other small phases gets a workgroup of its own, as attention's always do (its
  // waves then do not share their SIMDs with a second item), else two items share one
  const int small_stride = g_mlp + n_att + n_other <= kv->cus ? 2 : 1;
  const int o_stride = wide && g_mlp + n_att + cdiv(n_qkv, 2) + npairs <= kv->cus ? 2 : small_stride;
  // (No more workgroups than items: those of a launch wait for each other, and a smaller model's launch on another stream may be in what is left.)
  const int G = std::min(kv->cus, g_mlp + n_att + (wide ? cdiv(small_stride * n_qkv, 2) + cdiv(o_stride * npairs, 2) : cdiv(small_stride * n_other, 2)));
  // Wide, more than 12 rows of several sequences: the launches per operator where items of the small phases share workgroups with the MLP's, which with two k-tiles each
  // have no room for the second one's weights while they wait, and the prefixes are not long enough to make up for it (beyond 3072 positions the launches per
  // operator have that many more parts to merge).  With more than six tiles of attention, also of one sequence, they run whatever the prefix.  28 layers of width 1536, us in one launch and per
  // operator: 2 sequences of 8 rows behind 1200 / 2060 / 2600 / 3100 / 4096 positions 1235 / 1510 / 1534 / 1546 / 1603 and 1409 / 1460 / 1485 / 1520 / 1583; 3 of 5
  // 1234 / 1505 / 1521 / 1507 / 1536 and 1390 / 1441 / 1470 / 1529 / 1615; 5 of 3 behind 4096 1665 and 1538.  (12 rows: 2 of 6 1173 / 1420 / 1448 / 1440 / 1447 and
  // 1390 / 1437 / 1464 / 1497 / 1553, 4 of 3 1478 and 1710 behind 4096.)
  const bool shared = g_mlp + n_att + cdiv(n_other, 2) > kv->cus;
  const bool wide_batch = B * cdiv(rows.R * grp, 16) <= 6 && !(B > 1 && shared && kv->mlp_tiles == 2 && n_parts <= 3);
  // limits: one round of attention (its workgroups wait for each other's parts), query rows of an item, LDS staging capacity
  const bool fits = M <= 16 && rows.R * grp <= DF_ATT_ROWS && n_att <= G && n_parts <= kv->t_NP &&
                    M * (std::max(c.d_model, nqd) + 4) <= (wide ? DfWide::AW : DfNarrow::AW) && M * (c.d_model / 32) <= DF_SQ_WORDS &&
                    c.n_layers <= 128 && 2 + 10 * c.n_layers + 2 <= 512 &&
                    (!wide || M <= 12 || wide_batch);
  if (!fits) return -1;
  DArgs a;
  memset(&a, 0, sizeof a);
  a.n_layers = c.n_layers; a.d = c.d_model; a.nq = c.n_q_heads; a.nkv = c.n_kv_heads; a.ffn = c.d_ffn; a.vocab = c.vocab;
  a.n_embed = c.n_embed; a.eps = c.rms_eps; a.scale = 1.0f / sqrtf((float)c.head_dim);
  a.embed = (const bf16_t*)m->embed; a.final_norm = m->final_norm; a.head = m->head; a.rope = m->rope;
  a.layer0 = m->host_layers[0];
  a.layer_stride = m->layer_stride;
  a.kv = kv->v; a.rows = rows; a.pcap = pcap; a.n_seqs = B; a.tok_stride = tok_stride; a.with_head = with_head ? 1 : 0;
  a.tokens = dev_tokens;
  const size_t PR = kv->t_rows;
  a.tw = (uint32_t*)kv->t_base; a.st_set = kv->t_attp_at; a.state = kv->t_rowblk + 16; a.h = kv->t_h; a.hg = kv->t_hg; a.sq = kv->t_sq; a.q = kv->t_q; a.kvn = kv->t_kvn; a.attn = kv->t_attn;
  a.att_p = kv->t_att_p; a.logits = kv->logits;
  a.st_h = PR * c.d_model; a.st_sq = PR * (c.d_model / 8); a.st_q = PR * nqd; a.st_kvn = PR * 2 * c.n_kv_heads * c.head_dim;
  a.st_att_p = PR * c.n_q_heads * kv->t_NP * (c.head_dim / 64 * 96);
  a.rowblk = kv->t_rowblk;
  a.part = (float*)kv->t_part; a.st_part = (size_t)2 * (c.d_ffn / 32) * PR * c.d_model;
  a.NP = kv->t_NP; a.n_parts = n_parts; a.g_mlp = g_mlp; a.small_stride = small_stride;
  a.o_stride = o_stride; a.mlp_tiles = kv->mlp_tiles; a.n_sum = g_mlp;
  a.recip_d = cdiv(65536, cdiv(c.d_model, 512)); a.recip_q = cdiv(65536, cdiv(nqd, 512));
  a.bar = kv->bar;
  a.trace = kv->trace_on ? kv->trace : nullptr;
  kv->last_wgs = kv->capturing ? std::max(kv->last_wgs, G) : G;
  const ResidentLaunch order(kv, st, G);
  if (!order.admitted) return -1;
  ProfScope ps(PROF_PERSISTENT, st);
  kv->last_whole = kv->attn_whole && max_len + 16 <= DF_ONE_PART;      // (reported only)
  // The smallest instantiation whose flight of an operand staging holds the rows, where its sum tasks (of 8, 32, 32, 64, 64 columns) go well: those of
  // two rows in one round (a second one takes 2 us, tasks of 32 columns 1.1; with 224 tasks on 226 workgroups, beyond 1536 positions at width 896, they are
  // 1.5 us a layer slower than those of 32 columns all the same), those of 10 on the workgroups with MLP items; 2 also needs room for its sums of squares.
  int sb = M <= 2 && M * (c.d_model / 8) <= std::min(PBLOCK, G) ? 2 : M <= 4 ? 4 : M <= 6 && M * npairs <= g_mlp ? 10 : M <= 8 ? 16 : 18;
  if (kv->df_sb && M <= DF_PACK_ROWS) sb = kv->df_sb;
  if (sb == 2 && M * (c.d_model / 8) > DF_SQ_WORDS) sb = 10;
  if (wide) {
    // Sums of 32 columns for one or two rows, of 64 for more, which then go to workgroups with MLP items (28 layers of width 1536: one row 676 us with 8
    // columns, 639 with 32, 651 with 64; two 668 and 671, three 706 with 32 and 698 with 64, four 743 and 721).
    sb = kv->df_sb && M <= DF_PACK_ROWS ? (kv->df_sb <= 4 ? 4 : kv->df_sb == 18 ? 18 : 16) : M <= 2 ? 4 : M <= 8 ? 16 : 18;
#define DF_LAUNCH(S) hipLaunchKernelGGL((k_forward_wide<S>), dim3(G), dim3(PBLOCK), 0, st, a)
    if (sb == 4) DF_LAUNCH(4); else if (sb == 16) DF_LAUNCH(16); else DF_LAUNCH(18);
#undef DF_LAUNCH
    LAUNCH_CHECK();
    return SSD_OK;
  }
#define DF_LAUNCH(S) hipLaunchKernelGGL((k_forward_dataflow<S>), dim3(G), dim3(PBLOCK), 0, st, a)
  if (sb == 2) DF_LAUNCH(2); else if (sb == 4) DF_LAUNCH(4); else if (sb == 10) DF_LAUNCH(10); else if (sb == 16) DF_LAUNCH(16); else DF_LAUNCH(18);
#undef DF_LAUNCH
  LAUNCH_CHECK();
  return SSD_OK;
}

// The fp32 forward of a few rows as one launch (see small.h): up to 16 rows a sequence and 64 in all, of up to 16 sequences that attend in one part, with a compute
// unit for every item.  Returns -1 where that is not so, or where it is not admitted beside what other streams run; the launches per operator give the same bits.
static int forward_small(const ssd_model* m, ssd_kv* kv, Rows rows, int B, int pcap, const int32_t* dev_tokens, int tok_stride, bool with_head,
                         hipStream_t st) {
  const ssd_model_config& c = m->c;
  const int M = rows.M, T = cdiv(M, 16), grp = c.n_q_heads / c.n_kv_heads;
  int max_len = 0;
  for (int s = rows.seq0; s < rows.seq0 + B; ++s) max_len = std::max(max_len, kv->len_ub[s]);
  SArgs a;
  memset(&a, 0, sizeof a);
  a.first_gu = B * c.n_kv_heads * cdiv(rows.R * grp, 16);
  a.first_down = a.first_gu + c.d_ffn / 32 * T;
  a.first_end = a.first_down + c.d_model / 32 * T;
  const int G = a.first_end + 1;
  a.tiles = cdiv(rows.R * grp, 16);
  a.recip_tiles = cdiv(65536, a.tiles); a.recip_seqs = cdiv(65536, B); a.recip_T = cdiv(65536, T); a.recip_R = cdiv(65536, rows.R); a.recip_G = cdiv(65536, grp);
  if (M > kv->t_rows || rows.R > 16 || B > 16 || max_len + rows.R > att_f32_part<SF_HD>() * ATT_CHUNK || G > kv->cus) return -1;
  a.n_layers = c.n_layers; a.d = c.d_model; a.nq = c.n_q_heads; a.nkv = c.n_kv_heads; a.ffn = c.d_ffn; a.vocab = c.vocab; a.n_embed = c.n_embed;
  a.eps = c.rms_eps; a.scale = 1.0f / sqrtf((float)c.head_dim);
  a.embed = (const float*)m->embed; a.final_norm = m->final_norm; a.head = (const float*)m->head; a.rope = m->rope;
  a.layer0 = m->host_layers[0]; a.layer_stride = m->layer_stride;
  a.kv = kv->v; a.rows = rows; a.pcap = pcap; a.n_seqs = B; a.tok_stride = tok_stride; a.with_head = with_head ? 1 : 0; a.tokens = dev_tokens;
  a.tw = (uint32_t*)kv->t_base; a.st_set = kv->t_attp_at; a.cap = kv->t_rows; a.rowblk = kv->t_rowblk; a.state = kv->t_rowblk + SF_MAX_ROWS;
  a.logits = kv->logits; a.bar = kv->bar;
  const ResidentLaunch order(kv, st, G);
  if (!order.admitted) return -1;
  ProfScope ps(PROF_PERSISTENT, st);
  hipLaunchKernelGGL(k_forward_f32, dim3(G), dim3(PBLOCK), 0, st, a);
  LAUNCH_CHECK();
  return SSD_OK;
}

// One decoder forward for sequences [seq0, seq0+B), R rows each.  pcap = pending slots at the head of each
// sequence's rows (0: all rows take explicit tokens).  Leaves logits [B*R][vocab] in the workspace when
// with_head.  The caller has checked room.
template <typename DT>
static int forward(const ssd_model* m, ssd_kv* kv, int seq0, int B, int R, int pcap, const int32_t* dev_tokens,
                   int tok_stride, bool with_head, hipStream_t st) {
  const ssd_model_config& c = m->c;
  const int M = B * R, d = c.d_model, hd = c.head_dim, nq = c.n_q_heads, nkv = c.n_kv_heads;
  const int nqd = nq * hd, nqkv = m->n_qkv();
  Rows rows = kv->rows;
  rows.M = M; rows.R = R; rows.seq0 = seq0;
  {                                     // every forward is followed by a kernel that advances the cache's launch number
    const int rc = kv_launch_guard(kv, st, 1);
    if (rc) return rc;
    ++kv->launch_no;
    kv->publish = 0;
  }
  if (kv->capturing && !(kv->persistent_wgs > 0 && M <= kv->p_rows && kv->dataflow))
    return fail(SSD_ENOSUP, "this launch does not fit the barrier-free forward kernel: it cannot be captured");
  if (kv->persistent_wgs > 0 && M <= kv->p_rows) {
    if (kv->dataflow) {
      const int rc = forward_dataflow(m, kv, rows, B, pcap, dev_tokens, tok_stride, with_head, st);
      if (rc >= 0) { kv->last_path = kv->last_whole ? 4 : 3; return rc; }
    }
    if (kv->capturing) return fail(SSD_ENOSUP, "this launch does not fit the barrier-free forward kernel: it cannot be captured");
    const int rc = forward_persistent(m, kv, rows, B, pcap, dev_tokens, tok_stride, with_head, st);
    if (rc != -1) { kv->last_path = 2; return rc; }
  }
  if (kv->wide && M <= kv->t_rows) {
    const int rc = forward_dataflow(m, kv, rows, B, pcap, dev_tokens, tok_stride, with_head, st);
    if (rc >= 0) { kv->last_path = kv->last_whole ? 4 : 3; return rc; }
  }
  kv->last_path = 1;
  if (kv->small) {
    const int rc = forward_small(m, kv, rows, B, pcap, dev_tokens, tok_stride, with_head, st);
    if (rc >= 0) { kv->last_path = 5; return rc; }
  }

  EmbedArgs e;
  e.kv = kv->v; e.rows = rows; e.pcap = pcap; e.n_seqs = B; e.tokens = dev_tokens; e.tok_stride = tok_stride;
  constexpr bool bf16 = std::is_same<DT, BF16>::value;     // bf16: GEMM operands are kept as split rows (common.h)
  const dim3 row_block(std::min(1024, cdiv(d / 4, WAVE) * WAVE));          // a thread per four columns of a row
  e.embed = m->embed; e.n_embed = c.n_embed; e.d = d; e.h = kv->h;
  e.gain = m->layers[0].ln1; e.eps = c.rms_eps; e.xn = bf16 ? (bf16_t*)kv->xn : nullptr;
  hipLaunchKernelGGL((k_embed<DT>), dim3(M + 1), row_block, 0, st, e);
  LAUNCH_CHECK();

  int max_len = 0;
  for (int s = seq0; s < seq0 + B; ++s) max_len = std::max(max_len, kv->len_ub[s]);
  const int nchunks = cdiv(max_len + R, ATT_CHUNK), plan_chunks = pcap ? ATT_PLAN_CHUNKS : nchunks;

  GemmArgs g0;
  memset(&g0, 0, sizeof g0);
  g0.M = M; g0.kv = kv->v; g0.rows = rows; g0.nq = nq; g0.rope = m->rope; g0.rms_eps = c.rms_eps;
  const void* const normed = bf16 ? (const void*)kv->xn : kv->h;           // fp32: the GEMM normalises its operand itself
  const size_t part_stride = (size_t)M * d;
  const int pairs_d = cdiv(d, 32);
  const int max_slices = partial_slices(kv->max_seqs * kv->max_rows, M);
  // The output projection is not k-split: its epilogue adds the residual and prepares the norm before gate / up, and no add + norm
  // kernel runs between them (1024 rows: 10.8 us of width 896 and 21.4 of 1536, where two k-slices and the add + norm kernel took 9.8 + 7.6
  // and 16.2 + 12).
  auto add_norm = [&](int n_part_, const float* gain) -> int {
    if (!bf16) return SSD_OK;
    const auto kernel = n_part_ <= 4 ? k_add_norm<4> : k_add_norm<8>;       // (launch_gemm cuts k into 8 slices at most)
    hipLaunchKernelGGL(kernel, dim3(M), row_block, 0, st, kv->h, kv->part, n_part_, part_stride, gain, c.rms_eps, (bf16_t*)kv->xn, d);
    LAUNCH_CHECK();
    return SSD_OK;
  };
  int n_part = 0, pieces = 0, down_pieces = 0;             // (down_pieces: of the sums of squares that the down projection left, 0 where it left partials)
  int rc;
  for (int l = 0; l < c.n_layers; ++l) {
    const LayerW& L = m->layers[l];
    if (l > 0 && !down_pieces && (rc = add_norm(n_part, L.ln1))) return rc;      // (the first layer's: in k_embed)
    GemmArgs g = g0;                                       // QKV + bias + rotary + cache write
    g.A = normed; g.W0 = L.wqkv; g.W1 = L.wqkv; g.N = nqkv; g.K = d;
    g.bias = L.bqkv; g.q = kv->q; g.layer = l;
    if (down_pieces) { g.sumsq = kv->part; g.rms_d = d; g.sum_pieces = down_pieces; }
    {
      ProfScope ps(PROF_QKV, st);
      if constexpr (bf16) rc = std::min(0, launch_gemm<EPI_QKV>(g, kv->cus, 1, st));
      else { g.gain = L.ln1; rc = launch_gemm_f32<EPI_QKV>(g, (nq + 2 * nkv) * (hd / 32), st); }
    }
    if (rc) return rc;
    if (!with_head && l + 1 == c.n_layers) return SSD_OK;  // a prompt is its keys and values: nothing reads what comes behind the last layer's

    AttnArgs a;
    a.q = kv->q; a.kv = kv->v; a.rows = rows; a.layer = l; a.nq = nq; a.scale = 1.0f / sqrtf((float)hd);
    a.o_part = kv->o_part; a.ml_part = kv->ml_part; a.NC = kv->NC; a.out = kv->attn;
    a.split_kt = bf16 ? nqd / 32 : 0;
    {
      ProfScope ps(PROF_ATTN, st);
      if (hd == 32) rc = launch_attn<DT, 32>(a, nchunks, plan_chunks, pcap == 0, nkv, B, M, kv->attn_mfma, kv->cus, st);
      else if (hd == 64) rc = launch_attn<DT, 64>(a, nchunks, plan_chunks, pcap == 0, nkv, B, M, kv->attn_mfma, kv->cus, st);
      else rc = launch_attn<DT, 128>(a, nchunks, plan_chunks, pcap == 0, nkv, B, M, kv->attn_mfma, kv->cus, st);
    }
    if (rc) return rc;

    g = g0;                                                // output projection
    g.A = kv->attn; g.W0 = L.wo; g.W1 = L.wo; g.N = d; g.K = nqd;
    g.out = kv->part; g.out_split_stride = part_stride; g.ldo = d;
    {
      ProfScope ps(PROF_O, st);
      g.h = kv->h;
      if constexpr (!bf16) {
        rc = launch_gemm_f32<EPI_RESID>(g, pairs_d, st);
      } else {
        g.gain = L.ln2; g.hg = kv->xn; g.sumsq = kv->part; g.sum_pieces = M > 64 ? 1 : 0;        // (gate / up by k_gemm_kwave reads 16-column sums)
        rc = launch_gemm<EPI_RESID>(g, kv->cus, 1, st);
        if (rc > 0) { if (M > 64) pieces = rc; rc = SSD_OK; }
      }
    }
    if (rc) return rc;

    g = g0;                                                // gate / up + SwiGLU
    g.A = normed; g.W0 = L.wgate; g.W1 = L.wup; g.N = c.d_ffn; g.K = d; g.act = kv->act;
    g.act_split_kt = bf16 ? c.d_ffn / 32 : 0;
    g.sumsq = kv->part; g.rms_d = bf16 ? d : 0; g.sum_pieces = pieces;
    {
      ProfScope ps(PROF_GATEUP, st);
      if constexpr (bf16) rc = std::min(0, launch_gemm<EPI_SWIGLU>(g, kv->cus, 1, st));
      else { g.gain = L.ln2; rc = launch_gemm_f32<EPI_SWIGLU>(g, cdiv(c.d_ffn, 16), st); }
    }
    if (rc) return rc;

    g = g0;                                                // down projection
    g.A = kv->act; g.W0 = L.wdown; g.W1 = L.wdown; g.N = d; g.K = c.d_ffn;
    g.out = kv->part; g.out_split_stride = part_stride; g.ldo = d;
    {
      ProfScope ps(PROF_DOWN, st);
      if constexpr (bf16) {
        down_pieces = 0;
        if (!with_head && down_adds_residual(g, kv->cus, max_slices)) {
          g.gain = m->layers[l + 1].ln1; g.hg = kv->xn; g.h = kv->h; g.sumsq = kv->part; g.sum_pieces = 1;
          rc = down_pieces = launch_gemm<EPI_RESID>(g, kv->cus, 1, st);
        } else {
          rc = n_part = launch_gemm<EPI_PARTIAL>(g, kv->cus, max_slices, st);
        }
        rc = std::min(0, rc);
      }
      else { g.h = kv->h; rc = launch_gemm_f32<EPI_RESID>(g, pairs_d, st); }
    }
    if (rc) return rc;
  }
  if ((rc = add_norm(n_part, m->final_norm))) return rc;
  GemmArgs g = g0;
  g.A = normed; g.W0 = m->head; g.W1 = m->head; g.N = c.vocab; g.K = d;
  g.out = kv->logits; g.out_split_stride = 0; g.ldo = c.vocab;
  ProfScope ps(PROF_HEAD, st);
  if constexpr (bf16) return std::min(0, launch_gemm<EPI_PARTIAL>(g, kv->cus, 1, st));
  else { g.gain = m->final_norm; return launch_gemm_f32<EPI_PARTIAL>(g, cdiv(c.vocab, 32), st); }
}

static int forward_any(const ssd_model* m, ssd_kv* kv, int seq0, int B, int R, int pcap, const int32_t* dev_tokens,
                       int tok_stride, bool with_head, hipStream_t st) {
  return m->c.dtype == SSD_DTYPE_BF16 ? forward<BF16>(m, kv, seq0, B, R, pcap, dev_tokens, tok_stride, with_head, st)
                                      : forward<F32>(m, kv, seq0, B, R, pcap, dev_tokens, tok_stride, with_head, st);
}

static int check_pair(const ssd_model* m, const ssd_kv* kv) {
  if (!m || !kv) return fail(SSD_EINVAL, "null handle");
  if (kv->m != m) return fail(SSD_EINVAL, "the cache was created for another model");
  return SSD_OK;
}

static int check_sample(const ssd_sample_config* s) {
  if (!s) return fail(SSD_EINVAL, "null sample config");
  if (!(s->beta >= 0.0f)) return fail(SSD_EINVAL, "beta must be >= 0");
  if (!s->greedy && !(s->temperature > 0.0f)) return fail(SSD_EINVAL, "temperature must be > 0");
  if (s->top_k < 0) return fail(SSD_EINVAL, "top_k must be >= 0");
  return SSD_OK;
}

// ------------------------------------------------------------------------------------------------ prefill
// Rows of a prompt's launches: as many as the buffers have room for, max_seqs * max_rows; where that is 1024 for one sequence up to prompt_rows, if a launch of more than 1024
// rows attends in one part whatever its rows (its tiles alone are for more than half of the device: pick_attn_mfma), since the buffers of attention's partials have
// room for 1024.  Every launch of a layer costs 5 to 10 us beside its loop, and one
// of 1024 rows fills the device once, mostly not evenly: 4096 positions of the 0.5B shape took 10.62 ms in four launches and take 7.88 in one (8.85 with the
// tiles of 1024 rows), 1501 of the 1.5B shape 9.55 ms and 8.41.  8 layers of the 0.5B shape, 300 and 1000 positions into a cache of 16 sequences of 64 rows: 1509 and 4997 us in
// launches of 64 rows, 382 and 699 as one.
static int prompt_chunk(const ssd_kv* kv) {
  const ssd_model_config& c = kv->m->c;
  const int tiles = cdiv(MAX_ROWS * (c.n_q_heads / c.n_kv_heads), 16);
  const bool one_part = kv->attn_mfma && kv->v.bt == 16 && cdiv(tiles, 4) * c.n_kv_heads > kv->cus / 2;
  return one_part ? kv->prompt_rows : kv->max_seqs * kv->max_rows;
}

extern "C" int ssd_prefill(ssd_model* m, ssd_kv* kv, int seq, const int32_t* dev_tokens, int n, void* stream) {
  int rc = check_pair(m, kv);
  if (rc) return rc;
  if (!dev_tokens || n < 1) return fail(SSD_EINVAL, "prefill needs at least one token");
  if (seq < 0 || seq >= kv->max_seqs) return fail(SSD_EINVAL, "sequence %d out of range", seq);
  if ((rc = kv_check_flags(kv))) return rc;
  hipStream_t st = (hipStream_t)stream;
  hipLaunchKernelGGL(k_kv_set, dim3(1), dim3(BLOCK), 0, st, kv->v, seq, 0, 0, 0, 0, (const int32_t*)nullptr, 0u);
  LAUNCH_CHECK();
  kv->len_ub[seq] = 0;
  kv->npend_ub[seq] = 0;
  if ((rc = kv_check_room(kv, seq, 1, n - 1, st))) return rc;
  const int chunk = prompt_chunk(kv);
  for (int i = 0; i < n - 1; i += chunk) {
    const int R = std::min(chunk, n - 1 - i);
    if ((rc = forward_any(m, kv, seq, 1, R, 0, dev_tokens + i, 0, false, st))) return rc;
    hipLaunchKernelGGL(k_kv_set, dim3(1), dim3(BLOCK), 0, st, kv->v, seq, -1, R, 0, 0, (const int32_t*)nullptr, 2 * kv->publish + 1);
    LAUNCH_CHECK();
    kv->len_ub[seq] += R;
  }
  hipLaunchKernelGGL(k_kv_set, dim3(1), dim3(BLOCK), 0, st, kv->v, seq, -1, 0, 1, 0, dev_tokens + (n - 1), 0u);
  LAUNCH_CHECK();
  kv->npend_ub[seq] = 1;
  return SSD_OK;
}

// ------------------------------------------------------------------------------------------------ step
// Forward + warp + acceptance + commit for sequences 0..B-1.
// `step_dev`: when set, the cycle counter on the device is added to step_ctr (captured cycles); `bump_step`: this
// step's sampling kernel is the last of its cycle and advances that counter.
static int step(ssd_model* m, ssd_kv* kv, int B, int K, const int32_t* dev_x, const float* dev_pd,
                const ssd_sample_config* cfg, uint64_t step_ctr, int slot_base, int32_t* dev_n, int32_t* dev_next,
                int next_stride, float* probs_out, size_t probs_seq_stride, bool probs_last_row_only,
                float* logits_out, hipStream_t st, const int32_t* step_dev = nullptr, bool bump_step = false,
                bool full_pcap = false) {
  const ssd_model_config& c = m->c;
  // Rows per sequence that carry pending tokens: the cache's capacity, or less when the host knows that no sequence of
  // the launch holds that many (a draft cache owes two tokens only right after a fully accepted cycle; at 16 sequences
  // one row each instead of two keeps the draft steps on the persistent kernel).
  int pcap = 1;
  for (int s = 0; s < B; ++s) pcap = std::max(pcap, kv->npend_ub[s]);
  pcap = std::min(pcap, kv->v.pcap);
  if (full_pcap) pcap = kv->v.pcap;     // a captured step must hold whatever the sequences owe at any replay
  const int R = pcap + K, M = B * R, V = c.vocab;
  int rc;
  if (!kv->capturing && (rc = kv_check_room(kv, 0, B, R, st))) return rc;      // (a captured cycle checks before each replay)
  if ((rc = forward_any(m, kv, 0, B, R, pcap, dev_x, K, true, st))) return rc;
  if (logits_out) HIP_TRY(hipMemcpyAsync(logits_out, kv->logits, (size_t)M * V * 4, hipMemcpyDeviceToDevice, st));

  // rows that need a distribution: all K+1 of a verification, or the last row of a draft step
  WarpArgs w;
  w.ld = V; w.V = V; w.temperature = cfg->temperature; w.top_k = cfg->top_k; w.greedy = cfg->greedy;
  AcceptArgs a;
  memset(&a, 0, sizeof a);
  if (probs_last_row_only) {
    w.logits = kv->logits + (size_t)(R - 1) * V;
    w.ld = R * V;                       // one row per sequence
    w.probs = probs_out ? probs_out : kv->probs;
    w.probs_stride = probs_out ? probs_seq_stride : (size_t)V;
    a.pt = w.probs; a.pt_seq_stride = w.probs_stride;
  } else {
    w.logits = kv->logits + (size_t)(pcap - 1) * V;   // row of the last pending token, then the K drafts
    // rows pcap-1 .. R-1 of every sequence are consecutive only when pcap == 1 (a target cache)
    w.probs = probs_out ? probs_out : kv->probs;
    w.probs_stride = V;
    a.pt = w.probs; a.pt_seq_stride = (size_t)(K + 1) * V;
  }
  const bool one_row = probs_last_row_only || (K == 0 && pcap == 1);     // one row per sequence: fused with the sampling
  if (!one_row) {
    SAMPLER(k_warp_softmax, V, M, st, w);
    LAUNCH_CHECK();
  }
  a.pd = dev_pd; a.x = dev_x; a.uniforms = nullptr; a.seed = cfg->seed; a.step = step_ctr;
  a.step_dev = step_dev; a.bump_step = bump_step ? 1 : 0; a.launch = 2 * kv->publish + 1;
  a.B = B; a.K = K; a.V = V; a.beta = cfg->beta;
  a.n_acc = dev_n; a.next_tok = dev_next; a.tok_stride = next_stride; a.flags = nullptr;
  a.kv = kv->v; a.seq0 = 0;
  a.ticket = kv->ticket_alt ? kv->ticket_alt : kv->v.ctl + 2;
  a.slot_base = slot_base;
  if (one_row) SAMPLER(k_warp_accept, V, B, st, w, a);
  else SAMPLER(k_accept, V, B, st, a);
  LAUNCH_CHECK();
  return SSD_OK;
}

extern "C" int ssd_verify(ssd_model* target, ssd_kv* kv, int n_seqs, const int32_t* prefix_len,
                          const int32_t* dev_draft_tokens, const float* dev_draft_probs, int K,
                          const ssd_sample_config* cfg, uint64_t step_ctr, int32_t* dev_n_accepted,
                          int32_t* dev_next_token, float* dev_target_probs_opt, float* dev_logits_opt, void* stream) {
  int rc = check_pair(target, kv);
  if (rc) return rc;
  if ((rc = check_sample(cfg))) return rc;
  if (kv->v.pcap != 1) return fail(SSD_EINVAL, "ssd_verify needs a target cache (pending_cap 1)");
  if (n_seqs < 1 || n_seqs > kv->max_seqs) return fail(SSD_EINVAL, "n_seqs %d out of range", n_seqs);
  if (K < 0 || K > SSD_MAX_K || K + 1 > kv->max_rows) return fail(SSD_EINVAL, "K = %d out of range (max_rows %d)", K, kv->max_rows);
  if (K > 0 && (!dev_draft_tokens || !dev_draft_probs)) return fail(SSD_EINVAL, "draft tokens / probabilities are null");
  if (!dev_n_accepted || !dev_next_token) return fail(SSD_EINVAL, "output pointers are null");
  if ((rc = kv_check_flags(kv))) return rc;
  hipStream_t st = (hipStream_t)stream;
  if (prefix_len) {
    if ((rc = kv_refresh(kv, st))) return rc;
    for (int s = 0; s < n_seqs; ++s)
      if (prefix_len[s] != kv->len_ub[s] || kv->npend_ub[s] != 1)
        return fail(SSD_EINVAL, "sequence %d: prefix_len %d but the cache holds %d positions (%d pending)", s,
                    prefix_len[s], kv->len_ub[s], kv->npend_ub[s]);
  }
  rc = step(target, kv, n_seqs, K, dev_draft_tokens, dev_draft_probs, cfg, step_ctr, 0, dev_n_accepted, dev_next_token,
            1, dev_target_probs_opt, 0, false, dev_logits_opt, st);
  if (rc) return rc;
  for (int s = 0; s < n_seqs; ++s) { kv->len_ub[s] += K + 1; kv->npend_ub[s] = 1; }
  return SSD_OK;
}

// ------------------------------------------------------------------------------------------------ no-allocation variant
// Staging of ssd_verify_noalloc: [0, 256) the commit's arrival counter, then the logits rows, then the probability rows.
// One copy per GPU for the life of the process; every call on a GPU uses that GPU's copy.
constexpr size_t NOALLOC_MAX_ELEMS = SSD_NOALLOC_MAX_ELEMS;
static __device__ __align__(256) unsigned char scratch[256 + 2 * NOALLOC_MAX_ELEMS * sizeof(float)];
constexpr int NOALLOC_MAX_DEVICES = 64;
static unsigned char* g_scratch_dev[NOALLOC_MAX_DEVICES];      // device address of `scratch` on each GPU (0: not asked yet)

// The device address of this GPU's copy of `scratch` (the array's name is only a host-side handle of the symbol).
static int noalloc_scratch(unsigned char** out) {
  int dev = -1;
  HIP_TRY(hipGetDevice(&dev));
  if (dev < 0 || dev >= NOALLOC_MAX_DEVICES) return fail(SSD_ENOSUP, "device ordinal %d not supported", dev);
  if (!g_scratch_dev[dev]) {
    unsigned char* p = nullptr;
    HIP_TRY(hipGetSymbolAddress((void**)&p, HIP_SYMBOL(scratch)));
    if (!p) return fail(SSD_EHIP, "hipGetSymbolAddress returned a null address");
    g_scratch_dev[dev] = p;
  }
  *out = g_scratch_dev[dev];
  return SSD_OK;
}

extern "C" int ssd_verify_noalloc(ssd_model* target, ssd_kv* kv, int n_seqs, const int32_t* dev_draft_tokens,
                                  const float* dev_draft_probs, int K, const ssd_sample_config* cfg, uint64_t step_ctr,
                                  int32_t* dev_n_accepted, int32_t* dev_next_token, void* stream) {
  int rc = check_pair(target, kv);
  if (rc) return rc;
  if ((rc = check_sample(cfg))) return rc;
  if (kv->v.pcap != 1) return fail(SSD_EINVAL, "ssd_verify_noalloc needs a target cache (pending_cap 1)");
  if (n_seqs < 1 || n_seqs > kv->max_seqs) return fail(SSD_EINVAL, "n_seqs %d out of range", n_seqs);
  if (K < 0 || K > SSD_MAX_K || K + 1 > kv->max_rows) return fail(SSD_EINVAL, "K = %d out of range (max_rows %d)", K, kv->max_rows);
  if (K > 0 && (!dev_draft_tokens || !dev_draft_probs)) return fail(SSD_EINVAL, "draft tokens / probabilities are null");
  if (!dev_n_accepted || !dev_next_token) return fail(SSD_EINVAL, "output pointers are null");
  const size_t elems = (size_t)n_seqs * (K + 1) * target->c.vocab;
  if (elems > NOALLOC_MAX_ELEMS)
    return fail(SSD_ENOMEM, "ssd_verify_noalloc: n_seqs * (K+1) * vocab = %zu exceeds the static staging of %zu elements", elems,
                (size_t)NOALLOC_MAX_ELEMS);
  if ((rc = kv_check_flags(kv))) return rc;
  unsigned char* sp = nullptr;
  if ((rc = noalloc_scratch(&sp))) return rc;
  hipStream_t st = (hipStream_t)stream;
  // the arrival counter must start at zero whatever an earlier (possibly failed) call on this GPU left; the logits and
  // probability rows are written in full before they are read
  hipLaunchKernelGGL(k_zero_words, dim3(1), dim3(64), 0, st, (int32_t*)sp, 64);
  LAUNCH_CHECK();
  float* const ws_logits = kv->logits;
  float* const ws_probs = kv->probs;
  kv->logits = (float*)(sp + 256);
  kv->probs = (float*)(sp + 256) + NOALLOC_MAX_ELEMS;
  kv->ticket_alt = (int32_t*)sp;
  rc = step(target, kv, n_seqs, K, dev_draft_tokens, dev_draft_probs, cfg, step_ctr, 0, dev_n_accepted, dev_next_token, 1,
            nullptr, 0, false, nullptr, st);
  kv->logits = ws_logits;
  kv->probs = ws_probs;
  kv->ticket_alt = nullptr;
  if (rc) return rc;
  for (int s = 0; s < n_seqs; ++s) { kv->len_ub[s] += K + 1; kv->npend_ub[s] = 1; }
  return SSD_OK;
}

extern "C" int ssd_draft_step(ssd_model* draft, ssd_kv* kv_d, int n_seqs, const ssd_sample_config* cfg,
                              uint64_t step_ctr, int draft_idx, int32_t* dev_token_out, int token_stride,
                              float* dev_probs_out, size_t probs_stride, void* stream) {
  int rc = check_pair(draft, kv_d);
  if (rc) return rc;
  if ((rc = check_sample(cfg))) return rc;
  if (n_seqs < 1 || n_seqs > kv_d->max_seqs) return fail(SSD_EINVAL, "n_seqs %d out of range", n_seqs);
  if (draft_idx < 0 || draft_idx > SSD_MAX_K) return fail(SSD_EINVAL, "draft_idx out of range");
  if (!dev_token_out || token_stride < 1) return fail(SSD_EINVAL, "token output is null");
  if (dev_probs_out && probs_stride < (size_t)draft->c.vocab) return fail(SSD_EINVAL, "probs_stride < vocab");
  if (kv_d->max_rows < kv_d->v.pcap) return fail(SSD_EINVAL, "cache rows too small");
  if ((rc = kv_check_flags(kv_d))) return rc;
  hipStream_t st = (hipStream_t)stream;
  // the token is drawn with the uniform of slot SSD_DRAFT_SLOT0 + draft_idx of this cycle: the step's only slot
  ssd_sample_config c2 = *cfg;
  c2.beta = 0.0f;
  rc = step(draft, kv_d, n_seqs, 0, nullptr, nullptr, &c2, step_ctr, SSD_DRAFT_SLOT0 + draft_idx, nullptr, dev_token_out, token_stride,
            dev_probs_out, probs_stride, true, nullptr, st);
  if (rc) return rc;
  for (int s = 0; s < n_seqs; ++s) { kv_d->len_ub[s] += kv_d->npend_ub[s]; kv_d->npend_ub[s] = 1; }
  return SSD_OK;
}

extern "C" int ssd_kv_rollback(ssd_kv* kv, int seq, int new_len, int pending_token, void* stream) {
  if (!kv) return fail(SSD_EINVAL, "null handle");
  if (seq < 0 || seq >= kv->max_seqs) return fail(SSD_EINVAL, "sequence %d out of range", seq);
  hipStream_t st = (hipStream_t)stream;
  int rc = kv_check_flags(kv);
  if (rc) return rc;
  // The host knows an upper bound of the length only; beyond it the request is refused here.  Between the device's length
  // and that bound the kernel refuses it: the state stays as it is and the next call on this cache reports the error.
  if (new_len < 0 || new_len > kv->len_ub[seq]) {
    if ((rc = kv_refresh(kv, st))) return rc;
    if (new_len < 0 || new_len > kv->len_ub[seq])
      return fail(SSD_EINVAL, "rollback to %d but sequence %d holds %d positions", new_len, seq, kv->len_ub[seq]);
  }
  hipLaunchKernelGGL(k_kv_set, dim3(1), dim3(BLOCK), 0, st, kv->v, seq, new_len, 0, 1, pending_token, (const int32_t*)nullptr, 0u);
  LAUNCH_CHECK();
  kv->len_ub[seq] = new_len;
  kv->npend_ub[seq] = 1;
  return SSD_OK;
}

extern "C" int ssd_kv_follow(ssd_kv* kv_d, int n_seqs, int K, const int32_t* dev_n_accepted,
                             const int32_t* dev_next_token, const int32_t* dev_draft_tokens, void* stream) {
  if (!kv_d || !dev_n_accepted || !dev_next_token || !dev_draft_tokens) return fail(SSD_EINVAL, "null argument");
  if (kv_d->v.pcap != 2) return fail(SSD_EINVAL, "ssd_kv_follow needs a draft cache (pending_cap 2)");
  if (n_seqs < 1 || n_seqs > kv_d->max_seqs || K < 1 || K > SSD_MAX_K) return fail(SSD_EINVAL, "bad n_seqs / K");
  {
    const int rc = kv_check_flags(kv_d);
    if (rc) return rc;
  }
  hipLaunchKernelGGL(k_kv_follow, dim3(1), dim3(cdiv(n_seqs, 64) * 64), 0, (hipStream_t)stream, kv_d->v, n_seqs, K, dev_n_accepted,
                     dev_next_token, dev_draft_tokens, (int32_t*)nullptr, 0);
  LAUNCH_CHECK();
  for (int s = 0; s < n_seqs; ++s) kv_d->npend_ub[s] = 2;       // the length can only have shrunk
  return SSD_OK;
}

// ------------------------------------------------------------------------------------------------ pieces
extern "C" int ssd_verify_from_probs(const float* dev_pt, const float* dev_pd, const int32_t* dev_tokens,
                                     const float* dev_uniforms, int B, int K, int V, float beta,
                                     int32_t* dev_n_accepted, int32_t* dev_next_token, int32_t* dev_flags, void* stream) {
  if (!dev_pt || !dev_uniforms || !dev_n_accepted || !dev_next_token) return fail(SSD_EINVAL, "null argument");
  if (B < 1 || K < 0 || K > SSD_MAX_K || V < 1 || V > 16384) return fail(SSD_EINVAL, "bad B / K / V");
  if (K > 0 && (!dev_pd || !dev_tokens)) return fail(SSD_EINVAL, "draft tokens / probabilities are null");
  if (!(beta >= 0.0f)) return fail(SSD_EINVAL, "beta must be >= 0");
  AcceptArgs a;
  memset(&a, 0, sizeof a);
  a.pt = dev_pt; a.pt_seq_stride = (size_t)(K + 1) * V; a.pd = dev_pd; a.x = dev_tokens; a.uniforms = dev_uniforms;
  a.B = B; a.K = K; a.V = V; a.beta = beta; a.n_acc = dev_n_accepted; a.next_tok = dev_next_token; a.tok_stride = 1;
  a.flags = dev_flags;
  SAMPLER(k_accept, V, B, (hipStream_t)stream, a);
  LAUNCH_CHECK();
  return SSD_OK;
}

extern "C" int ssd_warp_probs(const float* dev_logits, int rows, int V, const ssd_sample_config* cfg, float* dev_probs,
                              void* stream) {
  int rc = check_sample(cfg);
  if (rc) return rc;
  if (!dev_logits || !dev_probs || rows < 1 || V < 1 || V > 16384) return fail(SSD_EINVAL, "bad argument");
  WarpArgs w;
  w.logits = dev_logits; w.ld = V; w.V = V; w.temperature = cfg->temperature; w.top_k = cfg->top_k; w.greedy = cfg->greedy;
  w.probs = dev_probs; w.probs_stride = V;
  SAMPLER(k_warp_softmax, V, rows, (hipStream_t)stream, w);
  LAUNCH_CHECK();
  return SSD_OK;
}

// ------------------------------------------------------------------------------------------------ state
extern "C" int ssd_kv_state(ssd_kv* kv, int seq, void* stream, int32_t* len, int32_t* n_pending, int32_t pending[2],
                            int32_t* n_owned, int32_t* block_table, int block_table_cap) {
  if (!kv) return fail(SSD_EINVAL, "null handle");
  if (seq < 0 || seq >= kv->max_seqs) return fail(SSD_EINVAL, "sequence %d out of range", seq);
  hipStream_t st = (hipStream_t)stream;
  int rc = kv_refresh(kv, st);
  if (rc && rc != SSD_ENOMEM) return rc;
  int32_t own = 0;
  HIP_TRY(hipMemcpy(&own, kv->v.owned + seq, 4, hipMemcpyDeviceToHost));
  if (len) *len = kv->len_ub[seq];
  if (n_pending) *n_pending = kv->npend_ub[seq];
  if (pending) HIP_TRY(hipMemcpy(pending, kv->v.pend + 2 * seq, 8, hipMemcpyDeviceToHost));
  if (n_owned) *n_owned = own;
  if (block_table) {
    if (block_table_cap < own) return fail(SSD_ENOMEM, "block_table_cap %d < %d owned blocks", block_table_cap, own);
    if (own) HIP_TRY(hipMemcpy(block_table, kv->v.table + (size_t)seq * kv->v.mbps, (size_t)own * 4, hipMemcpyDeviceToHost));
  }
  return SSD_OK;
}

extern "C" int ssd_kv_free_stack(ssd_kv* kv, void* stream, int32_t* free_stack, int cap, int32_t* n_free,
                                 int32_t* dev_error_flag) {
  if (!kv) return fail(SSD_EINVAL, "null handle");
  HIP_TRY(hipStreamSynchronize((hipStream_t)stream));
  int32_t ctl[4];
  HIP_TRY(hipMemcpy(ctl, kv->v.ctl, sizeof ctl, hipMemcpyDeviceToHost));
  if (n_free) *n_free = ctl[0];
  uint32_t bar_err = 0;
  HIP_TRY(hipMemcpy(&bar_err, kv->bar + 64, 4, hipMemcpyDeviceToHost));
  if (dev_error_flag) *dev_error_flag = (ctl[1] & KV_ERR_POOL) | (bar_err ? 2 : 0) | (ctl[1] & KV_ERR_ROLLBACK);
  if (free_stack) {
    if (cap < ctl[0]) return fail(SSD_ENOMEM, "cap %d < %d free blocks", cap, ctl[0]);
    if (ctl[0]) HIP_TRY(hipMemcpy(free_stack, kv->v.free_stack, (size_t)ctl[0] * 4, hipMemcpyDeviceToHost));
  }
  return SSD_OK;
}

// ------------------------------------------------------------------------------------------------ errors on the device
extern "C" int ssd_kv_clear_error(ssd_kv* kv, void* stream) {
  if (!kv) return fail(SSD_EINVAL, "null handle");
  return kv_clear_sync_state(kv, (hipStream_t)stream);
}

extern "C" int ssd_kv_test_hook(ssd_kv* kv, int what, long long value, void* stream) {
  if (!kv) return fail(SSD_EINVAL, "null handle");
  hipStream_t st = (hipStream_t)stream;
  if (what == SSD_HOOK_TIMEOUT) {
    hipLaunchKernelGGL(k_kv_poke, dim3(1), dim3(1), 0, st, kv->v, DEV_ERR_TIMEOUT, 0);
  } else if (what == SSD_HOOK_LAUNCH_NUMBER) {
    if (value < 1 || value >= (long long)TAG_LIMIT) return fail(SSD_EINVAL, "launch number out of range");
    hipLaunchKernelGGL(k_kv_poke, dim3(1), dim3(1), 0, st, kv->v, 0u, (int)value);
    kv->launch_no = (uint32_t)value;
  } else if (what == SSD_HOOK_LAUNCH_NUMBER_DEVICE_ONLY) {
    if (value < 1 || value > (long long)TAG_LIMIT) return fail(SSD_EINVAL, "launch number out of range");
    hipLaunchKernelGGL(k_kv_poke, dim3(1), dim3(1), 0, st, kv->v, 0u, (int)value);
  } else {
    return fail(SSD_EINVAL, "unknown hook %d", what);
  }
  LAUNCH_CHECK();
  return SSD_OK;
}

// ------------------------------------------------------------------------------------------------ captured cycle
struct ssd_cycle {
  ssd_model *target, *draft;
  ssd_kv *kv, *kv_d;
  int n_seqs, K;
  ssd_sample_config cfg, dcfg;
  int32_t* x;
  float* pd;
  int32_t *n_acc, *next;
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
  int cap_len_t = -1, cap_len_d = -1;     // the captured launch shapes hold while every length bound stays at or below these
  int captures = 0;
  int wgs = 0;                            // workgroups of its largest forward
};

static void cycle_drop(ssd_cycle* c) {
  if (c->exec) (void)hipGraphExecDestroy(c->exec);
  if (c->graph) (void)hipGraphDestroy(c->graph);
  c->exec = nullptr; c->graph = nullptr;
}

// Host bookkeeping of one cycle's calls (the bounds the eager calls would have left).
static void cycle_advance_bounds(ssd_cycle* c) {
  for (int s = 0; s < c->n_seqs; ++s) {
    c->kv_d->len_ub[s] += c->kv_d->npend_ub[s] + (c->K - 1);
    c->kv_d->npend_ub[s] = 2;
    c->kv->len_ub[s] += c->K + 1;
    c->kv->npend_ub[s] = 1;
  }
}

// The calls of one cycle, which leave the bounds as the eager calls do (a capture keeps the ones it is made for).
static int cycle_steps(ssd_cycle* c, hipStream_t st) {
  const int K = c->K, V = c->target->c.vocab;
  const bool capture = c->kv->capturing;
  const int32_t* step_dev = c->kv->v.ctl + 4;
  ssd_sample_config dc = c->dcfg;
  dc.beta = 0.0f;
  int rc = SSD_OK;
  for (int i = 0; i < K && !rc; ++i) {
    rc = step(c->draft, c->kv_d, c->n_seqs, 0, nullptr, nullptr, &dc, 0, SSD_DRAFT_SLOT0 + i, nullptr, c->x + i, K,
              c->pd + (size_t)i * V, (size_t)K * V, true, nullptr, st, step_dev, false, i == 0);
    if (rc) return rc;
    for (int s = 0; s < c->n_seqs; ++s) {
      if (!capture) c->kv_d->len_ub[s] += c->kv_d->npend_ub[s];
      c->kv_d->npend_ub[s] = 1;                            // after a draft step exactly one token is pending
    }
  }
  if ((rc = step(c->target, c->kv, c->n_seqs, K, c->x, c->pd, &c->cfg, 0, 0, c->n_acc, c->next, 1, nullptr, 0, false,
                 nullptr, st, step_dev, false, true))) return rc;
  hipLaunchKernelGGL(k_kv_follow, dim3(1), dim3(cdiv(c->n_seqs, 64) * 64), 0, st, c->kv_d->v, c->n_seqs, K, c->n_acc, c->next, c->x,
                     c->kv->v.ctl + 4, capture ? 1 : 0);
  if (hipGetLastError() != hipSuccess) return fail(SSD_EHIP, "k_kv_follow launch failed");
  for (int s = 0; s < c->n_seqs && !capture; ++s) { c->kv->len_ub[s] += K + 1; c->kv->npend_ub[s] = 1; c->kv_d->npend_ub[s] = 2; }
  return SSD_OK;
}

static int cycle_capture(ssd_cycle* c, hipStream_t st) {
  cycle_drop(c);
  int rc;
  // exact lengths, room for the replays this capture will serve, numbering that cannot run out inside them
  if ((rc = kv_refresh(c->kv, st)) || (rc = kv_refresh(c->kv_d, st))) return rc;
  const int K = c->K;
  int max_t = 0, max_d = 0;
  for (int s = 0; s < c->n_seqs; ++s) { max_t = std::max(max_t, c->kv->len_ub[s]); max_d = std::max(max_d, c->kv_d->len_ub[s]); }
  // launch shapes (attention parts, workgroups) are those of a prefix up to 256 positions longer than today's
  const int ahead = 256;
  const int lim_t = std::min(c->target->max_positions, c->kv->v.mbps * c->kv->v.bt) - (K + 1);
  const int lim_d = std::min(c->draft->max_positions, c->kv_d->v.mbps * c->kv_d->v.bt) - (K + 2);
  c->cap_len_t = std::min(max_t + ahead, lim_t);
  c->cap_len_d = std::min(max_d + ahead, lim_d);
  if (c->cap_len_t < max_t || c->cap_len_d < max_d + K + 1) return fail(SSD_ENOMEM, "no room for another cycle");
  if ((rc = kv_check_room(c->kv, 0, c->n_seqs, K + 1, st)) || (rc = kv_check_room(c->kv_d, 0, c->n_seqs, K + 1, st))) return rc;
  std::vector<int> lt = c->kv->len_ub, ld = c->kv_d->len_ub, nt = c->kv->npend_ub, nd = c->kv_d->npend_ub;
  const uint32_t ln_t = c->kv->launch_no, ln_d = c->kv_d->launch_no;
  for (int s = 0; s < c->n_seqs; ++s) {
    c->kv->len_ub[s] = c->cap_len_t; c->kv_d->len_ub[s] = c->cap_len_d;
    c->kv->npend_ub[s] = 1; c->kv_d->npend_ub[s] = 2;      // the first draft step of a cycle may owe two tokens
  }
  c->kv->capturing = c->kv_d->capturing = true;
  c->kv->last_wgs = c->kv_d->last_wgs = 0;
  auto restore = [&]() { c->kv->len_ub = lt; c->kv_d->len_ub = ld; c->kv->npend_ub = nt; c->kv_d->npend_ub = nd;
                         c->kv->launch_no = ln_t; c->kv_d->launch_no = ln_d; c->kv->capturing = c->kv_d->capturing = false; };
  hipError_t e = hipStreamBeginCapture(st, hipStreamCaptureModeThreadLocal);
  if (e != hipSuccess) { restore(); return fail(SSD_EHIP, "hipStreamBeginCapture: %s", hipGetErrorString(e)); }
  rc = cycle_steps(c, st);
  c->wgs = std::max(c->kv->last_wgs, c->kv_d->last_wgs);
  hipGraph_t g = nullptr;
  e = hipStreamEndCapture(st, &g);
  restore();
  if (rc) { if (g) (void)hipGraphDestroy(g); return rc; }
  if (e != hipSuccess) return fail(SSD_EHIP, "hipStreamEndCapture: %s", hipGetErrorString(e));
  c->graph = g;
  e = hipGraphInstantiate(&c->exec, g, nullptr, nullptr, 0);
  if (e != hipSuccess) { cycle_drop(c); return fail(SSD_EHIP, "hipGraphInstantiate: %s", hipGetErrorString(e)); }
  ++c->captures;
  return SSD_OK;
}

extern "C" int ssd_cycle_create(ssd_model* target, ssd_kv* kv, ssd_model* draft, ssd_kv* kv_d, int n_seqs, int K,
                                const ssd_sample_config* cfg, const ssd_sample_config* dcfg, int32_t* dev_draft_tokens,
                                float* dev_draft_probs, int32_t* dev_n_accepted, int32_t* dev_next_token,
                                uint64_t first_step, void* stream, ssd_cycle** out) {
  int rc = check_pair(target, kv);
  if (rc || (rc = check_pair(draft, kv_d)) || (rc = check_sample(cfg)) || (rc = check_sample(dcfg))) return rc;
  if (!out || !dev_draft_tokens || !dev_draft_probs || !dev_n_accepted || !dev_next_token) return fail(SSD_EINVAL, "null argument");
  if (kv->v.pcap != 1 || kv_d->v.pcap != 2) return fail(SSD_EINVAL, "needs a target cache (pending_cap 1) and a draft cache (pending_cap 2)");
  if (n_seqs < 1 || n_seqs > kv->max_seqs || n_seqs > kv_d->max_seqs) return fail(SSD_EINVAL, "n_seqs %d out of range", n_seqs);
  if (K < 1 || K > SSD_MAX_K || K + 1 > kv->max_rows || kv_d->max_rows < 2) return fail(SSD_EINVAL, "K = %d out of range", K);
  if (target->c.vocab != draft->c.vocab) return fail(SSD_EINVAL, "target and draft vocabularies differ");
  if (!kv->dataflow || !kv_d->dataflow) return fail(SSD_ENOSUP, "a cycle can be captured only on the barrier-free forward kernel");
  ssd_cycle* c = new (std::nothrow) ssd_cycle();
  if (!c) return fail(SSD_ENOMEM, "host allocation failed");
  c->target = target; c->draft = draft; c->kv = kv; c->kv_d = kv_d; c->n_seqs = n_seqs; c->K = K;
  c->cfg = *cfg; c->dcfg = *dcfg; c->x = dev_draft_tokens; c->pd = dev_draft_probs; c->n_acc = dev_n_accepted;
  c->next = dev_next_token;
  const int32_t words[2] = {(int32_t)(uint32_t)first_step, (int32_t)(uint32_t)(first_step >> 32)};
  hipError_t e = hipMemcpyAsync(kv->v.ctl + 4, words, sizeof words, hipMemcpyHostToDevice, (hipStream_t)stream);
  if (e == hipSuccess) e = hipStreamSynchronize((hipStream_t)stream);       // `words` is on this stack frame
  if (e != hipSuccess) { delete c; return fail(SSD_EHIP, "cycle counter: %s", hipGetErrorString(e)); }
  *out = c;
  return SSD_OK;
}

extern "C" int ssd_cycle_launch(ssd_cycle* c, void* stream) {
  if (!c) return fail(SSD_EINVAL, "null handle");
  if (!stream) return fail(SSD_EINVAL, "a cycle cannot be captured on the default (NULL) stream: pass a stream of its own");
  hipStream_t st = (hipStream_t)stream;
  int rc;
  if ((rc = kv_check_flags(c->kv)) || (rc = kv_check_flags(c->kv_d))) return rc;
  const int K = c->K;
  if ((rc = kv_launch_guard(c->kv, st, 1)) || (rc = kv_launch_guard(c->kv_d, st, (uint32_t)K))) return rc;
  bool fits = c->exec != nullptr;
  for (int s = 0; s < c->n_seqs && fits; ++s)
    fits = c->kv->len_ub[s] <= c->cap_len_t && c->kv_d->len_ub[s] + K + 1 <= c->cap_len_d;
  if (fits) {                                              // pool room for this cycle, from the bounds alone
    long bt = 0, bd = 0;
    for (int s = 0; s < c->kv->max_seqs; ++s) bt += cdiv(c->kv->len_ub[s] + (s < c->n_seqs ? K + 1 : 0), c->kv->v.bt);
    for (int s = 0; s < c->kv_d->max_seqs; ++s) bd += cdiv(c->kv_d->len_ub[s] + (s < c->n_seqs ? K + 1 : 0), c->kv_d->v.bt);
    fits = bt <= c->kv->v.n_blocks && bd <= c->kv_d->v.n_blocks;
  }
  if (!fits && (rc = cycle_capture(c, st))) return rc;
  bool admitted;
  {
    const uint32_t cycles = c->kv_d->cycles;
    const ResidentLaunch order(c->kv_d, st, c->wgs, true);
    admitted = order.admitted;
    if (const hipError_t e = admitted ? hipGraphLaunch(c->exec, st) : hipSuccess; e != hipSuccess) {
      c->kv_d->run.cycle = c->kv_d->cycles = cycles;       // (nothing of it will say that it is over)
      return fail(SSD_EHIP, "hipGraphLaunch: %s", hipGetErrorString(e));
    }
  }
  if (!admitted) return cycle_steps(c, st);                // (call by call: those of its forwards that are not admitted either run one launch per operator)
  c->kv->launch_no += 1;
  c->kv_d->launch_no += (uint32_t)K;
  c->kv->last_path = 3;
  cycle_advance_bounds(c);
  return SSD_OK;
}

extern "C" int ssd_cycle_captures(const ssd_cycle* c) { return c ? c->captures : 0; }

extern "C" int ssd_cycle_destroy(ssd_cycle* c) {
  if (!c) return SSD_OK;
  cycle_drop(c);
  delete c;
  return SSD_OK;
}

// ------------------------------------------------------------------------------------------------ barrier trace
extern "C" int ssd_kv_last_forward_path(const ssd_kv* kv) { return kv ? kv->last_path : 0; }

extern "C" int ssd_trace_barriers(ssd_kv* kv, int enable, void* stream, unsigned long long* out, int cap, int* n_wgs,
                                  int* n_samples) {
  if (!kv) return fail(SSD_EINVAL, "null handle");
#ifndef SSD_TRACE
  (void)enable; (void)stream; (void)out; (void)cap; (void)n_wgs; (void)n_samples;
  return fail(SSD_ENOSUP, "this build records no phase trace (build with -DSSD_TRACE)");
#else
  if (out) {
    HIP_TRY(hipStreamSynchronize((hipStream_t)stream));
    const int G = kv->dataflow || kv->wide ? std::min(kv->cus, 256) : kv->persistent_wgs, S = 2 * (1 + 5 * kv->m->c.n_layers);
    if (G <= 0 || S > 512) return fail(SSD_ENOSUP, "no persistent kernel trace for this cache");
    if (cap < G * 512) return fail(SSD_ENOMEM, "cap %d < %d samples", cap, G * 512);
    HIP_TRY(hipMemcpy(out, kv->trace, sizeof(unsigned long long) * 512 * G, hipMemcpyDeviceToHost));
    if (n_wgs) *n_wgs = G;
    if (n_samples) *n_samples = S;
  }
  kv->trace_on = enable != 0;
  return SSD_OK;
#endif
}

// ------------------------------------------------------------------------------------------------ launch plans (host only)
static int gemm_pick_of(int kind, int rows, int n, int k, int cus, GemmPick& c, int max_rows = MAX_ROWS) {
  if (rows < 1 || rows > max_rows || n < 1 || k < 32 || k % 32 || cus < 1) return fail(SSD_EINVAL, "bad GEMM size");
  GemmArgs g;
  memset(&g, 0, sizeof g);
  g.M = rows; g.N = n; g.K = k;
  switch (kind) {
    case PROF_QKV: c = pick_gemm<EPI_QKV>(g, cus, 1); break;
    case PROF_O: c = pick_gemm<EPI_RESID>(g, cus, 1); break;
    case PROF_GATEUP: c = pick_gemm<EPI_SWIGLU>(g, cus, 1); break;
    case PROF_DOWN: {
      const int slices = partial_slices(MAX_ROWS, std::max(rows, MAX_ROWS));
      c = down_adds_residual(g, cus, slices) ? pick_gemm<EPI_RESID>(g, cus, 1) : pick_gemm<EPI_PARTIAL>(g, cus, slices);
      break;
    }
    case PROF_HEAD: c = pick_gemm<EPI_PARTIAL>(g, cus, 1); break;
    default: return fail(SSD_EINVAL, "no GEMM of kind %d", kind);
  }
  return SSD_OK;
}

static int gemm_blocks_of(const GemmPick& c, int* blocks, int cap) {
  for (int w = 0; w < std::min(cap, 8 * c.p.per_xcd); ++w) {
    int* b = blocks + 3 * (size_t)w;
    if (!tile_block(c.p, w, b[0], b[1], b[2])) b[0] = b[1] = b[2] = -1;
  }
  return 8 * c.p.per_xcd;
}

extern "C" int ssd_gemm_plan(int kind, int rows, int n, int k, int cus, int plan[4]) {
  GemmPick c;
  if (!plan) return fail(SSD_EINVAL, "bad GEMM size");
  if (int rc = gemm_pick_of(kind, rows, n, k, cus, c)) return rc;
  plan[0] = c.kernel; plan[1] = c.rt; plan[2] = c.ct; plan[3] = c.p.n_slices;
  return SSD_OK;
}

extern "C" int ssd_gemm_blocks(int kind, int rows, int n, int k, int cus, int* blocks, int cap) {
  GemmPick c;
  if (cap > 0 && !blocks) return fail(SSD_EINVAL, "no room for the blocks");
  if (int rc = gemm_pick_of(kind, rows, n, k, cus, c)) return rc;
  return gemm_blocks_of(c, blocks, cap);
}

extern "C" int ssd_prompt_gemm_plan(int kind, int rows, int n, int k, int cus, int plan[4], int* blocks, int cap) {
  GemmPick c;
  if (!plan || kind == PROF_HEAD || (cap > 0 && !blocks)) return fail(SSD_EINVAL, "bad GEMM size");
  if (int rc = gemm_pick_of(kind, rows, n, k, cus, c, MAX_PROMPT_ROWS)) return rc;
  GemmArgs g;
  memset(&g, 0, sizeof g);
  g.M = rows; g.N = n; g.K = k;
  plan[0] = c.kernel; plan[1] = c.rt; plan[2] = c.ct;
  plan[3] = kind == PROF_DOWN && down_adds_residual(g, cus, partial_slices(MAX_ROWS, std::max(rows, MAX_ROWS))) ? 0 : c.p.n_slices;
  return gemm_blocks_of(c, blocks, cap);
}

extern "C" int ssd_attention_plan(int head_dim, int n_q_heads, int n_kv_heads, int n_seqs, int rows, int prompt_positions, int cus, int plan[3]) {
  if (!plan || (head_dim != 64 && head_dim != 128) || n_kv_heads < 1 || n_q_heads < n_kv_heads || n_q_heads % n_kv_heads || n_seqs < 1 || rows < 1 ||
      rows * n_seqs > MAX_ROWS || prompt_positions < 0 || cus < 1)
    return fail(SSD_EINVAL, "bad attention size");
  const AttnPick c = pick_attn_mfma(head_dim, rows, n_q_heads / n_kv_heads, prompt_positions ? cdiv(prompt_positions, ATT_CHUNK) : ATT_PLAN_CHUNKS,
                                    prompt_positions > 0, n_kv_heads, n_seqs, cus);
  plan[0] = c.wq; plan[1] = c.wk; plan[2] = c.part_chunks;
  return SSD_OK;
}

extern "C" int ssd_resident_fits(const int* running, int n, int stream, int wgs, int cus) {
  constexpr int MOST = 64;
  Resident r[MOST];
  if (n < 0 || n > MOST || (n && !running) || cus < 1 || wgs < 1 || wgs > cus) return fail(SSD_EINVAL, "bad launches");
  for (int i = 0; i < n; ++i) {
    if (running[2 * i + 1] < 1 || running[2 * i + 1] > cus) return fail(SSD_EINVAL, "bad launch %d", i);
    r[i] = {(const void*)(size_t)running[2 * i], running[2 * i + 1]};
  }
  return resident_fits(r, n, (const void*)(size_t)stream, wgs, cus) ? 1 : 0;
}
