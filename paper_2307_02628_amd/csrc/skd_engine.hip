// Host engine behind the C ABI of include/skd.h: configuration checks, weight
// upload, the layer-sparse paged KV cache and the skip-aware layer loop that
// launches kernels for the active layers only (Sections 2.1-2.4).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <vector>

#include "../../include/skd.h"
#include "gave_up.h"
#include "skd_kernels.h"

using namespace skd;

static thread_local int g_last_hip = 0;
extern "C" int skd_last_hip_error(void) { return g_last_hip; }

#define HIPCHECK(expr)                         \
  do {                                         \
    hipError_t e_ = (expr);                    \
    if (e_ != hipSuccess) {                    \
      g_last_hip = (int)e_;                    \
      return e_ == hipErrorOutOfMemory ? SKD_ERR_NOMEM : SKD_ERR_HIP; \
    }                                          \
  } while (0)
#define SKDCHECK(expr)       \
  do {                       \
    int r_ = (expr);         \
    if (r_ < 0) return r_;   \
  } while (0)

// Scratch of skd_logits_argmax_noalloc: the per-workgroup (max, argmax) partials of the LM head, fp32 maxima in
// the first half and int32 indices in the second.  Every GPU the library runs on holds its own copy of this
// array at its own address until the process ends.  In host code the name below is only a handle for
// hipGetSymbolAddress; kernels are given the resolved device address.
#define SKD_NOALLOC_MAX_PARTIALS (1 << 18) /* workgroups of the LM head x padded batch rows */
static __device__ __align__(256) unsigned char scratch[2 * 4 * SKD_NOALLOC_MAX_PARTIALS];  // 2 MiB

namespace {

constexpr int kMaxDevices = 64;
void *g_scratch_ptr[kMaxDevices] = {};  // device address of `scratch` on each device, resolved once per device

// Called with `device` current (skd_create): looks the array's address up on that device.
int resolve_scratch(int device) {
  if (device < 0 || device >= kMaxDevices) return SKD_ERR_RANGE;
  if (g_scratch_ptr[device]) return SKD_OK;
  void *ptr = nullptr;
  HIPCHECK(hipGetSymbolAddress((void **)&ptr, HIP_SYMBOL(scratch)));
  if (!ptr) return SKD_ERR_HIP;
  g_scratch_ptr[device] = ptr;
  return SKD_OK;
}

struct LayerW {
  // matrices: fp32 row-major (debug path) or bf16 fragment-major (production path)
  void *wqkv = nullptr, *wo = nullptr, *w1 = nullptr, *w2 = nullptr;
  float *ln1_g = nullptr, *ln1_b = nullptr, *bqkv = nullptr, *bo = nullptr;
  float *ln2_g = nullptr, *ln2_b = nullptr, *b1 = nullptr, *b2 = nullptr;
};

struct GemmPlan {
  int R = 1, split = 1, U = 1, waves = 8;
  bool ws = false;  // 96 and 128 batch rows: the wave-specialised kernel (weight-streaming waves + activation-loading waves)
  int ws_rot = 0;   // workgroups start their K range at different stages
  int slots = 0;    // LM head: workgroups that run at once (bf16_head_tiles)
};

}  // namespace

namespace skd {
thread_local LaunchTimer *g_launch_timer = nullptr;
}

// hands the launches of one kernel class their event pairs (skd_profile_enable mode 1)
struct StateTimer final : LaunchTimer {
  skd_state *st = nullptr;
  int cls = 0;
  void next(hipEvent_t *start, hipEvent_t *stop) override;
};

// Pinned host memory of a bf16 state with host buffers: the kernels read tokens and uniform numbers from it and write
// tokens to it, and small logits are written or copied into it, so that a call needs one wait instead of one per copy.  Every call
// waits for its work before it returns, so the next one finds the buffers free.
constexpr size_t kPinnedLogits = 1 << 20;  // bytes; larger logits are copied to the caller's memory directly
struct Pinned {
  int32_t tok_in[128], tok_out[128];
  float u_in[128];
  float logits[kPinnedLogits / sizeof(float)];
};

struct skd_state {
  skd_config cfg{};
  Pinned *pin = nullptr;           // null: device I/O, fp32 path
  hipStream_t stream = nullptr;
  int B_pad = 0, dh = 0;
  bool bf16 = true;
  std::vector<void *> allocs;
  // weights
  std::vector<LayerW> lw;
  void *tok_emb = nullptr;  // row-major (gather)
  void *pos_emb = nullptr;  // row-major
  void *head = nullptr;     // LM head: fp32 row-major or bf16 fragment-major
  float *lnf_g = nullptr, *lnf_b = nullptr;
  // KV cache
  KvGeom geom{};
  void *pool = nullptr;
  int32_t *bt_dev = nullptr;       // [L][B][max_pages]
  std::vector<int32_t> bt_host;
  std::vector<int> kv_len, kv_cap; // columns held / columns reserved, per layer
  int64_t pages_reserved = 0, pages_dense = 0;
  // per-step device buffers
  int32_t *tok_dev = nullptr;      // [B] input column
  int32_t *prompt_dev = nullptr;   // [P][B]
  int32_t *order_dev = nullptr;    // [B] rows by descending real length (attention dispatch order)
  bool ragged = false;             // rows differ in length: use order_dev
  int32_t *start_dev = nullptr;    // [B] first real column
  std::vector<int32_t> start_host, order_host;
  int32_t *argmax_dev = nullptr;   // [B]
  float *u_dev = nullptr;          // [B] uniform numbers of the sampling head
  SampleScratch sample{};          // its candidates
  float *x = nullptr;              // residual stream fp32 [B_pad][d]
  float *x2 = nullptr;             // its second buffer (fuse_ln)
  bool fuse_ln = false;            // few rows: the row reducers are prologues of the projections behind them
  void *a = nullptr;               // LayerNorm output
  void *q = nullptr;               // bf16: q [B_pad][d]; fp32: qkv [B][3d]
  void *o = nullptr;               // attention output
  void *u = nullptr;               // FFN hidden
  float *partial = nullptr;        // bf16: split-K partials
  bf16_t *kv_new = nullptr;        // bf16: k and v of the column being processed, [B][k | v][d]
  float *attn_part = nullptr;      // bf16: split-KV partials; fp32: score scratch
  float *logits_dev = nullptr;     // [B][V] (fp32 path always; bf16 path when asked)
  float *pmax = nullptr;
  int32_t *pidx = nullptr;
  // plans (bf16)
  GemmPlan p_qkv, p_out, p_ffn1, p_ffn2, p_head;
  bool head_parts = false;         // the LM head's K range is split (p_head.split parts): partial sums, bf16_logits_sum
  int max_split = 1, attn_splits = 1, attn_waves = 4;
  bool attn_fixed = false;         // by override: the same shape at every position
  int start_min = 0;               // first real column of the longest row
  // whole columns in one launch (narrow models)
  bool team = false;
  bool team_always = false;        // by override: at every number of cached keys
  TeamArgs team_args{};            // what is the same for every column
  GaveUp team_gave_up;             // pinned host memory
  std::vector<unsigned char> team_table;  // source of the copy at the head of its buffers
  // batched prompt workspace (allocated by the first batched skd_prefill)
  float *pf_x = nullptr;
  float *pf_partial = nullptr;     // K parts of the prompt projections
  bf16_t *pf_a = nullptr, *pf_q = nullptr, *pf_o = nullptr, *pf_u = nullptr;
  CacheTile *pf_tiles = nullptr;  // cache place of each 16-row tile of the prompt pass
  int32_t *pf_seq = nullptr, *pf_first = nullptr;  // row map of the prompt pass (sequence of each row, first row of each sequence)
  int prefill_mode = 1;            // 1 = whole prompt per layer (bf16 path), 0 = column by column
  int prefill_tiles = 1;           // 1 = prompt projections as plan_rows says, 0 = 128-row chunks on the skinny kernel
  int prefill_wr = 0, prefill_ar = 0, prefill_split = 1;  // forced tile of the prompt projections (0 = plan_rows decides)
  int device = 0;                  // HIP device the state lives on
  // sequencing
  bool prefilled = false, have_hidden = false, have_argmax = false;
  int steps_done = 0;
  std::vector<int32_t> layers_tmp;
  std::vector<int32_t> n_table;    // caller-supplied layer counts per position (empty = the linear schedule)
  // per-kernel timing (off by default): 1 = each kernel's own begin/end time stamps, 2 = event brackets
  int profiling = 0;
  StateTimer timer;
  struct ProfRec { int cls; hipEvent_t a, b; };
  std::vector<ProfRec> prof_pending;
  std::vector<hipEvent_t> prof_free;
  double prof_ms[SKD_PROF_CLASSES] = {};
  int64_t prof_n[SKD_PROF_CLASSES] = {};
};

namespace {

template <typename T>
int dev_alloc(skd_state *st, T **out, size_t count) {
  void *p = nullptr;
  HIPCHECK(hipMalloc(&p, std::max<size_t>(count * sizeof(T), 256)));
  st->allocs.push_back(p);
  *out = (T *)p;
  return SKD_OK;
}

int env_int(const char *name, int dflt) {
  const char *v = getenv(name);
  return v && *v ? atoi(v) : dflt;
}

int check_config(const skd_config &c) {
  if (c.L < 1 || c.d_model < 1 || c.n_heads < 1 || c.ffn < 1 || c.vocab < 1 || c.max_pos < 1) return SKD_ERR_SHAPE;
  if (c.d_model % c.n_heads) return SKD_ERR_SHAPE;
  if (c.batch < 1 || c.prompt_size < 1 || c.sequence_length <= c.prompt_size) return SKD_ERR_SHAPE;
  if (c.max_pos < c.sequence_length) return SKD_ERR_SHAPE;
  if (c.n_min < 1 || c.n_min > c.n_max || c.n_max > c.L) return SKD_ERR_SHAPE;
  if (c.warmup < 0 || c.warmup > c.n_min) return SKD_ERR_SHAPE;
  if (c.page_tokens < 0 || c.page_tokens % 32) return SKD_ERR_SHAPE;
  if (c.dtype != SKD_BF16 && c.dtype != SKD_FP32) return SKD_ERR_SHAPE;
  if (c.io_on_device != 0 && c.io_on_device != 1) return SKD_ERR_SHAPE;
  if (c.dtype == SKD_BF16) {
    const int dh = c.d_model / c.n_heads;
    if (dh != 64 && dh != 128) return SKD_ERR_SHAPE;
    if (c.d_model % 32 || c.ffn % 32 || c.d_model > 16384) return SKD_ERR_SHAPE;
    if (c.batch > 128) return SKD_ERR_SHAPE;
  }
  return SKD_OK;
}

// Upload one tensor (host or device, fp32 or bf16) into a device staging area.
int stage(skd_state *st, const skd_weights &w, const void *src, size_t n, void *staging, const void **dev_src) {
  if (!src) return SKD_ERR_NULL;
  if (w.location == SKD_DEVICE) {
    *dev_src = src;
    return SKD_OK;
  }
  const size_t bytes = n * (w.elem == SKD_W_BF16 ? 2 : 4);
  HIPCHECK(hipMemcpyAsync(staging, src, bytes, hipMemcpyHostToDevice, st->stream));
  HIPCHECK(hipStreamSynchronize(st->stream));  // the staging area is reused by the next tensor
  *dev_src = staging;
  return SKD_OK;
}

int upload_vec(skd_state *st, const skd_weights &w, const void *src, size_t n, void *staging, float **out) {
  const void *dsrc = nullptr;
  SKDCHECK(stage(st, w, src, n, staging, &dsrc));
  SKDCHECK(dev_alloc(st, out, n));
  prep_to_f32(st->stream, dsrc, w.elem == SKD_W_BF16, *out, (long)n);
  HIPCHECK(hipStreamSynchronize(st->stream));
  return SKD_OK;
}

// matrix [N][K]: fp32 path -> fp32 row-major; bf16 path -> fragment-major (frag > 0) or row-major bf16
// (frag = tile-group size of the fragment-major layout, 0 = row-major)
int upload_mat(skd_state *st, const skd_weights &w, const void *src, long N, long K, void *staging, int frag,
               void **out) {
  const void *dsrc = nullptr;
  SKDCHECK(stage(st, w, src, (size_t)N * K, staging, &dsrc));
  if (!st->bf16) {
    float *p = nullptr;
    SKDCHECK(dev_alloc(st, &p, (size_t)N * K));
    prep_to_f32(st->stream, dsrc, w.elem == SKD_W_BF16, p, N * K);
    *out = p;
  } else if (frag) {
    const long N_pad = (N + 191) / 192 * 192;  // whole groups of 1..4 tiles: no wave tile ever leaves the buffer
    bf16_t *p = nullptr;
    SKDCHECK(dev_alloc(st, &p, (size_t)N_pad * K));
    prep_matrix_frag(st->stream, dsrc, w.elem == SKD_W_BF16, p, N, K, N_pad, frag);
    *out = p;
  } else {
    bf16_t *p = nullptr;
    SKDCHECK(dev_alloc(st, &p, (size_t)N * K));
    prep_matrix_rm_bf16(st->stream, dsrc, w.elem == SKD_W_BF16, p, N * K);
    *out = p;
  }
  HIPCHECK(hipStreamSynchronize(st->stream));
  return SKD_OK;
}

// Launch shapes.  Measured on MI355X at the OPT-6.7B widths: up to batch 64, 8
// waves per workgroup interleaving k-steps with 48-64 weight rows per workgroup
// and one k-step per register buffer stream best; at batch 96 and 128 the 4 x 6 and
// 4 x 8 tile accumulators need the whole register file, so workgroups have 4 waves.
// Every CU should get a workgroup; when K is split across workgroups a wave
// should still see at least 2 k-steps.
int plan_waves(int B_pad) { return B_pad >= 96 ? 4 : 8; }
GemmPlan plan_direct(int N, int B_pad) {  // whole K inside the workgroup
  GemmPlan p;
  p.waves = plan_waves(B_pad);
  p.split = 1;
  // several rounds of workgroups (the LM head): tile rows that keep the activation re-reads at half the weight
  // stream; with one batch tile, 2 rows do that and leave twice the workgroups to even out the last round
  p.R = B_pad >= 32 ? 4 : 2;
  if (bf16_gemm_groups(N, p.R) >= 512) return p;
  // one or two rounds: the R that keeps the largest share of the 256 CUs busy over whole rounds; ties go to the
  // larger R (measured: 768 tiles -> R = 3, 256 workgroups; 384 tiles -> R = 2, 192 workgroups beats 384)
  double best = -1.0;
  for (int R = 1; R <= 4; ++R) {
    const int g = bf16_gemm_groups(N, R);
    const double e = (double)g / (256.0 * ((g + 255) / 256));
    if (e >= best) { best = e; p.R = R; }
  }
  return p;
}
// The LM head of a large vocabulary: whole rounds of 256 workgroups of 4 tiles, smaller ones for what is left (head_dispatch
// in kernels_bf16.hip; 256: the CUs of the part that this is written for).  Four tiles at 16 rows too, us with the argmax, 2
// tiles -> 4: 16 rows, 20000 x 4096 33.2 -> 32.2, 32000 x 4096 48.0 -> 44.5, 50272 x 4096 72.8 -> 70.9, 65000 x 4096 95.8 ->
// 88.7; one row 32.5 -> 31.5, 47.3 -> 44.3, 71.1 -> 69.5, 88.4 -> 85.3; 32000 x 2048 28.1 -> 25.2, 20000 x 256 8.9 -> 8.3.
GemmPlan plan_head(int V, int B_pad) {
  GemmPlan p = plan_direct(V, B_pad);
  if (bf16_gemm_groups(V, 4) >= 256) {
    p.R = 4;
    p.slots = 256;
  }
  return p;
}
// An LM head of few tiles leaves most CUs idle and is a chain of k-steps for the others: its K range in as many parts as
// fill 256 CUs, of 16 k-steps at least; the kernel that finds the token adds the sums.  0: whole K in the workgroup.  us a call
// with the argmax, whole -> parts: 1000 x 4096, 4 parts: 1 row 11.1 -> 7.8, 16 9.1 -> 7.8, 47 14.0 -> 9.0, 128 23.2 -> 11.5; 500 x
// 4096, 8 parts: 10.9 -> 7.4, 8.8 -> 7.6, 13.3 -> 8.0, 22.8 -> 10.4; 2000 x 4096, 2 parts: 11.4 -> 9.6, 11.0 -> 9.6, 14.3 -> 11.7,
// 24.0 -> 16.5; 1000 x 2048, 4 parts: 8.6 -> 7.4, 7.5 -> 7.3, 10.0 -> 8.3, 15.0 -> 10.0.  Two rounds of workgroups lose (3000 x
// 4096, 2 parts: 12.0 -> 12.4, 11.8 -> 11.9, 14.4 -> 16.9, 24.6 -> 28.0), and so do parts of 8 k-steps (1000 x 512, 2 parts: 7.3 -> 7.4,
// 7.2 -> 7.6, 7.3 -> 7.6, 8.6 -> 8.8).
int plan_head_split(int V, int K) {
  const int tiles = (V + 15) / 16, Kf = K / 32;
  int S = 1;
  while (2 * S <= LOGITS_SPLIT && tiles * 2 * S <= 256 && Kf % (2 * S) == 0 && Kf / (2 * S) >= 16) S *= 2;
  return S > 1 ? S : 0;
}
GemmPlan plan_split(int N, int K, int B_pad) {  // partial sums, reduced by the LayerNorm kernel
  GemmPlan p;
  p.waves = plan_waves(B_pad);
  // A wave of these K ranges has 1 (K = 256) to 32 k-steps (16384, split by 2): two per buffer with one batch tile (1.3B
  // model, 16 rows, 8 steps: 7172 -> 7029 us; 6.7B widths, 8 rows: 921 -> 918); four put too much in flight (7118), and
  // wider batches have no registers to gain from it.  At K = 256 and 384 two leave waves without a buffer of their own;
  // the launch takes 4.2 to 4.5 us either way
  if (B_pad <= 16) p.U = 2;
  const int Kf = K / 32;
  // tile rows per workgroup: enough that the activation re-reads (B_pad / (16 R) of the weight bytes) stay at
  // half the weight stream; more rows than that only force a deeper split, whose partials the reducer pays for
  p.R = B_pad >= 32 ? 4 : 2;
  while (p.R > 1 && N % (16 * p.R)) --p.R;
  for (;;) {
    int S = 1;
    while (S < 16 && bf16_gemm_groups(N, p.R) * S < 256 && Kf % (2 * S) == 0 && Kf / (2 * S) >= 2 * p.waves) S *= 2;
    p.split = S;
    if (bf16_gemm_groups(N, p.R) * S >= 256 || p.R == 1) break;
    --p.R;
    while (p.R > 1 && N % (16 * p.R)) --p.R;
  }
  return p;
}

// Active layers at position t for this state: the linear schedule of the
// configuration, or the caller's table (same shape of the set: warm-up layers
// at the bottom, the rest of the budget at the top).
int state_active_layers(const skd_state *st, int t, int32_t *out) {
  const skd_config &c = st->cfg;
  if (st->n_table.empty()) return skd_active_layers(t, &c, out);
  if (t < 0 || t >= c.sequence_length) return SKD_ERR_RANGE;
  const int n = st->n_table[t];
  int k = 0;
  for (int l = 0; l < c.warmup; ++l) out[k++] = l;
  for (int l = c.L - (n - c.warmup); l < c.L; ++l) out[k++] = l;
  return k;
}

int build_kv(skd_state *st) {
  const skd_config &c = st->cfg;
  const int pt = c.page_tokens ? c.page_tokens : 64;
  KvGeom &g = st->geom;
  g.page_tokens = pt;
  g.max_pages = (c.sequence_length + pt - 1) / pt;
  g.H = c.n_heads;
  g.dh = st->dh;
  g.page_elems = 2L * pt * c.d_model;
  // Static policy: the columns at which each layer runs are known before
  // generation starts, so each layer reserves exactly what it will hold.
  st->kv_cap.assign(c.L, 0);
  std::vector<int32_t> act(c.L);
  for (int t = 0; t < c.sequence_length; ++t) {
    const int n = state_active_layers(st, t, act.data());
    if (n < 0) return n;
    for (int i = 0; i < n; ++i) {
      if (st->kv_cap[act[i]] != t) return SKD_ERR_SCHEDULE;  // a layer re-entered: its cache would have a hole
      st->kv_cap[act[i]] = t + 1;
    }
  }
  st->bt_host.assign((size_t)c.L * c.batch * g.max_pages, -1);
  int64_t next = 0;
  // Page order inside a layer is position-major (all rows' page 0, then all
  // rows' page 1, ...): the B*H workgroups of the attention kernel advance
  // through their keys in step, so at any moment the chip reads one dense
  // B-MiB-scale window instead of B windows a fixed large stride apart
  // (measured: up to 13 % faster attention when a row holds 12 pages).
  for (int l = 0; l < c.L; ++l) {
    const int np = (st->kv_cap[l] + pt - 1) / pt;
    for (int p = 0; p < np; ++p)
      for (int b = 0; b < c.batch; ++b) st->bt_host[((size_t)l * c.batch + b) * g.max_pages + p] = (int32_t)next++;
  }
  if (next > 0x7fffffffLL) return SKD_ERR_NOMEM;
  st->pages_reserved = next;
  st->pages_dense = (int64_t)c.L * c.batch * g.max_pages;
  const size_t esz = st->bf16 ? 2 : 4;
  const size_t bytes = (size_t)next * g.page_elems * esz;
  void *pool = nullptr;
  HIPCHECK(hipMalloc(&pool, std::max<size_t>(bytes, 256)));
  st->allocs.push_back(pool);
  st->pool = pool;
  // unwritten slots must hold finite values: a masked key still meets its V in the MFMA
  HIPCHECK(hipMemsetAsync(pool, 0, bytes, st->stream));
  SKDCHECK(dev_alloc(st, &st->bt_dev, st->bt_host.size()));
  HIPCHECK(hipMemcpyAsync(st->bt_dev, st->bt_host.data(), st->bt_host.size() * sizeof(int32_t), hipMemcpyHostToDevice,
                          st->stream));
  HIPCHECK(hipStreamSynchronize(st->stream));
  st->kv_len.assign(c.L, 0);
  return SKD_OK;
}

hipEvent_t prof_event(skd_state *st) {
  if (!st->prof_free.empty()) {
    hipEvent_t e = st->prof_free.back();
    st->prof_free.pop_back();
    return e;
  }
  hipEvent_t e = nullptr;
  (void)hipEventCreate(&e);
  return e;
}
// Times the launches issued inside its scope when profiling is on: mode 1 gives every launch its own event
// pair, stamped with the kernel's begin and end; mode 2 records one event before and one after the launches.
struct ProfScope {
  skd_state *st;
  int cls;
  hipEvent_t a = nullptr;
  ProfScope(skd_state *s, int c) : st(s), cls(c) {
    if (st->profiling == 1) {
      st->timer.st = st;
      st->timer.cls = cls;
      skd::g_launch_timer = &st->timer;
    } else if (st->profiling == 2) {
      a = prof_event(st);
      if (a) (void)hipEventRecord(a, st->stream);
    }
  }
  ~ProfScope() {
    skd::g_launch_timer = nullptr;
    if (a) {
      hipEvent_t b = prof_event(st);
      if (b) (void)hipEventRecord(b, st->stream);
      st->prof_pending.push_back({cls, a, b});
    }
  }
};
}  // namespace
void StateTimer::next(hipEvent_t *start, hipEvent_t *stop) {
  *start = prof_event(st);
  *stop = prof_event(st);
  st->prof_pending.push_back({cls, *start, *stop});
}
namespace {
int prof_drain(skd_state *st) {
  HIPCHECK(hipStreamSynchronize(st->stream));
  for (auto &r : st->prof_pending) {
    float ms = 0.f;
    if (r.a && r.b && hipEventElapsedTime(&ms, r.a, r.b) == hipSuccess) {
      st->prof_ms[r.cls] += ms;
      st->prof_n[r.cls] += 1;
    }
    if (r.a) st->prof_free.push_back(r.a);
    if (r.b) st->prof_free.push_back(r.b);
  }
  st->prof_pending.clear();
  return SKD_OK;
}

const int32_t *bt_layer(const skd_state *st, int l) {
  return st->bt_dev + (size_t)l * st->cfg.batch * st->geom.max_pages;
}

// a decode projection on the kernel its plan names; returns the row groups launched or -1
int launch_gemm(hipStream_t s, GemmArgs &ga, int epi, const GemmPlan &p) {
  ga.ws_rot = p.ws_rot;
  return p.ws ? bf16_gemm_ws(s, ga, epi, p.R) : bf16_gemm(s, ga, epi, p.R, p.U, p.waves);
}
int check_gemm(const GemmArgs &ga, int epi, const GemmPlan &p) {
  return p.ws ? bf16_gemm_ws_check(ga, epi, p.R) : bf16_gemm_check(ga, epi, p.R, p.U, p.waves);
}

// The projections of a layer (the same shapes in every layer) and the LM head against what the kernels can launch.
bool decode_shapes_ok(const skd_state *st) {
  const skd_config &c = st->cfg;
  const int d = c.d_model, f = c.ffn;
  GemmArgs ga{};
  ga.B = c.batch; ga.B_pad = st->B_pad;
  auto ok = [&](int N, int K, const GemmPlan &p, int epi) {
    ga.N = N; ga.K = K; ga.G = p.R; ga.split = p.split;
    if (epi == EPI_LOGITS) bf16_head_tiles(ga, p.R, p.slots);
    return check_gemm(ga, epi, p) > 0;
  };
  const int head_n = st->head_parts ? (c.vocab + 15) / 16 * 16 : c.vocab;
  auto ok_ln = [&](int N, const GemmPlan &p, const GemmPlan &before, int epi) {  // behind the partial sums of `before`
    ga.N = N; ga.K = d; ga.G = p.R; ga.split = p.split; ga.ln_split = before.split;
    return bf16_gemm_ln_check(ga, epi, p.R) > 0;
  };
  return ok(3 * d, d, st->p_qkv, EPI_QKV) && ok(d, d, st->p_out, EPI_PARTIAL) && ok(f, d, st->p_ffn1, EPI_RELU) &&
         ok(d, f, st->p_ffn2, EPI_PARTIAL) && ok(head_n, d, st->p_head, st->head_parts ? EPI_PARTIAL : EPI_LOGITS) &&
         (!st->fuse_ln || (ok_ln(3 * d, st->p_qkv, st->p_ffn2, EPI_QKV) && ok_ln(f, st->p_ffn1, st->p_out, EPI_RELU)));
}

// Waves per workgroup and workgroups per (row, head) of decode attention at position t: no more waves than there are
// 32-key blocks, and up to 16 blocks in one workgroup (a split needs a second kernel: at 16 to 32 keys of two rows of 4
// heads, one block, attention + merge of 8 splits took 9.9 us, without a split 3.9).  Where fewer (row, head) pairs than
// CUs share long rows, the workgroups are spread over the CUs first and get the waves that are left (one row of 32
// heads at 2000 keys, 63 blocks: 8 workgroups of 8 waves instead of 8 of 16, half of them idle).
void attn_shape(const skd_state *st, int t, int &waves, int &splits) {
  waves = st->attn_waves;
  splits = st->attn_splits;
  if (st->attn_fixed) return;
  const int nblk = (t - st->start_min + 31) / 32;
  if (nblk <= 16) splits = 1;
  while (waves > 2 && waves / 2 * splits >= nblk) waves /= 2;
}

// One layer of the column at position t on the bf16 path.  st->a holds LayerNorm 1 of its input, st->x the residual
// stream; next: the active layer that follows (null: none), whose LayerNorm 1, or the final one, the reducer of the last
// sub-block applies.
// With few rows (st->fuse_ln) the reducers between the projections of a layer, and between layers, are the prologues of
// the projections that follow: prev (null: the first layer of the column) is the layer whose FFN2 partial sums are
// still to be added to st->x, and the residual stream alternates between st->x and st->x2.
int run_layer(skd_state *st, int l, int t, const LayerW *prev, const LayerW *next) {
  const skd_config &c = st->cfg;
  const int B = c.batch, d = c.d_model, f = c.ffn;
  hipStream_t s = st->stream;
  bf16_t *a = (bf16_t *)st->a, *q = (bf16_t *)st->q, *o = (bf16_t *)st->o, *u = (bf16_t *)st->u;
  const LayerW &w = st->lw[l];
  int grc = 0;
  GemmArgs ga{};
  ga.B = B; ga.B_pad = st->B_pad; ga.kv = st->geom; ga.d = d;
  // q, k, v projection; the attention kernel files k and v into this layer's page slot for column t
  ga.W = (const bf16_t *)w.wqkv; ga.G = st->p_qkv.R; ga.A = a; ga.bias = w.bqkv; ga.N = 3 * d; ga.K = d; ga.split = 1;
  ga.q_out = q; ga.kv_new = st->kv_new;
  ga.ln_partial = st->partial;
  if (st->fuse_ln && prev) {
    ga.ln_x = st->x2; ga.ln_x_out = st->x; ga.ln_split = st->p_ffn2.split; ga.ln_bias = prev->b2; ga.ln_g = w.ln1_g; ga.ln_b = w.ln1_b;
    { ProfScope ps_(st, SKD_PROF_GEMM_QKV); grc = bf16_gemm_ln(s, ga, EPI_QKV, st->p_qkv.R); }
  } else {
    ProfScope ps_(st, SKD_PROF_GEMM_QKV);
    grc = launch_gemm(s, ga, EPI_QKV, st->p_qkv);
  }
  if (grc < 0) return SKD_ERR_SHAPE;
  AttnArgs aa{};
  aa.q = q; aa.kv_new = st->kv_new; aa.pool = (bf16_t *)st->pool; aa.bt_layer = bt_layer(st, l); aa.start = st->start_dev; aa.order = st->ragged ? st->order_dev : nullptr;
  aa.t = t; aa.B = B; attn_shape(st, t, aa.waves, aa.splits); aa.kv = st->geom; aa.o = o; aa.part = st->attn_part;
  // output projection -> partials; bias + residual + LayerNorm 2 in the reducer
  ga.W = (const bf16_t *)w.wo; ga.G = st->p_out.R; ga.A = o; ga.N = d; ga.K = d; ga.split = st->p_out.split; ga.partial = st->partial;
  ga.attn_part = st->attn_part; ga.attn_splits = aa.splits;
  // one or two rows: the projection merges the attention's splits
  aa.merge = !(st->fuse_ln && bf16_gemm_merge_check(ga, st->p_out.R, st->p_out.waves) > 0);
  { ProfScope ps_(st, SKD_PROF_ATTENTION); bf16_attention(s, aa); }
  {
    ProfScope ps_(st, SKD_PROF_GEMM_OUT);
    grc = aa.splits > 1 && !aa.merge ? bf16_gemm_merge(s, ga, st->p_out.R, st->p_out.U, st->p_out.waves) : launch_gemm(s, ga, EPI_PARTIAL, st->p_out);
  }
  if (grc < 0) return SKD_ERR_SHAPE;
  if (!st->fuse_ln) { ProfScope ps_(st, SKD_PROF_REDUCE_LN); bf16_reduce_ln(s, st->partial, st->p_out.split, st->B_pad, w.bo, st->x, st->x, w.ln2_g, w.ln2_b, a, B, d); }
  ga.W = (const bf16_t *)w.w1; ga.G = st->p_ffn1.R; ga.A = a; ga.bias = w.b1; ga.N = f; ga.K = d; ga.split = 1; ga.act_out = u;
  if (st->fuse_ln) {
    ga.ln_x = st->x; ga.ln_x_out = st->x2; ga.ln_split = st->p_out.split; ga.ln_bias = w.bo; ga.ln_g = w.ln2_g; ga.ln_b = w.ln2_b;
    { ProfScope ps_(st, SKD_PROF_GEMM_FFN1); grc = bf16_gemm_ln(s, ga, EPI_RELU, st->p_ffn1.R); }
  } else {
    ProfScope ps_(st, SKD_PROF_GEMM_FFN1);
    grc = launch_gemm(s, ga, EPI_RELU, st->p_ffn1);
  }
  if (grc < 0) return SKD_ERR_SHAPE;
  ga.W = (const bf16_t *)w.w2; ga.G = st->p_ffn2.R; ga.A = u; ga.N = d; ga.K = f; ga.split = st->p_ffn2.split;
  { ProfScope ps_(st, SKD_PROF_GEMM_FFN2); grc = launch_gemm(s, ga, EPI_PARTIAL, st->p_ffn2); }
  if (grc < 0) return SKD_ERR_SHAPE;
  if (st->fuse_ln && next) return SKD_OK;  // the next layer adds the partial sums
  const float *next_g = next ? next->ln1_g : st->lnf_g, *next_b = next ? next->ln1_b : st->lnf_b;
  { ProfScope ps_(st, SKD_PROF_REDUCE_LN); bf16_reduce_ln(s, st->partial, st->p_ffn2.split, st->B_pad, w.b2, st->fuse_ln ? st->x2 : st->x, st->x, next_g, next_b, a, B, d); }
  return SKD_OK;
}

// Whether the column at position t is one that the one-launch kernel does faster (bf16_team_keys).
bool team_keys(const skd_state *st, int t) {
  int64_t total = 0;
  for (int b = 0; b < st->cfg.batch; ++b) total += std::max(0, t - (st->start_host.empty() ? 0 : st->start_host[b]));
  return st->team_always || bf16_team_keys(st->cfg.d_model, st->cfg.batch, t - st->start_min, total);
}

// Whether the list is what a schedule gives: warm-up layers, then the top of the stack.
bool scheduled_set(const skd_state *st, const int32_t *layers, int n) {
  const skd_config &c = st->cfg;
  for (int i = 0; i < n; ++i)
    if (layers[i] != (i < c.warmup ? i : c.L - n + i)) return false;
  return n >= c.warmup;
}

// One column (all B rows at position t) through the given ascending layer list.  Everything that can refuse
// the column (layer list, cache lengths, launch shapes) is checked before the first launch, so an error leaves
// the caches as they were.
int run_column(skd_state *st, int t, const int32_t *tokens_dev, const int32_t *layers, int n) {
  const skd_config &c = st->cfg;
  const int B = c.batch, d = c.d_model, f = c.ffn;
  hipStream_t s = st->stream;
  for (int i = 0; i < n; ++i) {
    const int l = layers[i];
    if (l < 0 || l >= c.L || (i && layers[i - 1] >= l)) return SKD_ERR_SCHEDULE;
    if (st->kv_len[l] != t) return SKD_ERR_ORDER;  // every earlier key of an active layer must exist
    if (t >= st->kv_cap[l]) return SKD_ERR_NOMEM;
  }
  if (st->bf16 && !decode_shapes_ok(st)) return SKD_ERR_SHAPE;  // before the first launch: nothing is half done
  if (!st->bf16) {
    float *a = (float *)st->a, *qkv = (float *)st->q, *o = (float *)st->o, *u = (float *)st->u;
    { ProfScope ps_(st, SKD_PROF_OTHER); f32_embed(s, st->x, (const float *)st->tok_emb, (const float *)st->pos_emb, tokens_dev, st->start_dev, t, B, d, c.vocab); }
    for (int i = 0; i < n; ++i) {
      const LayerW &w = st->lw[layers[i]];
      { ProfScope ps_(st, SKD_PROF_OTHER); f32_layernorm(s, st->x, w.ln1_g, w.ln1_b, a, B, d); }
      { ProfScope ps_(st, SKD_PROF_OTHER); f32_linear(s, (const float *)w.wqkv, w.bqkv, a, qkv, B, d, 3 * d, 0, 0); }
      { ProfScope ps_(st, SKD_PROF_OTHER); f32_kv_write(s, qkv, (float *)st->pool, bt_layer(st, layers[i]), t, B, st->geom); }
      { ProfScope ps_(st, SKD_PROF_OTHER); f32_attention(s, qkv, (const float *)st->pool, bt_layer(st, layers[i]), st->start_dev, t, o, st->attn_part, c.sequence_length, B, st->geom); }
      { ProfScope ps_(st, SKD_PROF_OTHER); f32_linear(s, (const float *)w.wo, w.bo, o, st->x, B, d, d, 0, 1); }
      { ProfScope ps_(st, SKD_PROF_OTHER); f32_layernorm(s, st->x, w.ln2_g, w.ln2_b, a, B, d); }
      { ProfScope ps_(st, SKD_PROF_OTHER); f32_linear(s, (const float *)w.w1, w.b1, a, u, B, d, f, 1, 0); }
      { ProfScope ps_(st, SKD_PROF_OTHER); f32_linear(s, (const float *)w.w2, w.b2, u, st->x, B, f, d, 0, 1); }
      st->kv_len[layers[i]] = t + 1;
    }
  } else if (st->team && !st->profiling && scheduled_set(st, layers, n) && team_keys(st, t)) {  // per-kernel timing times separate kernels
    TeamArgs ta = st->team_args;
    ta.n = n;
    ta.t = t;
    ta.longest = t - st->start_min;
    attn_shape(st, t, ta.attn_waves, ta.attn_splits);
    ta.tokens = tokens_dev;
    ta.order = st->ragged ? st->order_dev : nullptr;
    if (!bf16_team_column(s, ta)) return SKD_ERR_SHAPE;
    for (int i = 0; i < n; ++i) st->kv_len[layers[i]] = t + 1;
  } else {
    const LayerW &w0 = st->lw[layers[0]];
    { ProfScope ps_(st, SKD_PROF_EMBED_LN); bf16_embed_ln(s, tokens_dev, st->start_dev, t, (const bf16_t *)st->tok_emb, (const bf16_t *)st->pos_emb, w0.ln1_g, w0.ln1_b, st->x, (bf16_t *)st->a, B, d, c.vocab); }
    for (int i = 0; i < n; ++i) {
      SKDCHECK(run_layer(st, layers[i], t, i ? &st->lw[layers[i - 1]] : nullptr, i + 1 < n ? &st->lw[layers[i + 1]] : nullptr));
      st->kv_len[layers[i]] = t + 1;
    }
  }
  HIPCHECK(hipGetLastError());
  st->have_hidden = true;
  st->have_argmax = false;
  return SKD_OK;
}

}  // namespace

// Whether a launch shape of the separate decode kernels is forced: then they are what is to run.
static bool launch_overrides() {
  for (const char *p : {"SKD_R_", "SKD_S_", "SKD_U_", "SKD_W_"})
    for (const char *m : {"QKV", "OUT", "FFN1", "FFN2", "HEAD"}) {
      char name[16];
      snprintf(name, sizeof(name), "%s%s", p, m);
      if (getenv(name)) return true;
    }
  for (const char *name : {"SKD_ATTN_WAVES", "SKD_ATTN_SPLITS", "SKD_FUSE_LN", "SKD_GEMM_WS", "SKD_WS_ROT"})
    if (getenv(name)) return true;
  return false;
}

// Buffers and layer table of bf16_team_column.
static int prepare_team(skd_state *st) {
  const skd_config &c = st->cfg;
  const int L = c.L, d = c.d_model, f = c.ffn;
  TeamArgs &ta = st->team_args;
  ta.d = d; ta.f = f; ta.B = c.batch; ta.V = c.vocab;
  ta.kv = st->geom;
  ta.groups = bf16_team_groups(c.batch);
  auto sums = [](const GemmPlan &p) { return TeamSums{p.R, p.ws ? 4 : p.waves, p.ws ? 1 : p.U, p.split, p.ws && p.ws_rot}; };
  auto take_sums = [&](TeamStep *out, TeamStep *ffn2) {
    return bf16_team_sums(ta, st->B_pad, sums(st->p_qkv), sums(st->p_out), sums(st->p_ffn1), sums(st->p_ffn2), out, ffn2);
  };
  if (!take_sums(nullptr, nullptr) || !bf16_team_states(ta, st->attn_waves, st->attn_splits)) return SKD_OK;  // separate kernels
  void *word = nullptr;
  HIPCHECK(hipHostMalloc(&word, sizeof(uint32_t), hipHostMallocDefault));
  st->team_gave_up.word = (volatile uint32_t *)word;
  *st->team_gave_up.word = 0;
  ta.gave_up = (uint32_t *)word;
  int cus = 0;
  HIPCHECK(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, st->device));
  // one allocation and one copy: control words (zero), layer table and step tables, then the work buffers
  const size_t rows = bf16_team_rows(), steps = bf16_team_steps(d);
  const size_t head = (sizeof(TeamCtl) + L * sizeof(TeamLayer) + 2 * steps * sizeof(TeamStep) + 255) / 256 * 256;
  const size_t n16[] = {rows * d, rows * 2 * d, rows * d, rows * f}, n32[] = {rows * d, bf16_team_part()};  // multiples of 128 each
  unsigned char *base = nullptr;
  SKDCHECK(dev_alloc(st, &base, head + 2 * (n16[0] + n16[1] + n16[2] + n16[3]) + 4 * (n32[0] + n32[1])));
  st->team_table.assign(head, 0);
  TeamLayer *host = (TeamLayer *)(st->team_table.data() + sizeof(TeamCtl));
  for (int l = 0; l < L; ++l) {
    const LayerW &w = st->lw[l];
    host[l] = TeamLayer{(const bf16_t *)w.wqkv, (const bf16_t *)w.wo, (const bf16_t *)w.w1, (const bf16_t *)w.w2, w.ln1_g, w.ln1_b,
                        w.bqkv, w.bo, w.ln2_g, w.ln2_b, w.b1, w.b2, bt_layer(st, l)};
  }
  const size_t at_steps = sizeof(TeamCtl) + L * sizeof(TeamLayer);
  TeamStep *host_steps = (TeamStep *)(st->team_table.data() + at_steps);
  if (!take_sums(host_steps, host_steps + steps)) return SKD_ERR_SHAPE;
  HIPCHECK(hipMemcpyAsync(base, st->team_table.data(), head, hipMemcpyHostToDevice, st->stream));  // create waits for it
  ta.ctl = (TeamCtl *)base;
  ta.layers = (const TeamLayer *)(base + sizeof(TeamCtl));
  ta.out_steps = (const TeamStep *)(base + at_steps);
  ta.ffn2_steps = ta.out_steps + steps;
  base += head;
  bf16_t **p16[] = {&ta.work.q, &ta.work.kv, &ta.work.o, &ta.work.u};
  for (int i = 0; i < 4; base += 2 * n16[i++]) *p16[i] = (bf16_t *)base;
  ta.work.y = (float *)base;
  ta.work.part = (float *)(base + 4 * n32[0]);
  ta.warmup = c.warmup; ta.L = L;
  ta.workgroups = std::max(cus, 1);
  ta.members = bf16_team_members(cus, d);
  if (const int m = env_int("SKD_TEAM_WGS", 0); m >= 1 && m <= ta.members) ta.members = m;
  ta.start = st->start_dev;
  ta.tok_emb = (const bf16_t *)st->tok_emb; ta.pos_emb = (const bf16_t *)st->pos_emb;
  ta.lnf_g = st->lnf_g; ta.lnf_b = st->lnf_b;
  ta.pool = (bf16_t *)st->pool;
  ta.x_out = st->x; ta.a_out = (bf16_t *)st->a;
  st->team = true;
  st->team_always = env_int("SKD_TEAM", 1) == 2;
  return SKD_OK;
}

static int create_impl(const skd_config *cfg, const skd_weights *w, void *hip_stream, const int32_t *n_table,
                       skd_state **out) {
  if (!cfg || !w || !out) return SKD_ERR_NULL;
  *out = nullptr;
  SKDCHECK(check_config(*cfg));
  if (n_table) {  // monotone, within [max(1, warmup), L]
    for (int i = 0; i < cfg->sequence_length; ++i) {
      if (n_table[i] < 1 || n_table[i] > cfg->L) return SKD_ERR_RANGE;
      if (n_table[i] < cfg->warmup) return SKD_ERR_SHAPE;
      if (i && n_table[i] > n_table[i - 1]) return SKD_ERR_SCHEDULE;
    }
  }
  if ((w->location != SKD_HOST && w->location != SKD_DEVICE) || (w->elem != SKD_W_FP32 && w->elem != SKD_W_BF16))
    return SKD_ERR_SHAPE;
  if (!w->tok_emb || !w->pos_emb || !w->lnf_g || !w->lnf_b || !w->ln1_g || !w->ln1_b || !w->wqkv || !w->bqkv ||
      !w->wo || !w->bo || !w->ln2_g || !w->ln2_b || !w->w1 || !w->b1 || !w->w2 || !w->b2)
    return SKD_ERR_NULL;
  skd_state *st = new (std::nothrow) skd_state();
  if (!st) return SKD_ERR_NOMEM;
  auto fail = [&](int rc) {
    skd_destroy(st);
    return rc;
  };
  st->cfg = *cfg;
  if (n_table) st->n_table.assign(n_table, n_table + cfg->sequence_length);
  if (!st->cfg.page_tokens) st->cfg.page_tokens = 64;
  st->stream = (hipStream_t)hip_stream;
  st->bf16 = cfg->dtype == SKD_BF16;
  st->dh = cfg->d_model / cfg->n_heads;
  const skd_config &c = st->cfg;
  const int B = c.batch, d = c.d_model, f = c.ffn, V = c.vocab, L = c.L;
  for (int pad : {16, 32, 48, 64, 96, 128})  // batch tiles the bf16 kernels are compiled for
    if (st->B_pad < B) st->B_pad = pad;
  if (st->B_pad < B) st->B_pad = B;  // fp32 path only
  st->layers_tmp.resize(L);

  // ---- launch shapes (the weight layout below depends on them)
  auto ov = [&](const char *name, int &v, int lo, int hi) {  // whether there is an override, in range
    const int e = env_int(name, 0);
    if (e < lo || e > hi) return false;
    v = e;
    return true;
  };
  if (st->bf16) {
    const int Bp = st->B_pad;
    st->p_qkv = plan_direct(3 * d, Bp);
    st->p_ffn1 = plan_direct(f, Bp);
    st->p_head = plan_head(V, Bp);
    st->p_out = plan_split(d, d, Bp);
    st->p_ffn2 = plan_split(d, f, Bp);
    ov("SKD_R_QKV", st->p_qkv.R, 1, 4); ov("SKD_R_FFN1", st->p_ffn1.R, 1, 4);
    ov("SKD_R_OUT", st->p_out.R, 1, 4); ov("SKD_R_FFN2", st->p_ffn2.R, 1, 4);
    ov("SKD_S_OUT", st->p_out.split, 1, 32); ov("SKD_S_FFN2", st->p_ffn2.split, 1, 32);
    ov("SKD_U_QKV", st->p_qkv.U, 1, 4); ov("SKD_U_FFN1", st->p_ffn1.U, 1, 4);
    ov("SKD_U_OUT", st->p_out.U, 1, 4); ov("SKD_U_FFN2", st->p_ffn2.U, 1, 4);
    ov("SKD_W_QKV", st->p_qkv.waves, 4, 8); ov("SKD_W_FFN1", st->p_ffn1.waves, 4, 8);
    ov("SKD_W_OUT", st->p_out.waves, 4, 8); ov("SKD_W_FFN2", st->p_ffn2.waves, 4, 8);
    const bool head_r = ov("SKD_R_HEAD", st->p_head.R, 1, 4), head_u = ov("SKD_U_HEAD", st->p_head.U, 1, 4),
               head_w = ov("SKD_W_HEAD", st->p_head.waves, 4, 8);
    int parts = head_r || head_u || head_w ? 0 : plan_head_split(V, d);  // these are shapes of the whole K range
    ov("SKD_S_HEAD", parts, 1, LOGITS_SPLIT);
    if (parts > 1) {
      st->head_parts = true;
      st->p_head.R = 1;
      st->p_head.split = parts;
      st->p_head.U = Bp <= 16 ? 2 : 1;
    }
  }

  if (st->bf16) {
    st->max_split = std::max(st->p_out.split, st->p_ffn2.split);
    // The prologue reads x and the partial sums of every row in every workgroup, and bias, gain and offset once: up to
    // 128 KiB of the former (two rows of 4096 with a split of 2: 96, three of 2048 with 4: 120) that takes less than the
    // reducer's launch.  It is paid per workgroup, and the
    // activations come from LDS, so the projections behind it take the row groups of a wider batch: one workgroup per CU
    // instead of two for FFN1 at 4096 x 16384.  One row of 4096, 4 steps of 2 to 4 layers at 2000 keys: 1355 us with
    // separate reducers, 1300 with two workgroups per CU, 1287 with one; two rows of 256: 1910 -> 1740 us for 16 steps.
    st->fuse_ln = B <= 4 && d <= (B <= 2 ? 4096 : 2048) && (long)B * d * 4 * (1 + st->max_split) <= (128L << 10) &&
                  env_int("SKD_FUSE_LN", 1) != 0;
    if (st->fuse_ln) {
      st->p_qkv = plan_direct(3 * d, 32);
      st->p_ffn1 = plan_direct(f, 32);
      ov("SKD_R_QKV", st->p_qkv.R, 1, 4); ov("SKD_R_FFN1", st->p_ffn1.R, 1, 4);
      ov("SKD_U_QKV", st->p_qkv.U, 1, 4); ov("SKD_U_FFN1", st->p_ffn1.U, 1, 4);
      ov("SKD_W_QKV", st->p_qkv.waves, 4, 8); ov("SKD_W_FFN1", st->p_ffn1.waves, 4, 8);
    }
  }
  if (st->bf16 && st->B_pad >= 96 && env_int("SKD_GEMM_WS", 1) != 0) {
    // 96 and 128 batch rows: every projection whose K range divides into stages of 4 k-steps per workgroup
    GemmArgs ga{};
    ga.B = B; ga.B_pad = st->B_pad;
    auto pick = [&](int N, int K, GemmPlan &p, int epi) {
      ga.N = N; ga.K = K; ga.G = p.R; ga.split = p.split;
      if (epi == EPI_LOGITS) bf16_head_tiles(ga, p.R, 0);
      p.ws = bf16_gemm_ws_check(ga, epi, p.R) > 0;
      // rotated K start: pays while the XCD's L2 (4 MiB) holds the activation matrix beside the weight stream
      // (measured at 128 x 4096: FFN1 35.5 -> 33.7 us; at 128 x 16384, 4 MiB, FFN2 36.3 -> 38.8 us)
      // Not for the LM head: there every vocabulary row keeps the same summation order, so that identical rows give
      // identical logits at every batch size (ties are then broken by index, as documented), and it gains nothing.
      const bool head = &p == &st->p_head;
      p.ws_rot = !head && (long)st->B_pad * K * 2 <= (2L << 20);
      const int e = env_int("SKD_WS_ROT", -1);
      if (e == 0 || (e == 1 && !head)) p.ws_rot = e;
    };
    pick(3 * d, d, st->p_qkv, EPI_QKV); pick(d, d, st->p_out, EPI_PARTIAL); pick(f, d, st->p_ffn1, EPI_RELU);
    pick(d, f, st->p_ffn2, EPI_PARTIAL); pick(st->head_parts ? (V + 15) / 16 * 16 : V, d, st->p_head, st->head_parts ? EPI_PARTIAL : EPI_LOGITS);
  }
  if (st->bf16 && !decode_shapes_ok(st)) return fail(SKD_ERR_SHAPE);  // an override the kernels cannot launch
  {  // the device this state lives on, and that device's copy of the static scratch array
    hipError_t e = hipGetDevice(&st->device);
    if (e != hipSuccess) { g_last_hip = (int)e; return fail(SKD_ERR_HIP); }
    const int src = resolve_scratch(st->device);
    if (src != SKD_OK) return fail(src);
  }

  // ---- weights
  const size_t esz = w->elem == SKD_W_BF16 ? 2 : 4;
  size_t biggest = std::max({(size_t)V * d, (size_t)c.max_pos * d, (size_t)3 * d * d, (size_t)f * d});
  void *staging = nullptr;
  if (w->location == SKD_HOST) {
    hipError_t e = hipMalloc(&staging, biggest * esz);
    if (e != hipSuccess) { g_last_hip = (int)e; return fail(SKD_ERR_NOMEM); }
  }
  int rc = SKD_OK;
  auto vec = [&](const void *src, size_t n, float **o) { if (rc == SKD_OK) rc = upload_vec(st, *w, src, n, staging, o); };
  auto mat = [&](const void *src, long N, long K, int frag, void **o) { if (rc == SKD_OK) rc = upload_mat(st, *w, src, N, K, staging, frag, o); };
  mat(w->tok_emb, V, d, 0, &st->tok_emb);
  mat(w->pos_emb, c.max_pos, d, 0, &st->pos_emb);
  if (st->bf16 || w->lm_head) mat(w->lm_head ? w->lm_head : w->tok_emb, V, d, st->bf16 ? st->p_head.R : 1, &st->head);
  else st->head = st->tok_emb;
  vec(w->lnf_g, d, &st->lnf_g);
  vec(w->lnf_b, d, &st->lnf_b);
  st->lw.resize(L);
  for (int l = 0; l < L && rc == SKD_OK; ++l) {
    LayerW &lw = st->lw[l];
    vec(w->ln1_g[l], d, &lw.ln1_g); vec(w->ln1_b[l], d, &lw.ln1_b);
    mat(w->wqkv[l], 3L * d, d, st->p_qkv.R, &lw.wqkv); vec(w->bqkv[l], 3 * (size_t)d, &lw.bqkv);
    mat(w->wo[l], d, d, st->p_out.R, &lw.wo); vec(w->bo[l], d, &lw.bo);
    vec(w->ln2_g[l], d, &lw.ln2_g); vec(w->ln2_b[l], d, &lw.ln2_b);
    mat(w->w1[l], f, d, st->p_ffn1.R, &lw.w1); vec(w->b1[l], f, &lw.b1);
    mat(w->w2[l], d, f, st->p_ffn2.R, &lw.w2); vec(w->b2[l], d, &lw.b2);
  }
  if (staging) (void)hipFree(staging);
  if (rc != SKD_OK) return fail(rc);

  // ---- KV cache
  rc = build_kv(st);
  if (rc != SKD_OK) return fail(rc);

  // ---- workspaces
  const int Bp = st->B_pad;
  auto A = [&](auto **p, size_t n) { if (rc == SKD_OK) rc = dev_alloc(st, p, n); };
  A(&st->tok_dev, B); A(&st->prompt_dev, (size_t)c.prompt_size * B); A(&st->start_dev, B); A(&st->order_dev, B); A(&st->argmax_dev, B); A(&st->u_dev, B);
  if (const size_t parts = (size_t)B * sample_chunks(V)) {
    A(&st->sample.z, (size_t)B * SAMPLE_CHUNK_CAND); A(&st->sample.idx, (size_t)B * SAMPLE_CHUNK_CAND);
    A(&st->sample.max_mass, parts * 3); A(&st->sample.count, parts);
  }
  A(&st->x, (size_t)Bp * d);
  if (st->bf16) {
    st->prefill_mode = env_int("SKD_PREFILL_BATCHED", 1) != 0 ? 1 : 0;
    st->prefill_tiles = env_int("SKD_PREFILL_TILES", 1) != 0 ? 1 : 0;
    {  // "<weight rows>x<activation rows>x<split>": one tile for every prompt projection that it divides
      int wr = 0, ar = 0, sp = 1;
      const char *e = getenv("SKD_PREFILL_TILE");
      if (e && sscanf(e, "%dx%dx%d", &wr, &ar, &sp) == 3 && sp >= 1 && sp <= 16 &&
          (wr == 256 || wr == 128 || wr == 64) && (ar == 256 || ar == 128 || ar == 64) && wr * ar != 256 * 64) {
        st->prefill_wr = wr;
        st->prefill_ar = ar;
        st->prefill_split = sp;
      }
    }
    // split the key range of one head over several workgroups only when rows*heads alone cannot fill the chip
    // decode attention wants 16 waves on every CU: few (row, head) pairs get wider workgroups first (merged in
    // LDS), then splits of the key range (merged by a second kernel)
    // (one wave per pair streams 4 % faster with the arithmetic removed, but not with it: measured 128.7 vs 127.2 us
    // at 128 rows x 32 heads, so the planner starts at two; SKD_ATTN_WAVES=1 forces it)
    int waves = 2, splits = 1;
    while (B * c.n_heads * waves < 4096 && waves < 16) waves *= 2;
    while (B * c.n_heads * waves * splits < 4096 && splits < 8) splits *= 2;
    ov("SKD_ATTN_WAVES", waves, 1, 16);
    ov("SKD_ATTN_SPLITS", splits, 1, 16);
    st->attn_waves = waves;
    st->attn_splits = splits;
    st->attn_fixed = env_int("SKD_ATTN_WAVES", 0) > 0 || env_int("SKD_ATTN_SPLITS", 0) > 0;
    if (st->fuse_ln) A(&st->x2, (size_t)Bp * d);
    bf16_t *t16 = nullptr;
    A(&t16, (size_t)Bp * d); st->a = t16; if (rc == SKD_OK) rc = hipMemsetAsync(st->a, 0, (size_t)Bp * d * 2, st->stream) == hipSuccess ? SKD_OK : SKD_ERR_HIP;
    A(&t16, (size_t)Bp * d); st->q = t16;
    A(&t16, (size_t)Bp * d); st->o = t16; if (rc == SKD_OK) rc = hipMemsetAsync(st->o, 0, (size_t)Bp * d * 2, st->stream) == hipSuccess ? SKD_OK : SKD_ERR_HIP;
    A(&t16, (size_t)Bp * f); st->u = t16;
    A(&st->kv_new, (size_t)B * 2 * d);
    A(&st->partial, std::max((size_t)st->max_split * Bp * d, st->head_parts ? (size_t)st->p_head.split * Bp * ((V + 15) / 16 * 16) : 0));
    A(&st->attn_part, (size_t)st->attn_splits * B * c.n_heads * (st->dh + 4));
    GemmArgs ga{};
    ga.N = V;
    const int groups = std::max(bf16_head_tiles(ga, st->p_head.R, st->p_head.slots), bf16_gemm_groups(V, st->p_head.R));
    A(&st->pmax, (size_t)groups * Bp); A(&st->pidx, (size_t)groups * Bp);
    A(&st->logits_dev, (size_t)B * V);
  } else {
    float *t32 = nullptr;
    A(&t32, (size_t)B * d); st->a = t32;
    A(&t32, (size_t)B * 3 * d); st->q = t32;
    A(&t32, (size_t)B * d); st->o = t32;
    A(&t32, (size_t)B * f); st->u = t32;
    A(&st->attn_part, (size_t)B * c.n_heads * c.sequence_length);
    A(&st->logits_dev, (size_t)B * V);
  }
  if (rc == SKD_OK && st->bf16 && bf16_team_ok(d, f, B) && env_int("SKD_TEAM", 1) != 0 && !launch_overrides()) rc = prepare_team(st);
  if (rc != SKD_OK) return fail(rc);
  if (st->bf16 && !c.io_on_device) {
    const hipError_t e = hipHostMalloc((void **)&st->pin, sizeof(Pinned), hipHostMallocDefault);
    if (e != hipSuccess) { g_last_hip = (int)e; st->pin = nullptr; return fail(SKD_ERR_NOMEM); }
  }
  if (hipStreamSynchronize(st->stream) != hipSuccess) return fail(SKD_ERR_HIP);
  *out = st;
  return SKD_OK;
}

extern "C" int skd_create(const skd_config *cfg, const skd_weights *w, void *hip_stream, skd_state **out) {
  return create_impl(cfg, w, hip_stream, nullptr, out);
}

extern "C" int skd_create_with_schedule(const skd_config *cfg, const skd_weights *w, void *hip_stream,
                                        const int32_t *n_table, skd_state **out) {
  if (!n_table) return SKD_ERR_NULL;
  return create_impl(cfg, w, hip_stream, n_table, out);
}

extern "C" int skd_state_active_layers(const skd_state *st, int32_t t, int32_t *layers_out) {
  if (!st || !layers_out) return SKD_ERR_NULL;
  return state_active_layers(st, t, layers_out);
}

extern "C" void skd_destroy(skd_state *st) {
  if (!st) return;
  (void)hipStreamSynchronize(st->stream);
  for (auto &r : st->prof_pending) { if (r.a) (void)hipEventDestroy(r.a); if (r.b) (void)hipEventDestroy(r.b); }
  for (hipEvent_t e : st->prof_free) (void)hipEventDestroy(e);
  for (void *p : st->allocs) (void)hipFree(p);
  if (st->pin) (void)hipHostFree(st->pin);
  if (st->team_gave_up.word) (void)hipHostFree((void *)st->team_gave_up.word);
  delete st;
}

// where a state's one-launch columns report a wait that ran out (null: it has none)
namespace skd {
volatile uint32_t *team_gave_up(const skd_state *st) { return st->team_gave_up.word; }
}
// SKD_ERR_HIP once a column's kernel had to go on without a workgroup that it waited for: caches, hidden rows and tokens
// behind it are not to be used.
static int intact(const skd_state *st) {
  if (!GaveUp{team_gave_up(st)}.seen()) return SKD_OK;
  g_last_hip = (int)hipErrorLaunchTimeOut;
  return SKD_ERR_HIP;
}
static int wait_stream(skd_state *st) {
  HIPCHECK(hipStreamSynchronize(st->stream));
  return intact(st);
}

// per-row padding offsets and the dispatch order of the attention workgroups (longest rows first)
static void set_start(skd_state *st, const std::vector<int32_t> &start) {
  const int B = st->cfg.batch;
  st->order_host.resize(B);
  for (int b = 0; b < B; ++b) st->order_host[b] = b;
  std::stable_sort(st->order_host.begin(), st->order_host.end(), [&](int x, int y) { return start[x] < start[y]; });
  st->start_min = *std::min_element(start.begin(), start.end());
  st->ragged = *std::max_element(start.begin(), start.end()) != st->start_min;
  st->start_host = start;
}
static int upload_start(skd_state *st) {
  const int B = st->cfg.batch;
  HIPCHECK(hipMemcpyAsync(st->start_dev, st->start_host.data(), B * sizeof(int32_t), hipMemcpyHostToDevice, st->stream));
  HIPCHECK(hipMemcpyAsync(st->order_dev, st->order_host.data(), B * sizeof(int32_t), hipMemcpyHostToDevice, st->stream));
  HIPCHECK(hipStreamSynchronize(st->stream));
  return SKD_OK;
}

// Kernel and launch shape of a prompt projection (N outputs, `rows` activation rows in whole 16-row tiles).
struct RowsGemm {
  enum Kind { SKINNY, MID, TILE, CHUNKS } kind = CHUNKS;
  int B_pad = 128;      // SKINNY: padded rows, R and split as in a decode projection of that batch
  int R = 4, split = 1; // split > 1, or SKINNY with split_ok: partial sums, added by the row reducer
  int wr = 128, ar = 128;  // MID: tile
  bool partial = false;
};
constexpr long kRowsPartialMax = 32L << 20;  // fp32 partial sums of one projection (128 MiB)

// Up to 64 rows a projection is a weight stream, as in decode: 6.7B shape, 64 rows, us on the 256 x 256 tiles / on
// the decode kernel: QKV 80 / 23, output 87 / 9.9, FFN1 80 / 26, FFN2 292 / 27.
// Beyond, the tile and the K split with the least estimated time.  The estimate is (k-steps of a workgroup) x (time of
// a k-step with the number of workgroups a CU then holds), summed over the rounds of workgroups, plus the traffic of
// the partial sums.  Step times measured at the 6.7B and 1.3B shapes, 64 to 4096 rows (us): 256 x 256 0.57 (few
// workgroups) to 0.75 (all CUs: the clock drops); 256 x 128 and 128 x 256 0.45 to 0.51; 128 x 128 0.32 alone on a CU,
// 0.52 for two; 64 x 128 0.255 / 0.44; 64 x 64 0.19 / 0.33 / 0.44 / 0.55 for one to four.  So the small tiles win only while the chip is not full:
// at 1024 rows of the 6.7B shape FFN1 takes 100 us on 256 x 256 and 138 on 128 x 128, at 256 rows 80 and 44.
// The epilogue is not in the estimate, and the traffic of the partial sums counts the reducer's reads: at 912 rows of the
// 1.3B shape estimate and launch are 34 / 39 us (QKV), 23.5 / 30 (k | v alone), 35 / 36 (FFN1) and 45 / 37 (FFN2, split 4).
// For that reason the 8-wave tiles keep these step times although their two waves of a SIMD take turns now.  256 x 128 and
// 128 x 256: a step takes 0.325 (64 workgroups) to 0.44 (256); with those times prompts of 1200 to 2000 rows of the 6.7B
// shape were 1 to 3 % faster, but 360 and from 800 rows on of the 1.3B shape 2 to 5 % slower.  256 x 256: 0.47 to 0.72;
// with those, us (these -> those): 1.3B, four layers, 672 rows 526 -> 531, 4320 rows (FFN2 without its split of 3) 1667 ->
// 1702, 4800 and 5120 rows alike; (512, ffn 1536), 8640 rows 438 -> 460; 6.7B, two layers, 144 rows 377 -> 383, 672 rows 509
// -> 507.  And another split is another order of the sums.
RowsGemm plan_rows(int N, int K, int rows, bool split_ok) {
  RowsGemm best;
  const int Kf = K / 32;
  if (rows <= 64) {
    best.kind = RowsGemm::SKINNY;
    best.B_pad = rows <= 16 ? 16 : rows <= 32 ? 32 : rows <= 48 ? 48 : 64;
    const GemmPlan p = split_ok ? plan_split(N, K, best.B_pad) : plan_direct(N, best.B_pad);
    best.R = p.R;
    best.split = p.split;
    best.partial = split_ok;
    return best;
  }
  // tile, workgroups a CU holds, step time by workgroups on the CU, what a full chip adds
  static const struct { int wr, ar, cap; double step[4], full; } cfg[] = {
      {256, 256, 1, {0.57}, 0.18}, {256, 128, 1, {0.455}, 0.06}, {128, 256, 1, {0.45}, 0.05}, {128, 128, 2, {0.32, 0.52}, 0.0},
      {64, 128, 2, {0.255, 0.44}, 0.0}, {128, 64, 2, {0.255, 0.44}, 0.0}, {64, 64, 4, {0.19, 0.33, 0.44, 0.55}, 0.0}};
  static const int splits[] = {1, 2, 3, 4, 6, 8, 12, 16};
  double best_t = 1e30;
  for (const auto &c : cfg) {
    if (N % c.wr) continue;
    const long tiles = (long)(N / c.wr) * ((rows + c.ar - 1) / c.ar);
    for (int sp : splits) {
      if (sp > 1 && (!split_ok || Kf / sp < 8 || (long)sp * (rows + 255) * N > kRowsPartialMax)) break;
      const long wgs = tiles * sp, slots = 256L * c.cap, full = wgs / slots, rem = wgs % slots;
      const double clock = c.full * std::min(1.0, wgs / 256.0);
      double step = full * (c.step[c.cap - 1] + clock);
      if (rem) step += c.step[(rem + 255) / 256 - 1] + clock;
      const double t = 3.0 + (double)((Kf + sp - 1) / sp) * step + (sp > 1 ? (sp - 1) * 8.0 * rows * N / 4.5e6 : 0.0);
      if (t < best_t) {
        best_t = t;
        best.kind = c.wr == 256 && c.ar == 256 ? RowsGemm::TILE : RowsGemm::MID;
        best.wr = c.wr;
        best.ar = c.ar;
        best.split = sp;
        best.partial = sp > 1;
      }
    }
  }
  return best;  // CHUNKS when no tile divides N
}

// Whole prompt at once, layer by layer (Section 2.3: the prompt needs no generation, so it can be batched over
// positions): activation rows are the real (sequence, position) pairs (left padding gets no rows), attention is
// causal over the pages the QKV projection has just filled.  A row depends on rows of its own sequence before it
// only, so what padding rows hold never matters.
static int prefill_batched(skd_state *st, const int32_t *cols) {
  const skd_config &c = st->cfg;
  const int B = c.batch, P = c.prompt_size, d = c.d_model, f = c.ffn, L = c.L;
  const int P_pad = (P + 15) / 16 * 16;
  const long cap = ((long)B * P_pad + 255) / 256 * 256;  // workspace rows: every position of every sequence
  hipStream_t s = st->stream;
  if (!st->pf_x) {
    auto rows_alloc = [&](auto **p, size_t n) -> int {
      SKDCHECK(dev_alloc(st, p, n));
      HIPCHECK(hipMemsetAsync(*p, 0, n * sizeof(**p), s));  // once: padding rows are read by the projections
      return SKD_OK;
    };
    SKDCHECK(rows_alloc(&st->pf_a, (size_t)cap * d));
    SKDCHECK(rows_alloc(&st->pf_q, (size_t)cap * d));
    SKDCHECK(rows_alloc(&st->pf_o, (size_t)cap * d));
    SKDCHECK(rows_alloc(&st->pf_u, (size_t)cap * f));
    SKDCHECK(dev_alloc(st, &st->pf_partial, (size_t)std::min(kRowsPartialMax, 16 * cap * d)));
    SKDCHECK(dev_alloc(st, &st->pf_seq, (size_t)cap));
    SKDCHECK(dev_alloc(st, &st->pf_tiles, (size_t)cap / 16));
    SKDCHECK(dev_alloc(st, &st->pf_first, (size_t)B));
    SKDCHECK(rows_alloc(&st->pf_x, (size_t)cap * d));
  }
  // only real tokens get rows: sequence b owns its P - start[b] positions, padded to whole 16-row tiles
  PromptMap pm{};
  int rows = 0, max_len = 0;
  for (int b = 0; b < B; ++b) {
    max_len = std::max(max_len, P - st->start_host[b]);
    pm.start[b] = st->start_host[b];
    pm.first[b] = rows;
    pm.order[b] = (uint8_t)st->order_host[b];
    rows += (P - st->start_host[b] + 15) / 16 * 16;
  }
  const int rows_pad = (rows + 255) / 256 * 256;
  bf16_prompt_map(s, pm, B, rows, rows_pad, P, st->geom, st->start_dev, st->order_dev, st->pf_first, st->pf_seq, st->pf_tiles);
  RowMap rm{st->pf_seq, st->pf_first, st->start_dev, P};
  bf16_embed_ln_rows(s, cols, rm, rows, (const bf16_t *)st->tok_emb, (const bf16_t *)st->pos_emb, st->lw[0].ln1_g,
                     st->lw[0].ln1_b, st->pf_x, st->pf_a, B, d, c.vocab);
  auto plan = [&](int N, int K, bool split_ok) {
    RowsGemm p;
    if (st->prefill_tiles && !st->prefill_wr) return plan_rows(N, K, rows, split_ok);
    if (st->prefill_tiles && N % st->prefill_wr == 0) {  // forced tile
      p.kind = st->prefill_wr == 256 && st->prefill_ar == 256 ? RowsGemm::TILE : RowsGemm::MID;
      p.wr = st->prefill_wr;
      p.ar = st->prefill_ar;
      p.split = split_ok ? std::min(st->prefill_split, K / 32) : 1;
      if ((long)p.split * rows_pad * N > kRowsPartialMax) p.split = 1;
      p.partial = p.split > 1;
    }
    return p;
  };
  const RowsGemm r_qkv = plan(3 * d, d, false), r_out = plan(d, d, true), r_ffn1 = plan(f, d, false), r_ffn2 = plan(d, f, true);
  auto stride = [&](const RowsGemm &p) { return p.kind == RowsGemm::SKINNY ? p.B_pad : rows_pad; };  // of the partial sums
  auto proj = [&](GemmArgs g, int epi, const RowsGemm &p) {
    if (p.partial) epi = EPI_PARTIAL;
    g.split = p.split;
    g.B_pad = stride(p);
    g.rows = rows;
    if (p.kind == RowsGemm::TILE) return bf16_gemm_tile(s, g, epi);
    if (p.kind == RowsGemm::MID) return bf16_gemm_mid(s, g, epi, p.wr, p.ar);
    if (p.kind == RowsGemm::SKINNY) {
      g.rows = p.B_pad;
      return bf16_gemm(s, g, epi, p.R, 1, 8);
    }
    g.B_pad = 128;  // 128-row chunks through the skinny kernel
    g.rows = (rows + 127) / 128 * 128;
    return bf16_gemm(s, g, epi, g.N % 64 ? 1 : 4, 1, 4);
  };
  // What leaves the prompt pass is the cache of every layer and the hidden state of each sequence's last position, so
  // of the top layer's rows only the last positions are needed beyond their keys and values: its q | k | v projection
  // computes k | v for all rows, and the last positions go through that layer as a decode column at position P - 1.
  // From 512 rows on: at 912 rows of the 1.3B shape 165 us against 70, at 16384 of the 6.7B shape 5200 against 950.  Below,
  // a layer of all rows costs little more than streaming its weights, which the column streams too; at 256 rows of the
  // 6.7B shape the column was estimated at 130 us against 165, so the line lies on the safe side of where the two cross,
  // which has not been measured.
  const RowsGemm r_kv = plan(2 * d, d, false);
  const bool last_as_column = rows >= 512 && (r_kv.kind == RowsGemm::TILE || r_kv.kind == RowsGemm::MID);
  for (int l = 0; l < L; ++l) {
    const LayerW &w = st->lw[l];
    GemmArgs ga{};
    ga.B = B; ga.rm = rm; ga.cache_tiles = st->pf_tiles; ga.kv = st->geom; ga.d = d; ga.partial = st->pf_partial; ga.x = st->pf_x;
    ga.W = (const bf16_t *)w.wqkv; ga.G = st->p_qkv.R; ga.A = st->pf_a; ga.bias = w.bqkv; ga.N = 3 * d; ga.K = d;
    ga.q_out = st->pf_q; ga.kv_pool = (bf16_t *)st->pool; ga.bt_layer = bt_layer(st, l);
    if (l == L - 1 && last_as_column) {
      ga.t0 = d / 16;
      ga.N = 2 * d;
      if (proj(ga, EPI_QKV_ROWS, r_kv) < 0) return SKD_ERR_SHAPE;
      bf16_last_rows_ln(s, st->pf_x, rm, nullptr, 0, 0, nullptr, w.ln1_g, w.ln1_b, st->x, (bf16_t *)st->a, B, d);
      const int profiling = st->profiling;
      st->profiling = 0;  // the timed classes are those of decode steps
      const int rc = run_layer(st, l, P - 1, nullptr, nullptr);
      st->profiling = profiling;
      SKDCHECK(rc);
      st->kv_len[l] = P;
      break;
    }
    if (proj(ga, EPI_QKV_ROWS, r_qkv) < 0) return SKD_ERR_SHAPE;
    AttnRowsArgs aa{};
    aa.q = st->pf_q; aa.pool = (const bf16_t *)st->pool; aa.bt_layer = bt_layer(st, l); aa.rm = rm;
    aa.B = B; aa.max_len = max_len; aa.kv = st->geom; aa.o = st->pf_o;
    bf16_attention_rows(s, aa);
    ga.W = (const bf16_t *)w.wo; ga.G = st->p_out.R; ga.A = st->pf_o; ga.bias = w.bo; ga.N = d; ga.K = d;
    if (proj(ga, EPI_RESID, r_out) < 0) return SKD_ERR_SHAPE;
    if (r_out.partial) bf16_reduce_ln(s, st->pf_partial, r_out.split, stride(r_out), w.bo, st->pf_x, st->pf_x, w.ln2_g, w.ln2_b, st->pf_a, rows, d);
    else bf16_ln_rows(s, st->pf_x, w.ln2_g, w.ln2_b, st->pf_a, rows, d);
    ga.W = (const bf16_t *)w.w1; ga.G = st->p_ffn1.R; ga.A = st->pf_a; ga.bias = w.b1; ga.N = f; ga.K = d; ga.act_out = st->pf_u;
    if (proj(ga, EPI_RELU, r_ffn1) < 0) return SKD_ERR_SHAPE;
    ga.W = (const bf16_t *)w.w2; ga.G = st->p_ffn2.R; ga.A = st->pf_u; ga.bias = w.b2; ga.N = d; ga.K = f;
    if (proj(ga, EPI_RESID, r_ffn2) < 0) return SKD_ERR_SHAPE;
    if (l + 1 < L) {
      const LayerW &nw = st->lw[l + 1];
      if (r_ffn2.partial) bf16_reduce_ln(s, st->pf_partial, r_ffn2.split, stride(r_ffn2), w.b2, st->pf_x, st->pf_x, nw.ln1_g, nw.ln1_b, st->pf_a, rows, d);
      else bf16_ln_rows(s, st->pf_x, nw.ln1_g, nw.ln1_b, st->pf_a, rows, d);
    }
    st->kv_len[l] = P;
  }
  // hidden state of the last prompt column, and its final LayerNorm, where the heads expect them
  if (!last_as_column)
    bf16_last_rows_ln(s, st->pf_x, rm, st->pf_partial, r_ffn2.partial ? r_ffn2.split : 0, stride(r_ffn2), st->lw[L - 1].b2,
                      st->lnf_g, st->lnf_b, st->x, (bf16_t *)st->a, B, d);
  HIPCHECK(hipGetLastError());
  st->have_hidden = true;
  st->have_argmax = false;
  return SKD_OK;
}

extern "C" int skd_prefill(skd_state *st, const int32_t *tokens, const uint8_t *attn_mask) {
  if (!st || !tokens) return SKD_ERR_NULL;
  SKDCHECK(intact(st));
  const skd_config &c = st->cfg;
  const int B = c.batch, P = c.prompt_size;
  std::vector<int32_t> start(B, 0);
  if (attn_mask) {
    for (int b = 0; b < B; ++b) {
      int j = 0;
      while (j < P && attn_mask[(size_t)b * P + j] == 0) ++j;
      if (j == P) return SKD_ERR_SHAPE;  // a row needs at least one real token
      start[b] = j;
      for (; j < P; ++j)
        if (attn_mask[(size_t)b * P + j] == 0) return SKD_ERR_SHAPE;  // only left padding
    }
  }
  const int32_t *cols = nullptr;
  if (c.io_on_device) {
    cols = tokens;
  } else {
    std::vector<int32_t> tr((size_t)P * B);
    for (int b = 0; b < B; ++b)
      for (int j = 0; j < P; ++j) {
        const int32_t tok = tokens[(size_t)b * P + j];
        if (tok < 0 || tok >= c.vocab) return SKD_ERR_RANGE;
        tr[(size_t)j * B + b] = tok;
      }
    HIPCHECK(hipMemcpyAsync(st->prompt_dev, tr.data(), tr.size() * sizeof(int32_t), hipMemcpyHostToDevice, st->stream));
    HIPCHECK(hipStreamSynchronize(st->stream));
    cols = st->prompt_dev;
  }
  set_start(st, start);
  std::fill(st->kv_len.begin(), st->kv_len.end(), 0);
  st->prefilled = false;
  st->steps_done = 0;
  bool full_depth_prompt = true;  // a caller's table may decay inside the prompt: then columns differ in depth
  for (int i = 0; i < P && full_depth_prompt; ++i)
    if (!st->n_table.empty() && st->n_table[i] != c.L) full_depth_prompt = false;
  if (st->bf16 && st->prefill_mode == 1 && full_depth_prompt) {
    SKDCHECK(prefill_batched(st, cols));
  } else {
    SKDCHECK(upload_start(st));
    for (int i = 0; i < P; ++i) {  // column by column
      const int n = state_active_layers(st, i, st->layers_tmp.data());
      if (n < 0) return n;
      SKDCHECK(run_column(st, i, cols + (size_t)i * B, st->layers_tmp.data(), n));
    }
  }
  st->prefilled = true;
  return c.io_on_device ? SKD_OK : wait_stream(st);
}

extern "C" int skd_decode_step(skd_state *st, int32_t t, const int32_t *tokens_in) {
  if (!st) return SKD_ERR_NULL;
  const skd_config &c = st->cfg;
  if (!st->prefilled) return SKD_ERR_ORDER;
  if (t < 0 || t >= c.sequence_length) return SKD_ERR_RANGE;
  if (t != c.prompt_size + st->steps_done) return SKD_ERR_ORDER;
  SKDCHECK(intact(st));
  const int32_t *tok = nullptr;
  if (!tokens_in) {
    if (!st->have_argmax) return SKD_ERR_ORDER;
    tok = st->argmax_dev;
  } else if (c.io_on_device) {
    tok = tokens_in;
  } else {
    for (int b = 0; b < c.batch; ++b)
      if (tokens_in[b] < 0 || tokens_in[b] >= c.vocab) return SKD_ERR_RANGE;
    if (st->pin) {
      std::copy(tokens_in, tokens_in + c.batch, st->pin->tok_in);
      tok = st->pin->tok_in;
    } else {
      HIPCHECK(hipMemcpyAsync(st->tok_dev, tokens_in, c.batch * sizeof(int32_t), hipMemcpyHostToDevice, st->stream));
      HIPCHECK(hipStreamSynchronize(st->stream));
      tok = st->tok_dev;
    }
  }
  const int n = state_active_layers(st, t, st->layers_tmp.data());
  if (n < 0) return n;
  SKDCHECK(run_column(st, t, tok, st->layers_tmp.data(), n));
  st->steps_done += 1;
  return c.io_on_device ? SKD_OK : wait_stream(st);
}

// The two launches of an LM head whose K range is split (plan_head_split): partial sums in the state's own buffer, which the
// layers use before it and nothing reads behind it; then their sum, to logits (optional) and greedy tokens (optional; tokens2:
// second destination, or null).  head_parts_gemm < 0: not launched.
static int head_parts_gemm(skd_state *st) {
  GemmArgs ga{};
  ga.B = st->cfg.batch; ga.B_pad = st->B_pad; ga.W = (const bf16_t *)st->head; ga.G = st->p_head.R; ga.A = (const bf16_t *)st->a;
  ga.N = (st->cfg.vocab + 15) / 16 * 16; ga.K = st->cfg.d_model; ga.split = st->p_head.split; ga.partial = st->partial;
  return launch_gemm(st->stream, ga, EPI_PARTIAL, st->p_head);
}
static void head_parts_sum(skd_state *st, float *logits, int32_t *tokens, int32_t *tokens2) {
  bf16_logits_sum(st->stream, st->partial, st->p_head.split, st->B_pad, (st->cfg.vocab + 15) / 16 * 16, st->cfg.vocab, logits, tokens,
                  tokens2, st->cfg.batch);
}

// Final LayerNorm + LM head (+ greedy argmax into argmax_dev).  logits_target: device buffer [B][V] or null.
// final LayerNorm output -> logits (optional) and, unless the caller picks the token itself, the greedy token
// tokens_target: second destination of the greedy token (device memory), or null
static int head_logits(skd_state *st, float *logits_target, bool want_argmax, int32_t *tokens_target) {
  const skd_config &c = st->cfg;
  const int B = c.batch, d = c.d_model, V = c.vocab;
  hipStream_t s = st->stream;
  if (!st->bf16) {
    float *lg = logits_target ? logits_target : st->logits_dev;
    { ProfScope ps_(st, SKD_PROF_OTHER); f32_layernorm(s, st->x, st->lnf_g, st->lnf_b, (float *)st->a, B, d); }
    { ProfScope ps_(st, SKD_PROF_OTHER); f32_linear(s, (const float *)st->head, nullptr, (const float *)st->a, lg, B, d, V, 0, 0); }
    if (want_argmax) { ProfScope ps_(st, SKD_PROF_OTHER); f32_argmax(s, lg, st->argmax_dev, B, V); }
  } else {
    if (st->head_parts) {
      { ProfScope ps_(st, SKD_PROF_LM_HEAD); if (head_parts_gemm(st) < 0) return SKD_ERR_SHAPE; }
      { ProfScope ps_(st, SKD_PROF_ARGMAX); head_parts_sum(st, logits_target, want_argmax ? st->argmax_dev : nullptr, want_argmax ? tokens_target : nullptr); }
      HIPCHECK(hipGetLastError());
      return SKD_OK;
    }
    GemmArgs ga{};
    ga.B = B; ga.B_pad = st->B_pad; ga.W = (const bf16_t *)st->head; ga.G = st->p_head.R; ga.A = (const bf16_t *)st->a;  // a = final LayerNorm output
    ga.N = V; ga.K = d; ga.split = 1; ga.logits = logits_target; ga.pmax = st->pmax; ga.pidx = st->pidx;
    int groups = bf16_head_tiles(ga, st->p_head.R, st->p_head.slots);
    { ProfScope ps_(st, SKD_PROF_LM_HEAD); groups = launch_gemm(s, ga, EPI_LOGITS, st->p_head); }
    if (groups < 0) return SKD_ERR_SHAPE;
    if (want_argmax) { ProfScope ps_(st, SKD_PROF_ARGMAX); bf16_argmax_final(s, st->pmax, st->pidx, groups, st->B_pad, st->argmax_dev, tokens_target, B); }
  }
  HIPCHECK(hipGetLastError());
  return SKD_OK;
}

// Whether logits go through the pinned buffer.  The argmax head's kernels write them there themselves (nothing on the device
// reads them again): the copy behind them took 2 us of a step of 61 with 1 or 2 rows of 1000, 7 to 10 of 70 to 100 with 8
// to 128.  us a call of the head, copied -> written there: one row of 50272 x 4096 100 -> 86, five (981 KiB) 133 -> 119, 128
// rows of 2000 x 256 (1000 KiB) 70 -> 65.  Larger ones, and those that the sampler reads, are written to device memory and
// copied.
static bool pin_logits(const skd_state *st) {
  return st->pin && (size_t)st->cfg.batch * st->cfg.vocab * sizeof(float) <= kPinnedLogits;
}

// Host buffers: waits for the head and hands its results over.  direct: the logits are in the pinned buffer already.
static int head_results(skd_state *st, int32_t *tokens_out, float *logits_out, bool direct) {
  const skd_config &c = st->cfg;
  const size_t n = (size_t)c.batch * c.vocab;
  hipStream_t s = st->stream;
  const bool pinned = pin_logits(st);
  if (tokens_out && !st->pin)
    HIPCHECK(hipMemcpyAsync(tokens_out, st->argmax_dev, c.batch * sizeof(int32_t), hipMemcpyDeviceToHost, s));
  if (logits_out && !direct)
    HIPCHECK(hipMemcpyAsync(pinned ? st->pin->logits : logits_out, st->logits_dev, n * sizeof(float), hipMemcpyDeviceToHost, s));
  SKDCHECK(wait_stream(st));
  if (tokens_out && st->pin) std::copy(st->pin->tok_out, st->pin->tok_out + c.batch, tokens_out);
  if (logits_out && pinned) std::copy(st->pin->logits, st->pin->logits + n, logits_out);
  return SKD_OK;
}

extern "C" int skd_logits_argmax(skd_state *st, int32_t *tokens_out, float *logits_out) {
  if (!st) return SKD_ERR_NULL;
  if (!st->have_hidden) return SKD_ERR_ORDER;
  SKDCHECK(intact(st));
  const skd_config &c = st->cfg;
  const int B = c.batch;
  hipStream_t s = st->stream;
  float *logits_target = nullptr;  // where the kernels write logits, if anywhere
  const bool direct = logits_out && pin_logits(st);  // the LM head writes them where the host reads them
  if (logits_out) logits_target = c.io_on_device ? logits_out : direct ? st->pin->logits : st->logits_dev;
  SKDCHECK(head_logits(st, logits_target, true, c.io_on_device ? tokens_out : st->pin ? st->pin->tok_out : nullptr));
  st->have_argmax = true;
  if (c.io_on_device) {
    if (tokens_out && !st->bf16)  // the bf16 path has written it
      HIPCHECK(hipMemcpyAsync(tokens_out, st->argmax_dev, B * sizeof(int32_t), hipMemcpyDeviceToDevice, s));
    return SKD_OK;
  }
  return head_results(st, tokens_out, logits_out, direct);
}

// skd_logits_argmax for callers that cannot allocate: same kernels, with the LM head's per-workgroup partials in
// the static device array instead of the buffers skd_create reserved (a head whose K range is split has none: its partial
// sums go to the state's own buffer, and it needs no static array).  No hipMalloc / hipFree, no event creation, whatever the
// profiling mode, no host-side staging: outputs are device memory and the call only enqueues work on the state's stream.
extern "C" int skd_logits_argmax_noalloc(skd_state *st, int32_t *tokens_out, float *logits_out) {
  if (!st) return SKD_ERR_NULL;
  if (!st->have_hidden) return SKD_ERR_ORDER;
  const skd_config &c = st->cfg;
  if (!st->bf16 || !c.io_on_device) return SKD_ERR_SHAPE;
  SKDCHECK(intact(st));
  if (st->head_parts) {
    if (head_parts_gemm(st) < 0) return SKD_ERR_SHAPE;
    head_parts_sum(st, logits_out, st->argmax_dev, tokens_out);
    HIPCHECK(hipGetLastError());
    st->have_argmax = true;
    return SKD_OK;
  }
  GemmArgs ga{};
  ga.N = c.vocab;
  int groups = bf16_head_tiles(ga, st->p_head.R, st->p_head.slots);
  if ((int64_t)groups * st->B_pad > SKD_NOALLOC_MAX_PARTIALS) groups = bf16_head_tiles(ga, st->p_head.R, 0);  // fewer, equal ones
  if ((int64_t)groups * st->B_pad > SKD_NOALLOC_MAX_PARTIALS) return SKD_ERR_RANGE;  // beyond the static scratch
  void *base = (st->device >= 0 && st->device < kMaxDevices) ? g_scratch_ptr[st->device] : nullptr;
  if (!base) return SKD_ERR_ORDER;  // resolved by skd_create on the state's device
  float *pmax = (float *)base;
  int32_t *pidx = (int32_t *)((unsigned char *)base + 4 * (size_t)SKD_NOALLOC_MAX_PARTIALS);
  hipStream_t s = st->stream;
  ga.B = c.batch; ga.B_pad = st->B_pad; ga.W = (const bf16_t *)st->head; ga.G = st->p_head.R; ga.A = (const bf16_t *)st->a;
  ga.K = c.d_model; ga.split = 1; ga.logits = logits_out; ga.pmax = pmax; ga.pidx = pidx;
  if (check_gemm(ga, EPI_LOGITS, st->p_head) != groups) return SKD_ERR_SHAPE;
  // every partial the final reduction reads is written by the projection of this same call: nothing to clear
  (void)launch_gemm(s, ga, EPI_LOGITS, st->p_head);
  bf16_argmax_final(s, pmax, pidx, groups, st->B_pad, st->argmax_dev, tokens_out, c.batch);
  HIPCHECK(hipGetLastError());
  st->have_argmax = true;
  return SKD_OK;
}

extern "C" int skd_logits_sample(skd_state *st, const float *u, float temperature, float top_p, int32_t *tokens_out,
                                 float *logits_out) {
  if (!st || !u) return SKD_ERR_NULL;
  if (!st->have_hidden) return SKD_ERR_ORDER;
  if (!(temperature > 0.f) || !(top_p > 0.f) || top_p > 1.f) return SKD_ERR_RANGE;
  const skd_config &c = st->cfg;
  const int B = c.batch, V = c.vocab;
  if (V > 65536) return SKD_ERR_SHAPE;
  SKDCHECK(intact(st));
  hipStream_t s = st->stream;
  const float *u_dev = u;
  if (!c.io_on_device) {
    for (int b = 0; b < B; ++b)
      if (!(u[b] >= 0.f) || u[b] >= 1.f) return SKD_ERR_RANGE;
    if (st->pin) {
      std::copy(u, u + B, st->pin->u_in);
      u_dev = st->pin->u_in;
    } else {
      HIPCHECK(hipMemcpyAsync(st->u_dev, u, B * sizeof(float), hipMemcpyHostToDevice, s));
      HIPCHECK(hipStreamSynchronize(s));
      u_dev = st->u_dev;
    }
  }
  float *lg = (logits_out && c.io_on_device) ? logits_out : st->logits_dev;
  SKDCHECK(head_logits(st, lg, false, nullptr));
  { ProfScope ps_(st, SKD_PROF_ARGMAX); if (sample_top_p(s, lg, B, V, temperature, top_p, u_dev, st->argmax_dev, c.io_on_device ? tokens_out : st->pin ? st->pin->tok_out : nullptr, st->sample) < 0) return SKD_ERR_SHAPE; }
  HIPCHECK(hipGetLastError());
  st->have_argmax = true;  // skd_decode_step(.., NULL) continues from the sampled tokens
  if (c.io_on_device) return SKD_OK;  // the sampler has written tokens_out
  return head_results(st, tokens_out, logits_out, false);
}

extern "C" int skd_rewind(skd_state *st, int32_t t) {
  if (!st) return SKD_ERR_NULL;
  if (!st->prefilled) return SKD_ERR_ORDER;
  const skd_config &c = st->cfg;
  if (t < c.prompt_size || t > c.prompt_size + st->steps_done) return SKD_ERR_RANGE;
  for (int l = 0; l < c.L; ++l) st->kv_len[l] = std::min(st->kv_len[l], (int)t);
  st->steps_done = t - c.prompt_size;
  st->have_hidden = false;  // the residual stream on the device belongs to a later column
  st->have_argmax = false;
  return SKD_OK;
}

extern "C" int skd_profile_enable(skd_state *st, int32_t on) {
  if (!st) return SKD_ERR_NULL;
  if (on < 0 || on > 2) return SKD_ERR_RANGE;
  SKDCHECK(prof_drain(st));
  st->profiling = on;
  return SKD_OK;
}

extern "C" int skd_profile_read(skd_state *st, double *ms, int64_t *launches) {
  if (!st) return SKD_ERR_NULL;
  SKDCHECK(prof_drain(st));
  for (int i = 0; i < SKD_PROF_CLASSES; ++i) {
    if (ms) ms[i] = st->prof_ms[i];
    if (launches) launches[i] = st->prof_n[i];
    st->prof_ms[i] = 0;
    st->prof_n[i] = 0;
  }
  return SKD_OK;
}

extern "C" int skd_kv_len(const skd_state *st, int32_t layer) {
  if (!st) return SKD_ERR_NULL;
  if (layer < 0 || layer >= st->cfg.L) return SKD_ERR_RANGE;
  return st->kv_len[layer];
}
extern "C" int64_t skd_kv_pages_reserved(const skd_state *st) { return st ? st->pages_reserved : SKD_ERR_NULL; }
extern "C" int64_t skd_kv_pages_dense(const skd_state *st) { return st ? st->pages_dense : SKD_ERR_NULL; }

extern "C" int skd_synchronize(skd_state *st) {
  if (!st) return SKD_ERR_NULL;
  return wait_stream(st);
}

extern "C" int skd_debug_read_hidden(skd_state *st, float *x_out) {
  if (!st || !x_out) return SKD_ERR_NULL;
  if (!st->have_hidden) return SKD_ERR_ORDER;
  HIPCHECK(hipMemcpyAsync(x_out, st->x, (size_t)st->cfg.batch * st->cfg.d_model * sizeof(float), hipMemcpyDeviceToHost,
                          st->stream));
  return wait_stream(st);
}

extern "C" int skd_debug_kv_load(skd_state *st, int32_t cols, const float *const *Kin, const float *const *Vin,
                                 const int32_t *start_in) {
  if (!st) return SKD_ERR_NULL;
  const skd_config &c = st->cfg;
  if (cols < c.prompt_size || cols >= c.sequence_length) return SKD_ERR_RANGE;
  const int B = c.batch, d = c.d_model;
  if (start_in)
    for (int b = 0; b < B; ++b)
      if (start_in[b] < 0 || start_in[b] >= cols) return SKD_ERR_RANGE;
  {
    std::vector<int32_t> start(B, 0);
    if (start_in) start.assign(start_in, start_in + B);
    set_start(st, start);
    SKDCHECK(upload_start(st));  // the bf16 pages are addressed by real position
  }
  const size_t n = (size_t)B * cols * d;
  float *kd = nullptr, *vd = nullptr;
  HIPCHECK(hipMalloc((void **)&kd, n * sizeof(float)));
  if (hipMalloc((void **)&vd, n * sizeof(float)) != hipSuccess) { (void)hipFree(kd); return SKD_ERR_NOMEM; }
  int rc = SKD_OK;
  for (int l = 0; l < c.L && rc == SKD_OK; ++l) {
    if (st->kv_cap[l] < cols) {  // the layer left the window before column `cols`: it never runs again
      st->kv_len[l] = st->kv_cap[l];
      continue;
    }
    const float *ks = Kin ? Kin[l] : nullptr, *vs = Vin ? Vin[l] : nullptr;
    const bool have = ks && vs;
    if (have && (hipMemcpyAsync(kd, ks, n * sizeof(float), hipMemcpyHostToDevice, st->stream) != hipSuccess ||
                 hipMemcpyAsync(vd, vs, n * sizeof(float), hipMemcpyHostToDevice, st->stream) != hipSuccess)) {
      rc = SKD_ERR_HIP;
      break;
    }
    if (st->bf16)
      kv_load_bf16(st->stream, have ? kd : nullptr, have ? vd : nullptr, (bf16_t *)st->pool, bt_layer(st, l), st->start_dev, cols, B, st->geom);
    else
      kv_load_f32(st->stream, have ? kd : nullptr, have ? vd : nullptr, (float *)st->pool, bt_layer(st, l), cols, B, st->geom);
    if (hipStreamSynchronize(st->stream) != hipSuccess) { rc = SKD_ERR_HIP; break; }
    st->kv_len[l] = cols;
  }
  (void)hipFree(kd);
  (void)hipFree(vd);
  if (rc != SKD_OK) return rc;
  st->prefilled = true;
  st->steps_done = cols - c.prompt_size;
  st->have_hidden = false;
  st->have_argmax = false;
  return SKD_OK;
}

extern "C" int skd_debug_kv_read(skd_state *st, int32_t layer, int32_t b, float *k_out, float *v_out) {
  if (!st || !k_out || !v_out) return SKD_ERR_NULL;
  const skd_config &c = st->cfg;
  if (layer < 0 || layer >= c.L || b < 0 || b >= c.batch) return SKD_ERR_RANGE;
  const int len = st->kv_len[layer], d = c.d_model;
  if (len == 0) return SKD_OK;
  float *kd = nullptr, *vd = nullptr;
  HIPCHECK(hipMalloc((void **)&kd, (size_t)len * d * sizeof(float)));
  if (hipMalloc((void **)&vd, (size_t)len * d * sizeof(float)) != hipSuccess) { (void)hipFree(kd); return SKD_ERR_NOMEM; }
  const int32_t *row = bt_layer(st, layer) + (size_t)b * st->geom.max_pages;
  if (st->bf16) kv_read_bf16(st->stream, (const bf16_t *)st->pool, row, st->start_host.empty() ? 0 : st->start_host[b], len, kd, vd, st->geom);
  else kv_read_f32(st->stream, (const float *)st->pool, row, len, kd, vd, st->geom);
  int rc = SKD_OK;
  if (hipMemcpyAsync(k_out, kd, (size_t)len * d * sizeof(float), hipMemcpyDeviceToHost, st->stream) != hipSuccess ||
      hipMemcpyAsync(v_out, vd, (size_t)len * d * sizeof(float), hipMemcpyDeviceToHost, st->stream) != hipSuccess ||
      hipStreamSynchronize(st->stream) != hipSuccess)
    rc = SKD_ERR_HIP;
  (void)hipFree(kd);
  (void)hipFree(vd);
  return rc != SKD_OK ? rc : intact(st);
}
