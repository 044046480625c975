// Internal launch interface between the host engine and the gfx950 kernels.
// Not part of the public ABI (include/skd.h is).
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <stdint.h>

#include "kv_pages.h"

namespace skd {

typedef uint16_t bf16_t;  // raw bfloat16 bit pattern in host-visible signatures

// Per-launch timing.  While a thread has a LaunchTimer installed, every kernel launch it makes through
// SKD_LAUNCH takes a (start, stop) event pair from the timer and goes through hipExtLaunchKernelGGL, which
// stamps the two events with the begin and end of that kernel itself (the dispatch's own time stamps, what a
// kernel trace reports), not with the time of extra marker packets around it.
struct LaunchTimer {
  virtual void next(hipEvent_t *start, hipEvent_t *stop) = 0;

 protected:
  ~LaunchTimer() = default;
};
extern thread_local LaunchTimer *g_launch_timer;

#define SKD_LAUNCH(kernel, grid, blk, lds, stream, ...)                                        \
  do {                                                                                         \
    if (skd::g_launch_timer) {                                                                 \
      hipEvent_t e0_ = nullptr, e1_ = nullptr;                                                 \
      skd::g_launch_timer->next(&e0_, &e1_);                                                   \
      hipExtLaunchKernelGGL(kernel, grid, blk, lds, stream, e0_, e1_, 0, __VA_ARGS__);         \
    } else {                                                                                   \
      hipLaunchKernelGGL(kernel, grid, blk, lds, stream, __VA_ARGS__);                         \
    }                                                                                          \
  } while (0)

// Sum over the wave, the same value in every lane: rotations inside the rows of 16 lanes (DPP, no LDS round trip as in
// __shfl_xor), then the four row sums as scalars.
__device__ inline float wave_sum_f(float v) {
#define SKD_ROR(n) v += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x120 + n, 0xF, 0xF, true))
  SKD_ROR(8);
  SKD_ROR(4);
  SKD_ROR(2);
  SKD_ROR(1);
#undef SKD_ROR
  const int i = __builtin_bit_cast(int, v);
  auto row = [&](int l) { return __builtin_bit_cast(float, __builtin_amdgcn_readlane(i, l)); };
  return (row(0) + row(16)) + (row(32) + row(48));
}

// ---------------------------------------------------------------- fp32 debug path
// Everything row-major fp32.  KV page layout: [K|V][page_tokens][H*dh].
void f32_embed(hipStream_t s, float *x, const float *tok_emb, const float *pos_emb, const int32_t *tokens,
               const int32_t *start, int t, int B, int d, int V);
void f32_layernorm(hipStream_t s, const float *x, const float *g, const float *b, float *out, int B, int d);
// out[b][n] = (accumulate ? out[b][n] : 0) + bias[n] + sum_k W[n][k] * in[b][k]; optional ReLU
void f32_linear(hipStream_t s, const float *W, const float *bias, const float *in, float *out, int B, int K, int N,
                int relu, int accumulate);
void f32_kv_write(hipStream_t s, const float *qkv, float *pool, const int32_t *bt_layer, int t, int B, KvGeom g);
void f32_attention(hipStream_t s, const float *qkv, const float *pool, const int32_t *bt_layer, const int32_t *start,
                   int t, float *o, float *scores, int score_stride, int B, KvGeom g);
void f32_argmax(hipStream_t s, const float *logits, int32_t *tokens, int B, int V);
// Candidates of the sampling head's first pass, SAMPLE_CHUNK_CAND per row, shared out among the chunks of the vocabulary
// (the chunks are few: cap >= 315); z null: single pass.
constexpr int SAMPLE_CHUNK_CAND = 4096;
struct SampleScratch {
  float *z;         // [B][chunks][cap] logit / temperature
  int32_t *idx;     // the same, token
  float *max_mass;  // [B][chunks][3] maximum, mass, bound of the candidates relative to the maximum
  int32_t *count;   // [B][chunks], above cap: none listed
  int chunks, cap, first;  // set by sample_top_p
};
int sample_chunks(int V);
// temperature + top-p sampling from fp32 logits [B][V] with one uniform number per row; -1 if V > 65536.
// tokens2: second destination, or null
int sample_top_p(hipStream_t s, const float *logits, int B, int V, float temperature, float top_p, const float *u,
                 int32_t *tokens, int32_t *tokens2, SampleScratch sc);

// ---------------------------------------------------------------- bf16 production path
// Weights [N][K] are "fragment-major": 16-row x 32-column fragments stored as
// 64 lanes x 8 elements, lane = (row % 16) + 16 * ((col % 32) / 8), element =
// col % 8: one lane-wide 16-byte load is exactly one A operand of
// v_mfma_f32_16x16x32_bf16.  The 16-row tiles are bundled in groups of G
// (1..4, chosen per matrix as the tile rows one workgroup owns) and stored
// [tile / G][col / 32][tile % G], so that the G fragments a wave needs for one
// k-step are G KiB of consecutive addresses.
// Activations [rows][K] (rows padded to 16) use the same 16 x 32 tiles in the
// order [row / 16][col / 32], but row-major inside a tile (16 rows of 64
// bytes): one tile is still one 1 KiB B-operand load (lane l reads 16-byte
// slot (l % 16) * 4 + l / 16), while a producer that owns a row stores 64-byte
// runs instead of scattered 8- or 16-byte pieces.
// Rows of the batched prompt pass.  Only real tokens get rows: sequence b owns P - start[b] rows (its real
// positions, in order), padded to a multiple of 16, starting at first_row[b].
struct RowMap {
  const int32_t *seq;        // [rows] sequence of each row (rows past the last sequence: -1)
  const int32_t *first_row;  // [B] multiple of 16
  const int32_t *start;      // [B] first real column of each sequence
  int P;                     // prompt columns
};

struct PromptMap {  // by-value kernel argument
  int32_t start[128], first[128];
  uint8_t order[128];
};
// start, order, first [B], seq [rows_pad] and tiles [rows_pad / 16] from pm; rows = rows of all sequences (each padded to 16)
void bf16_prompt_map(hipStream_t s, const PromptMap &pm, int B, int rows, int rows_pad, int P, const KvGeom &kv, int32_t *start,
                     int32_t *order, int32_t *first, int32_t *seq, CacheTile *tiles);

enum GemmEpilogue {
  EPI_PARTIAL = 0,  // fp32 partial sums [split][B_pad][N], no bias
  EPI_QKV = 1,      // + bias; q -> row-major bf16, k/v -> row-major staging rows (filed into the page by bf16_attention)
  EPI_RELU = 2,     // + bias, ReLU -> activation tiles bf16 [B_pad][N]
  EPI_LOGITS = 3,   // optional fp32 logits [B][N] + per-workgroup (max, argmax) partials
  EPI_QKV_ROWS = 4, // batched prompt: + bias; q -> activation tiles [rows][d]; k/v -> KV page slot of (sequence, position)
  EPI_RESID = 5     // batched prompt: x[row][n] += value + bias (fp32 residual stream)
};

struct GemmArgs {
  const bf16_t *W;     // fragment-major [Nt_pad*16][K], tiles in groups of G
  int G;               // tile-group size of W's layout (Nt_pad is a multiple of 12, so of every G)
  const bf16_t *A;     // activation tiles [B_pad][K]
  const float *bias;   // [N] or null
  int N, K, B, B_pad;
  int t0;              // bf16_gemm_tile, bf16_gemm_mid: first weight tile (N outputs from row 16 t0 on; EPI_QKV_ROWS only)
  int split;           // workgroups along K (grid.y)
  int ws_rot;          // bf16_gemm_ws: workgroups start their K range at different stages
  // batched prompt processing: activation rows are the real (sequence, position) pairs of `rm`, handled in
  // output tiles or in chunks of B_pad rows along grid.z.  rows = 0: one chunk whose rows are the batch (decode).
  int rows;            // rows of the prompt pass (whole 16-row tiles)
  RowMap rm;           // EPI_QKV_ROWS
  float *x;            // EPI_RESID: [rows][N] fp32
  // outputs (by epilogue)
  float *partial;      // EPI_PARTIAL
  bf16_t *q_out;       // EPI_QKV: [B_pad][d] row-major
  union {
    bf16_t *kv_new;                // EPI_QKV: [B][k | v][d] row-major
    const CacheTile *cache_tiles;  // EPI_QKV_ROWS in bf16_gemm_tile, bf16_gemm_mid: [rows / 16], padded to 256 rows
  };
  bf16_t *kv_pool;     // EPI_QKV_ROWS
  const int32_t *bt_layer;  // EPI_QKV_ROWS: [B][max_pages]
  int d;               // EPI_QKV, EPI_QKV_ROWS: d_model (N = 3d)
  KvGeom kv;           // EPI_QKV_ROWS
  bf16_t *act_out;     // EPI_RELU
  // bf16_gemm_ln: A = LayerNorm(ln_x + ln_bias + sum of ln_split partial sums [ln_split][B_pad][K]; ln_g, ln_b), made by
  // every workgroup; ln_x_out (another buffer than ln_x) receives the sum
  const float *ln_x, *ln_partial, *ln_bias, *ln_g, *ln_b;
  float *ln_x_out;
  int ln_split;
  float *logits;       // EPI_LOGITS (nullable)
  const float *attn_part;  // bf16_gemm_merge: the attention's shares (AttnArgs::part), attn_splits of them
  int attn_splits;
  int head_full, head_mid, head_mid_r;  // EPI_LOGITS: workgroups of R = G tiles, of head_mid_r; then single tiles (bf16_head_tiles)
  float *pmax;         // EPI_LOGITS: [groups][B_pad]
  int32_t *pidx;       // EPI_LOGITS
};
// R in 1..4: 16-row weight tiles per workgroup (each wave accumulates all of them over its share of K); U in {1,2,4}: k-steps per register buffer (prefetch depth);
// waves in {4,8}: waves per workgroup.  K/32 must be a multiple of a.split.
// Returns the number of row groups launched (grid.x), or -1 for an unsupported shape.
int bf16_gemm(hipStream_t s, const GemmArgs &a, int epilogue, int R, int U, int waves);
// At most 4 rows, K <= 4096 (2048 for 3 and 4), EPI_QKV or EPI_RELU: with the row reducer in the prologue (ln_*; a.A is
// not read).  The check launches nothing (N, K, B, B_pad, G, split, rows and ln_split of `a` are read): groups or -1.
int bf16_gemm_ln(hipStream_t s, const GemmArgs &a, int epilogue, int R);
int bf16_gemm_ln_check(const GemmArgs &a, int epilogue, int R);
// The output projection (EPI_PARTIAL) of one or two rows, K <= 4096, behind an attention of 2 to 8 splits that were not merged:
// merges them itself (attn_*, kv.dh; a.A is not read).  R is 1 or 2.  Groups or -1.
int bf16_gemm_merge(hipStream_t s, const GemmArgs &a, int R, int U, int waves);
int bf16_gemm_merge_check(const GemmArgs &a, int R, int waves);
// The same shape checks without a launch (only N, K, B_pad, G, split and rows of `a` are read): groups or -1.
int bf16_gemm_check(const GemmArgs &a, int epilogue, int R, int U, int waves);
int bf16_gemm_groups(int N, int R);
// Sets head_* of `a` for workgroups of R tiles of which `slots` run at once (0: equal groups) and returns their number.
int bf16_head_tiles(GemmArgs &a, int R, int slots);
// Decode projections with B_pad = 96 or 128 on the wave-specialised kernel (weight-streaming waves + activation-loading
// waves); (K / 32 / split) must be a multiple of 4.  Returns the row groups launched, or -1 (nothing launched) for
// shapes it does not handle; bf16_gemm_ws_check answers the same without launching.
int bf16_gemm_ws(hipStream_t s, const GemmArgs &a, int epilogue, int R);
int bf16_gemm_ws_check(const GemmArgs &a, int epilogue, int R);
// Batched prompt only (a.rows > 0; EPI_QKV_ROWS, EPI_RESID, EPI_RELU or EPI_PARTIAL; a.split > 1 with EPI_PARTIAL
// only): output tiles with LDS-staged operands.  Buffers are padded to whole tiles of 256 rows: the rows past a.rows of
// the last tile are read and written.  EPI_PARTIAL: fp32 sums [split][B_pad][N], B_pad = rows of that buffer.
// Both return -1 for shapes that do not tile (nothing launched).
// 256 x 256 tiles: N % 256 == 0.
int bf16_gemm_tile(hipStream_t s, const GemmArgs &a, int epilogue);
// weight_rows x act_rows = 256 x 128, 128 x 256, 128 x 128, 64 x 128, 128 x 64 or 64 x 64 tiles: N % weight_rows == 0.
int bf16_gemm_mid(hipStream_t s, const GemmArgs &a, int epilogue, int weight_rows, int act_rows);

void bf16_embed_ln(hipStream_t s, const int32_t *tokens, const int32_t *start, int t, const bf16_t *tok_emb,
                   const bf16_t *pos_emb, const float *g, const float *b, float *x, bf16_t *a_out, int B, int d,
                   int V);
// x[b][:] = x_in[b][:] + bias + sum_s partial[s][b][:] (x_in may be x); a_out = LayerNorm(x; g, b) as bf16 activation tiles
void bf16_reduce_ln(hipStream_t s, const float *partial, int split, int B_pad, const float *bias, const float *x_in,
                    float *x, const float *g, const float *b, bf16_t *a_out, int B, int d);
// Decode attention at position t.  Keys of columns start[b] .. t-1 (slots 0 .. t-start[b]-1) come from the pages; k and v of position t itself come
// from kv_new (written by the EPI_QKV projection) and are stored into the page slot of t by this kernel.
struct AttnArgs {
  const bf16_t *q;          // [B_pad][d] row-major
  const bf16_t *kv_new;     // [B][k | v][d] row-major
  bf16_t *pool;
  const int32_t *bt_layer;  // [B][max_pages]
  const int32_t *start;     // [B] first real column of each row
  const int32_t *order;     // [B] rows sorted by descending length: workgroup x/H handles row order[x/H] (null = identity)
  int t;                    // position being processed: cached keys start[b] .. t-1, plus t itself from kv_new
  int B, splits;
  int waves;                // waves per workgroup: 2, 4, 8 or 16
  KvGeom kv;
  bf16_t *o;                // activation tiles [B_pad][d]
  bool merge;               // splits > 1: whether their merge is launched too (else bf16_gemm_merge reads `part`)
  float *part;              // splits > 1: [splits][B*H][dh + 4], numerators, maximum and denominator
};
void bf16_attention(hipStream_t s, const AttnArgs &a);
// Causal attention of a whole prompt: query rows (b, pos), up to 128 positions per workgroup, keys of columns start[b] .. pos.
struct AttnRowsArgs {
  const bf16_t *q;          // activation tiles [rows][d]
  const bf16_t *pool;
  const int32_t *bt_layer;  // [B][max_pages]
  RowMap rm;
  int B, max_len;           // sequences, positions of the longest one
  KvGeom kv;
  bf16_t *o;                // activation tiles [rows][d]
};
void bf16_attention_rows(hipStream_t s, const AttnRowsArgs &a);
// Batched prompt row kernels; tokens laid out [P][B].
void bf16_embed_ln_rows(hipStream_t s, const int32_t *tokens, RowMap rm, int rows, const bf16_t *tok_emb,
                        const bf16_t *pos_emb, const float *g, const float *b, float *x, bf16_t *a_out, int B, int d,
                        int V);
void bf16_ln_rows(hipStream_t s, float *x, const float *g, const float *b, bf16_t *a_out, int rows, int d);
// x_out[b][:] = row of sequence b's last prompt position (+ bias + sum of `split` partial sums [split][stride][d] when
// split > 0); a_out = its LayerNorm
void bf16_last_rows_ln(hipStream_t s, const float *x_rows, RowMap rm, const float *partial, int split, int stride,
                       const float *bias, const float *g, const float *b, float *x_out, bf16_t *a_out, int B, int d);
// tokens2: second destination, or null
void bf16_argmax_final(hipStream_t s, const float *pmax, const int32_t *pidx, int groups, int B_pad, int32_t *tokens,
                       int32_t *tokens2, int B);

// logits [B][V] (optional) = partial sums [split][B_pad][N] of an LM head (N = V in whole tiles; EPI_PARTIAL) added up, and the
// greedy tokens (optional; tokens2: second destination, or null)
constexpr int LOGITS_SPLIT = 8;       // K parts at most
void bf16_logits_sum(hipStream_t s, const float *partial, int split, int B_pad, int N, int V, float *logits, int32_t *tokens,
                     int32_t *tokens2, int B);

// A whole decode column of a narrow model in one launch (team_column.hip).
struct TeamLayer {
  const bf16_t *wqkv, *wo, *w1, *w2;  // fragment-major
  const float *ln1_g, *ln1_b, *bqkv, *bo, *ln2_g, *ln2_b, *b1, *b2;
  const int32_t *bt;                  // [B][max_pages]
};
constexpr int TEAM_SLOTS = 16;        // XCDs at most
struct TeamSlot {                     // a line each: one XCD
  uint32_t registered, team, next, pad0[29];
  uint32_t arrived, pad1[31];
};
struct TeamCtl {                      // zero before the first launch; every launch leaves it zero
  TeamSlot slot[TEAM_SLOTS];
  uint32_t next_group, pad0[31];
  uint32_t left, pad1[31];
};
struct TeamWork {                     // for 8 groups of 16 rows each
  bf16_t *q, *kv, *o, *u;             // [16][d] | [16][k | v][d] | activation tiles [16][d] | activation tiles [16][f]
  float *y;                           // [16][d]
  float *part;                        // [128][132]: numerators, maximum and denominator of a share of a pair's keys
};
struct TeamStep {                     // k-steps of a wave and a tile, in order (team_steps)
  uint16_t e[8];
};
struct TeamSums {                     // of the separate kernel
  int tiles, waves, unit, split;      // tiles of a workgroup and of a group of the layout, waves, k-steps of a buffer, K parts
  bool rotate;
};
struct TeamArgs {
  const TeamLayer *layers;            // device, all L
  int n, warmup, L;                   // active: 0 .. warmup - 1 and L - n + warmup .. L - 1
  int d, f, B, V, t;
  int groups;                         // bf16_team_groups(B)
  int longest;                        // cached positions of the longest row
  int attn_waves, attn_splits;        // waves and splits of the separate attention
  const TeamStep *out_steps, *ffn2_steps;  // [d / 16][8 waves]
  int out_parts, ffn2_parts;          // K parts
  int rot_qkv, rot_ffn1;              // waves begin rotated
  bool wide;                          // 96 or 128 padded rows
  int workgroups;                     // of the launch: one per CU
  int members;                        // of a team, at most
  const int32_t *tokens, *start, *order;  // [B]; order: rows by descending length, or null
  const bf16_t *tok_emb, *pos_emb;
  const float *lnf_g, *lnf_b;
  bf16_t *pool;
  KvGeom kv;
  TeamWork work;
  TeamCtl *ctl;
  uint32_t *gave_up;                  // host memory: written if a wait runs out (GaveUp)
  float *x_out;                       // [B][d] residual rows behind the last layer
  bf16_t *a_out;                      // activation tiles [B_pad][d]: their final LayerNorm
};
bool bf16_team_ok(int d, int f, int B);
// Whether a column of B rows whose longest has `longest` cached keys, and all of them `total`, is faster this way.
bool bf16_team_keys(int d, int B, long longest, long total);
int bf16_team_groups(int B);
int bf16_team_members(int cus, int d);
size_t bf16_team_rows();              // rows of each work buffer
size_t bf16_team_part();              // floats of work.part
// Sets what `a` says about sums (d, f given) and the two tables of bf16_team_steps(d) entries, or only checks (null);
// false: not among those that the column can take.
bool bf16_team_sums(TeamArgs &a, int B_pad, const TeamSums &qkv, const TeamSums &out, const TeamSums &ffn1, const TeamSums &ffn2,
                    TeamStep *out_steps, TeamStep *ffn2_steps);
size_t bf16_team_steps(int d);
bool bf16_team_states(const TeamArgs &a, int states, int splits);
bool bf16_team_column(hipStream_t s, const TeamArgs &a);

// weight preparation (source fp32 or bf16 row-major, on device)
void prep_matrix_frag(hipStream_t s, const void *src, int src_is_bf16, bf16_t *dst, long N, long K, long N_pad,
                      int G);
void prep_matrix_rm_bf16(hipStream_t s, const void *src, int src_is_bf16, bf16_t *dst, long n);
void prep_to_f32(hipStream_t s, const void *src, int src_is_bf16, float *dst, long n);
// KV debug hooks: [B][cols][d] fp32 <-> pages
void kv_load_f32(hipStream_t s, const float *K, const float *V, float *pool, const int32_t *bt_layer, int cols, int B,
                 KvGeom g);
void kv_load_bf16(hipStream_t s, const float *K, const float *V, bf16_t *pool, const int32_t *bt_layer,
                  const int32_t *start, int cols, int B, KvGeom g);
void kv_read_f32(hipStream_t s, const float *pool, const int32_t *bt_row, int len, float *K, float *V, KvGeom g);
void kv_read_bf16(hipStream_t s, const bf16_t *pool, const int32_t *bt_row, int start, int len, float *K, float *V,
                  KvGeom g);

}  // namespace skd
