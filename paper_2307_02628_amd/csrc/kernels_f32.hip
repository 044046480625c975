// fp32 debug path: small, straightforward kernels (no MFMA, no tiling) whose
// only job is to be an easily-audited GPU implementation of the decode step
// for the tight-tolerance parity build.  Not tuned.
#include "skd_kernels.h"

namespace skd {

__device__ inline float row_max_f(float v) {  // over each row of 16 lanes, the same value in every lane of the row
#define SKD_ROR(n) v = fmaxf(v, __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x120 + n, 0xF, 0xF, true)))
  SKD_ROR(8);
  SKD_ROR(4);
  SKD_ROR(2);
  SKD_ROR(1);
#undef SKD_ROR
  return v;
}
__device__ inline float wave_max(float v) {
  const int i = __builtin_bit_cast(int, row_max_f(v));
  auto row = [&](int l) { return __builtin_bit_cast(float, __builtin_amdgcn_readlane(i, l)); };
  return fmaxf(fmaxf(row(0), row(16)), fmaxf(row(32), row(48)));
}
// sum over a 256-thread workgroup; `sh` holds >= 4 floats; result to all threads
__device__ inline float block_sum(float v, float *sh) {
  v = wave_sum_f(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  float r = 0;
  for (unsigned w = 0; w < (blockDim.x >> 6); ++w) r += sh[w];
  return r;
}

__global__ void k_f32_embed(float *x, const float *tok_emb, const float *pos_emb, const int32_t *tokens,
                            const int32_t *start, int t, int d, int V) {
  const int b = blockIdx.x;
  int tok = tokens[b];
  tok = tok < 0 ? 0 : (tok >= V ? V - 1 : tok);
  int pos = t - start[b];  // real tokens before this column
  if (pos < 0) pos = 0;    // padding column: never read later
  for (int k = threadIdx.x; k < d; k += blockDim.x) x[(long)b * d + k] = tok_emb[(long)tok * d + k] + pos_emb[(long)pos * d + k];
}

__global__ void k_f32_layernorm(const float *x, const float *g, const float *bt, float *out, int d) {
  __shared__ float sh[4];
  const float *xr = x + (long)blockIdx.x * d;
  float s = 0;
  for (int k = threadIdx.x; k < d; k += blockDim.x) s += xr[k];
  const float mean = block_sum(s, sh) / d;
  float v = 0;
  for (int k = threadIdx.x; k < d; k += blockDim.x) v += (xr[k] - mean) * (xr[k] - mean);
  const float rstd = 1.0f / sqrtf(block_sum(v, sh) / d + 1e-5f);
  for (int k = threadIdx.x; k < d; k += blockDim.x) out[(long)blockIdx.x * d + k] = (xr[k] - mean) * rstd * g[k] + bt[k];
}

// one wave per output element (b, n): lanes stride over k
__global__ void k_f32_linear(const float *W, const float *bias, const float *in, float *out, int K, int N, int relu,
                             int accumulate) {
  const int n = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  const int b = blockIdx.y;
  if (n >= N) return;
  const float *w = W + (long)n * K, *a = in + (long)b * K;
  float acc = 0;
  for (int k = threadIdx.x & 63; k < K; k += 64) acc += w[k] * a[k];
  acc = wave_sum_f(acc);
  if ((threadIdx.x & 63) == 0) {
    float v = acc + (bias ? bias[n] : 0.f);
    if (relu) v = fmaxf(v, 0.f);
    float *o = out + (long)b * N + n;
    *o = accumulate ? *o + v : v;
  }
}

__device__ inline long f32_kv_off(const int32_t *bt_row, int pos, int which, const KvGeom &g) {
  const int page = bt_row[pos / g.page_tokens];
  return (long)page * g.page_elems + ((long)which * g.page_tokens + pos % g.page_tokens) * (g.H * g.dh);
}

__global__ void k_f32_kv_write(const float *qkv, float *pool, const int32_t *bt_layer, int t, KvGeom g) {
  const int b = blockIdx.x, d = g.H * g.dh;
  const int32_t *bt_row = bt_layer + (long)b * g.max_pages;
  float *Kd = pool + f32_kv_off(bt_row, t, 0, g), *Vd = pool + f32_kv_off(bt_row, t, 1, g);
  for (int k = threadIdx.x; k < d; k += blockDim.x) {
    Kd[k] = qkv[(long)b * 3 * d + d + k];
    Vd[k] = qkv[(long)b * 3 * d + 2 * d + k];
  }
}

// one 64-lane workgroup per (b, h); scores kept in a global scratch row
__global__ void k_f32_attention(const float *qkv, const float *pool, const int32_t *bt_layer, const int32_t *start,
                                int t, float *o, float *scores, int score_stride, KvGeom g) {
  const int b = blockIdx.x / g.H, h = blockIdx.x % g.H, d = g.H * g.dh, lane = threadIdx.x;
  const int32_t *bt_row = bt_layer + (long)b * g.max_pages;
  const float *q = qkv + (long)b * 3 * d + h * g.dh;
  float *sc = scores + (long)blockIdx.x * score_stride;
  const int j0 = start[b];
  const float inv = 1.0f / sqrtf((float)g.dh);
  float mx = -3.0e38f;
  for (int j = j0 + lane; j <= t; j += 64) {
    const float *kr = pool + f32_kv_off(bt_row, j, 0, g) + h * g.dh;
    float s = 0;
    for (int e = 0; e < g.dh; ++e) s += q[e] * kr[e];
    s *= inv;
    sc[j] = s;
    mx = fmaxf(mx, s);
  }
  mx = wave_max(mx);
  float den = 0;
  for (int j = j0 + lane; j <= t; j += 64) {
    const float p = expf(sc[j] - mx);
    sc[j] = p;
    den += p;
  }
  den = wave_sum_f(den);
  __syncthreads();  // scores written by other lanes are read below
  for (int e = lane; e < g.dh; e += 64) {
    float acc = 0;
    for (int j = j0; j <= t; ++j) acc += sc[j] * pool[f32_kv_off(bt_row, j, 1, g) + h * g.dh + e];
    o[(long)b * d + h * g.dh + e] = (j0 <= t) ? acc / den : 0.f;
  }
}

__global__ void k_f32_argmax(const float *logits, int32_t *tokens, int V) {
  __shared__ float sv[256];
  __shared__ int si[256];
  const float *z = logits + (long)blockIdx.x * V;
  float best = -3.0e38f;
  int bi = 0x7fffffff;
  for (int v = threadIdx.x; v < V; v += blockDim.x)
    if (z[v] > best) { best = z[v]; bi = v; }  // ascending v per thread: first maximum kept
  sv[threadIdx.x] = best;
  si[threadIdx.x] = bi;
  __syncthreads();
  for (int s = blockDim.x / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) {
      const float ov = sv[threadIdx.x + s];
      const int oi = si[threadIdx.x + s];
      if (ov > sv[threadIdx.x] || (ov == sv[threadIdx.x] && oi < si[threadIdx.x])) { sv[threadIdx.x] = ov; si[threadIdx.x] = oi; }
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) tokens[blockIdx.x] = si[0];
}

// ------------------------------------------------------------------ sampling head (both paths; fp32 logits)
// Temperature + nucleus (top-p) sampling, one 1024-thread workgroup per row.
// Wave w keeps the contiguous index range [w*R*64, (w+1)*R*64) in registers, R = ceil(V / 1024) <= 64 rows of 64
// tokens, lane l holding token w*R*64 + 64 i + l of row i (coalesced 256-byte loads).
//   p_i = exp((z_i - max z) / T);  nucleus = {p_i >= tau}, tau = the largest value whose upper set has mass
//   >= top_p * sum p  (found bit by bit on the float bit pattern; tokens tied with tau are in);
//   token = first index of the nucleus whose running mass (ascending index) exceeds u * mass(nucleus).
// Every sum is taken in a fixed order, so a given (logits, u) always yields the same token.
constexpr int SAMPLE_C = 64;
constexpr int SAMPLE_CAND = 4096;  // candidates that four waves finish, 16 per lane
constexpr int SAMPLE_MID = 1024;   // tokens between the bounds of the threshold that one wave searches, 16 per lane

// Sums over each row of 16 lanes, the same value in every lane of the row (the pairs that are added are the same seen
// from each lane, so the float result is too).
__device__ inline int row_sum_i(int v) {
#define SKD_ROR(n) v += __builtin_amdgcn_mov_dpp(v, 0x120 + n, 0xF, 0xF, true)
  SKD_ROR(8);
  SKD_ROR(4);
  SKD_ROR(2);
  SKD_ROR(1);
#undef SKD_ROR
  return v;
}
__device__ inline int wave_sum_i(int v) {  // the same value in every lane, as wave_sum_f
  v = row_sum_i(v);
  return (__builtin_amdgcn_readlane(v, 0) + __builtin_amdgcn_readlane(v, 16)) + (__builtin_amdgcn_readlane(v, 32) + __builtin_amdgcn_readlane(v, 48));
}
__device__ inline unsigned wave_max_u(unsigned v) {
#define SKD_ROR(n) v = max(v, (unsigned)__builtin_amdgcn_mov_dpp((int)v, 0x120 + n, 0xF, 0xF, true))
  SKD_ROR(8);
  SKD_ROR(4);
  SKD_ROR(2);
  SKD_ROR(1);
#undef SKD_ROR
  auto row = [&](int l) { return (unsigned)__builtin_amdgcn_readlane((int)v, l); };
  return max(max(row(0), row(16)), max(row(32), row(48)));
}
__device__ inline float row_sum_f(float v) {
#define SKD_ROR(n) v += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x120 + n, 0xF, 0xF, true))
  SKD_ROR(8);
  SKD_ROR(4);
  SKD_ROR(2);
  SKD_ROR(1);
#undef SKD_ROR
  return v;
}

// Place of candidate k in LDS: a lane reads 16 (or 4) in a row, and without the gap 16 waves that do so have 16 lanes on a
// bank at a time (2 us of the sampling kernel).
__device__ inline int cand_at(int k) { return k + (k >> 4); }

struct SampleExchange {  // LDS of the finishing waves
  float sums[2][4];
  int pick[4], tail[4];
  float mass[2][16];  // sample_search: one set per round in turn
  int count[2][16];
  float at[64];       // sample_search_few
};
// The searches below find the largest value of [lower, upper) whose upper set has the target mass (or `lower`).  All of them
// add up the masses as sample_finish does, PER consecutive candidates to a lane, so that which one runs does not show where
// rounding decides.

// At most 64 candidates: the masses from every candidate on, four to a wave; one round.
__device__ inline unsigned sample_search_few(const float *cand_p, int C, unsigned lower, unsigned upper, float target, SampleExchange &ex) {
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  float v[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) v[j] = 4 * lane + j < C ? cand_p[cand_at(4 * lane + j)] : 0.f;
#pragma unroll
  for (int i = 0; i < 4; ++i) {  // candidates 4 w + i
    const float t = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v[i]), w));
    float m = 0.f;
#pragma unroll
    for (int j = 0; j < 4; ++j) m += __float_as_uint(v[j]) >= __float_as_uint(t) ? v[j] : 0.f;
    m = wave_sum_f(m);
    if (lane == 0) ex.at[4 * w + i] = m;
  }
  __syncthreads();
  // (candidates at or above `upper`: what they have together counts from upper - 1 on)
  unsigned T = lane < C && ex.at[lane] >= target ? min(__float_as_uint(cand_p[cand_at(lane)]), upper - 1u) : lower;
  return wave_max_u(T);
}
// C <= 64 PER candidates, by all 16 waves: every wave holds all of them and sums the masses at or above
// a trial value of its own, so a round divides the interval [lo, hi) by 17; it ends where one candidate is left in it
// (ties: where its bits are known).  One wave alone, two bits a round, took 8.6 us for 260 to 820 candidates.
template <int PER>
__device__ inline unsigned sample_search(const float *cand_p, int C, unsigned lo, unsigned hi, float target, SampleExchange &ex) {
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  float v[PER];
#pragma unroll
  for (int j = 0; j < PER; ++j) v[j] = PER * lane + j < C ? cand_p[cand_at(PER * lane + j)] : 0.f;
  int c_lo = C, c_hi = -1;  // candidates at or above lo, hi (-1: not counted)
  for (int set = 0; hi - lo > 1 && (c_hi < 0 || c_lo - c_hi > 1); set ^= 1) {
    // ascending with the wave; the largest lies above lo and none reaches hi, so the interval shrinks
    const unsigned q = (hi - lo) / 17, r = (hi - lo) % 17;
    auto trial = [&](int k) { return lo + q * (k + 1) + r * (k + 1) / 17; };
    const unsigned t = trial(w);
    float m = 0.f;
    int c = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const bool in = __float_as_uint(v[j]) >= t;
      m += in ? v[j] : 0.f;
      c += in ? 1 : 0;
    }
    m = wave_sum_f(m);
    c = wave_sum_i(c);
    if (lane == 0) {
      ex.mass[set][w] = m;
      ex.count[set][w] = c;
    }
    __syncthreads();  // (a set is written again two rounds later)
    const float mk = ex.mass[set][lane & 15];
    const int ck = ex.count[set][lane & 15];
    // descending with the wave: sums of the same terms in the same order, fewer of them
    const int K = __popcll(__ballot(mk >= target) & 0xffffull);
    if (K < 16) {
      hi = trial(K);
      c_hi = __builtin_amdgcn_readlane(ck, K);
    }
    if (K > 0) {
      const unsigned at = trial(K - 1);
      c_lo = __builtin_amdgcn_readlane(ck, K - 1);
      lo = at;
    }
  }
  return lo;
}
// The rest of a row on its C <= 64 PER NW candidates (ascending index), by the first NW (1 or 4) waves of the workgroup: the
// draw among those at or above the threshold, which one wave is given (T) and four find bit by bit (16 candidates a lane keep
// the SIMDs busy; dividing by 17 would take more work than it saves rounds: 9000 tokens of a flat row 42 -> 45 us).
template <int PER, int NW>
__device__ inline void sample_finish(const float *cand_p, const int *cand_i, int C, unsigned lower, unsigned upper,
                                     float target, unsigned T, float u, int32_t *token, int32_t *token2, SampleExchange &ex) {
  const int lane = threadIdx.x & 63, w = NW == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c0 = (w * 64 + lane) * PER;  // this lane's candidates c0 .. c0 + PER - 1 (index order)
  float v[PER];
#pragma unroll
  for (int j = 0; j < PER; ++j) v[j] = c0 + j < C ? cand_p[cand_at(c0 + j)] : 0.f;
  int set = 0;
  if constexpr (NW > 1) {
    T = 0;
    for (int bit = 29; bit >= 0; --bit) {
      const unsigned cand = T | (1u << bit);
      if (cand >= upper) continue;
      if (cand <= lower) { T = cand; continue; }
      float m = 0;
#pragma unroll
      for (int j = 0; j < PER; ++j) m += (__float_as_uint(v[j]) >= cand) ? v[j] : 0.f;
      m = wave_sum_f(m);
      set ^= 1;
      if (lane == 0) ex.sums[set][w] = m;
      __syncthreads();  // the set is written again two rounds later, after the next round's barrier
      m = (ex.sums[set][0] + ex.sums[set][1]) + (ex.sums[set][2] + ex.sums[set][3]);
      if (m >= target) T = cand;
    }
  }
  float lm = 0;
  int last = -1;
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    if (__float_as_uint(v[j]) < T) v[j] = 0.f;
    lm += v[j];
    if (v[j] > 0.f) last = c0 + j;
  }
  float inc = lm;  // inclusive prefix of the lanes' masses = prefix in index order
  for (int off = 1; off < 64; off <<= 1) {
    const float t = __shfl_up(inc, off);
    if (lane >= off) inc += t;
  }
  float before = 0, mass = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, inc), 63));
  if constexpr (NW > 1) {
    if (lane == 0) ex.sums[set ^ 1][w] = mass;  // last read before the barrier of the last round
    __syncthreads();
    float run = 0;
#pragma unroll
    for (int k = 0; k < NW; ++k) {
      if (k == w) before = run;
      run += ex.sums[set ^ 1][k];
    }
    mass = run;
  }
  const float goal = u * mass;
  const unsigned long long over = __ballot(before + inc > goal);
  int k = -1;
  if (over) {
    const int L = (int)__builtin_ctzll(over);
    if (lane == L) {
      float run = before + (inc - lm);
#pragma unroll
      for (int j = 0; j < PER; ++j) {
        run += v[j];
        if (k < 0 && v[j] > 0.f && run > goal) k = c0 + j;
      }
      if (k < 0) k = last;  // rounding between the lane's two summation orders: its last member
    }
    k = __builtin_amdgcn_readlane(k, L);
  }
  const unsigned long long members = __ballot(last >= 0);  // ascending with the lane
  last = members ? __builtin_amdgcn_readlane(last, 63 - (int)__builtin_clzll(members)) : -1;
  if constexpr (NW > 1) {  // the first wave that found it
    if (lane == 0) {
      ex.pick[w] = k;
      ex.tail[w] = last;
    }
    __syncthreads();
    if (w) return;
    for (int i = 1; i < NW; ++i) {
      if (k < 0) k = ex.pick[i];
      last = max(last, ex.tail[i]);
    }
  }
  if (k < 0) k = last;  // rounding at the very end: the last member of the nucleus
  if (lane == 0) {
    const int tok = k >= 0 ? cand_i[k] : 0;
    *token = tok;
    if (token2) *token2 = tok;
  }
}

__device__ __forceinline__ void sample_rest(const float *cand_p, const int *cand_i, int C, unsigned lower, unsigned upper, float target,
                                   const float *u, int b, int32_t *tokens, int32_t *tokens2, SampleExchange &ex) {
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (C <= 64) {
    const unsigned T = sample_search_few(cand_p, C, lower, upper, target, ex);
    if (w == 0) sample_finish<4, 1>(cand_p, cand_i, C, lower, upper, target, T, u[b], &tokens[b], tokens2 ? &tokens2[b] : nullptr, ex);
  } else if (C <= 256) {
    const unsigned T = sample_search<4>(cand_p, C, lower, upper, target, ex);
    if (w == 0) sample_finish<4, 1>(cand_p, cand_i, C, lower, upper, target, T, u[b], &tokens[b], tokens2 ? &tokens2[b] : nullptr, ex);
  } else if (C <= 1024) {
    const unsigned T = sample_search<16>(cand_p, C, lower, upper, target, ex);
    if (w == 0) sample_finish<16, 1>(cand_p, cand_i, C, lower, upper, target, T, u[b], &tokens[b], tokens2 ? &tokens2[b] : nullptr, ex);
  } else if (w < 4) {  // the barriers in there are those of the waves that remain
    sample_finish<16, 4>(cand_p, cand_i, C, lower, upper, target, 0u, u[b], &tokens[b], tokens2 ? &tokens2[b] : nullptr, ex);
  }
}

// First pass over a large vocabulary, spread over the chip: a workgroup takes SAMPLE_CHUNK tokens of a row, relative to
// their own maximum (the row's is not known yet): the chunk's maximum and mass, and, in index order, the tokens at or
// above the lowest of four bounds that no more than sc.cap of them reach (with one bound for all, 2^-10, any chunk with
// more than 512 tokens above it sent its row back to a single workgroup).  A factor of 0.99 covers the rounding of expf.
// One workgroup per row read and exponentiated 200 KB on one of 256 CUs: 50272 tokens, 32 rows, 46 us for everything;
// 18 us for both kernels (8 and 10).
constexpr int SAMPLE_CHUNK = 4096;
constexpr int SAMPLE_BOUNDS = 4;
// 2^-first, 2^-(first + 3), .. of the chunk's maximum; first = 4 or, for nuclei that reach deep (top_p above 0.97), 10
__device__ inline float sample_bound(int first, int j) { return __uint_as_float((127u - (first + 3u * j)) << 23); }
template <int NW>  // waves
__global__ __launch_bounds__(NW * 64) void k_sample_chunk(const float *logits, int V, float inv_temp, SampleScratch sc) {
  constexpr int NR = SAMPLE_CHUNK / (64 * NW);  // tokens per lane
  __shared__ float sh[2][NW];
  __shared__ int wcount[NW][SAMPLE_BOUNDS];
  const int b = blockIdx.y, ch = blockIdx.x, lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int base = ch * SAMPLE_CHUNK + wave * (SAMPLE_CHUNK / NW) + lane;
  const float *zr = logits + (long)b * V;
  float z[NR], mx = -3.0e38f;
#pragma unroll
  for (int i = 0; i < NR; ++i) z[i] = base + 64 * i < V ? zr[base + 64 * i] * inv_temp : -3.0e38f;  // sentinel: no such token
#pragma unroll
  for (int i = 0; i < NR; ++i) mx = fmaxf(mx, z[i]);
  mx = wave_max(mx);
  if (lane == 0) sh[0][wave] = mx;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < NW; ++w) mx = fmaxf(mx, sh[0][w]);
  float p[NR], mass = 0;
  int cnt[SAMPLE_BOUNDS] = {};
#pragma unroll
  for (int i = 0; i < NR; ++i) {
    p[i] = z[i] > -1.0e38f ? expf(z[i] - mx) : 0.f;
    mass += p[i];
#pragma unroll
    for (int j = 0; j < SAMPLE_BOUNDS; ++j) cnt[j] += p[i] >= 0.99f * sample_bound(sc.first, j) ? 1 : 0;
  }
  mass = wave_sum_f(mass);
  if (lane == 0) sh[1][wave] = mass;
#pragma unroll
  for (int j = 0; j < SAMPLE_BOUNDS; ++j) {
    const int n = wave_sum_i(cnt[j]);
    if (lane == 0) wcount[wave][j] = n;
  }
  __syncthreads();
  int total = sc.cap + 1, pos = 0;  // none of the bounds: too many tokens close to the maximum
  float bound = 0;
#pragma unroll
  for (int j = 0; j < SAMPLE_BOUNDS; ++j) {
    int n = 0, before = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const int c = wcount[w][j];
      before += w < wave ? c : 0;
      n += c;
    }
    if (n <= sc.cap) {
      total = n;
      pos = before;
      bound = sample_bound(sc.first, j);
    }
  }
  const long part = (long)b * sc.chunks + ch;
  if (threadIdx.x == 0) {
    mass = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) mass += sh[1][w];
    sc.max_mass[3 * part] = mx;
    sc.max_mass[3 * part + 1] = mass;
    sc.max_mass[3 * part + 2] = bound;
    sc.count[part] = total;
  }
  if (total > sc.cap) return;
  float *zc = sc.z + part * sc.cap;
  int32_t *ic = sc.idx + part * sc.cap;
#pragma unroll
  for (int i = 0; i < NR; ++i) {
    const bool c = p[i] >= 0.99f * bound;
    const unsigned long long m = __ballot(c);
    if (m == 0) continue;
    if (c) {
      const int k = pos + __popcll(m & ((1ull << lane) - 1ull));
      zc[k] = z[i];
      ic[k] = base + 64 * i;
    }
    pos += __popcll(m);
  }
}

// What is known of the threshold's bit pattern: lower <= threshold < upper, above = mass of the tokens at or above upper.
struct SampleBounds {
  unsigned lower, upper;
  float above;
};
// One step of the search: the trial value `cand` of a prefix T, given the mass at or above it.
__device__ inline void sample_decide(SampleBounds &s, unsigned &T, unsigned cand, float m, float target) {
  if (__builtin_amdgcn_readfirstlane(m >= target)) {  // uniform: every thread has the same sum
    T = s.lower = cand;
  } else {
    s.upper = cand;
    s.above = m;
  }
}

// RC: rows compiled in (>= R); 52 rows cover vocabularies up to 53248 without register spills
template <int RC>
__global__ __launch_bounds__(1024) void k_sample_top_p(const float *logits, int V, float inv_temp, float top_p,
                                                       const float *u, int32_t *tokens, int32_t *tokens2, SampleScratch sc) {
  __shared__ float sh[16], wmass[16], mass_at[3][16], sums[2][16];
  __shared__ int wcount[2][16];
  __shared__ float cand_p[SAMPLE_CAND + SAMPLE_CAND / 16];  // candidates of the short cut, ascending token index (cand_at)
  __shared__ int cand_i[SAMPLE_CAND];
  __shared__ SampleExchange ex;
  __shared__ float rows[RC * 64];  // the rows of the one wave that walks its range
  __shared__ int last_in, hit_tok;
  __shared__ unsigned threshold;
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int R = (V + 1023) / 1024, base = wave * R * 64 + lane;
  const float *z = logits + (long)b * V;
  SampleBounds s{1u, 1u << 30, 0.f};  // upper 2: p <= 1
  // (1 - top_p) total / (2 V): all tokens below it together hold less than half of the mass that may be left out (the
  // other half covers rounding, except where top_p is so close to 1 that the bound keeps everything anyway)
  auto left_out = [&](float total) { return max(__float_as_uint((1.0f - top_p) * total / (2.0f * (float)V)), 1u); };  // 0 = absent or underflowed
  float mx = -3.0e38f, target = 0.f;
  bool known = false;  // (uniform) mx, target and s from the first pass
  if constexpr (RC <= 52) if (sc.chunks) {  // the first pass's candidates, if they hold the target mass
    constexpr int NK = (SAMPLE_CHUNK_CAND + 1023) / 1024;
    __shared__ int kw[NK][16];
    // lane 16 r + c of every wave holds chunk c: no barrier
    const int c16 = lane & 15;
    const bool have = c16 < sc.chunks;
    const long part = (long)b * sc.chunks + c16;
    const float cm = have ? sc.max_mass[3 * part] : -3.0e38f, cs = have ? sc.max_mass[3 * part + 1] : 0.f, cb = have ? sc.max_mass[3 * part + 2] : 0.f;
    int n = have ? sc.count[part] : 0;
    if (n > sc.cap) n = SAMPLE_CHUNK_CAND + 1;  // not listed: none of this
    for (int off = 1; off < 16; off <<= 1) {
      const int t = __shfl_up(n, off, 16);
      if (c16 >= off) n += t;
    }
    const int N = __builtin_amdgcn_readlane(n, 15);
    const float M = row_max_f(cm), e = expf(cm - M), total = row_sum_f(cs * e);
    float beta = row_max_f(cb * e);
    mx = M;
    target = top_p * total;
    known = true;
    s.lower = left_out(total);
    if (N <= SAMPLE_CHUNK_CAND) {
      // every token of the row at or above beta (and 1 % for rounding) is among the candidates
      beta = fmaxf(1.01f * beta, 0x1p-40f);
      const float bound[3] = {fmaxf(0x1p-5f, beta), fmaxf(0x1p-10f, beta), beta};
      float pc[NK], q[3] = {};
      int ic[NK];
#pragma unroll
      for (int k = 0; k < NK; ++k) {
        const int i = tid + 1024 * k;
        pc[k] = 0;
        ic[k] = 0;
        if (i < N) {
          int c = 0, first = 0;
#pragma unroll
          for (int j = 1; j < 16; ++j) {  // the chunk whose candidates start at or before i (the last of equal starts: empty ones)
            const int start = __builtin_amdgcn_readlane(n, j - 1);
            if (i >= start) { c = j; first = start; }
          }
          const long at = ((long)b * sc.chunks + c) * sc.cap + (i - first);
          pc[k] = expf(sc.z[at] - M);
          ic[k] = sc.idx[at];
        }
#pragma unroll
        for (int j = 0; j < 3; ++j) q[j] += pc[k] >= bound[j] ? pc[k] : 0.f;
      }
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        q[j] = wave_sum_f(q[j]);
        if (lane == 0) mass_at[j][wave] = q[j];
      }
#pragma unroll
      for (int k = 0; k < NK; ++k) {  // how many candidates of each wave reach each bound, 10 bits each (64 at most)
        int c = 0;
#pragma unroll
        for (int j = 0; j < 3; ++j) c += __popcll(__ballot(pc[k] >= bound[j])) << (10 * j);
        if (lane == 0) kw[k][wave] = c;
      }
      __syncthreads();
      // the highest bound whose upper set has the target mass, and the next one above it, which has not
      int at_bound = -1;
      s.upper = 1u << 30;
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        const float sum = row_sum_f(mass_at[j][lane & 15]);
        if (at_bound >= 0) continue;
        if (sum >= target) {
          at_bound = j;
          s.lower = __float_as_uint(bound[j]);
        } else {
          s.upper = __float_as_uint(bound[j]);
          s.above = sum;
        }
      }
      at_bound = __builtin_amdgcn_readfirstlane(at_bound);  // uniform: every thread has the same sums
      if (at_bound >= 0) {
        int C = 0;
#pragma unroll
        for (int k = 0; k < NK; ++k) {
          const int c = (kw[k][lane & 15] >> (10 * at_bound)) & 1023;
          int at = C + row_sum_i((lane & 15) < wave ? c : 0);
          C += row_sum_i(c);
          const bool in = __float_as_uint(pc[k]) >= s.lower;
          at += __popcll(__ballot(in) & ((1ull << lane) - 1ull));
          if (in) {
            cand_p[cand_at(at)] = pc[k];
            cand_i[at] = ic[k];
          }
        }
        C = __builtin_amdgcn_readfirstlane(C);
        __syncthreads();
        sample_rest(cand_p, cand_i, C, __builtin_amdgcn_readfirstlane(s.lower), __builtin_amdgcn_readfirstlane(s.upper), target, u, b, tokens, tokens2, ex);
        return;
      }
    }
  }
  float p[RC];
#pragma unroll
  for (int i = 0; i < RC; ++i) p[i] = (i < R && base + 64 * i < V) ? z[base + 64 * i] * inv_temp : -3.0e38f;  // sentinel: no such token
  if (tid == 0) { last_in = -1; hit_tok = -1; }
  if (known) {
#pragma unroll
    for (int i = 0; i < RC; ++i) p[i] = p[i] > -1.0e38f ? expf(p[i] - mx) : 0.f;
  } else {
#pragma unroll
    for (int i = 0; i < RC; ++i) mx = fmaxf(mx, p[i]);
    mx = wave_max(mx);
    if (lane == 0) sh[wave] = mx;
    __syncthreads();
    mx = sh[0];
    for (int w = 1; w < 16; ++w) mx = fmaxf(mx, sh[w]);
    // Masses of all tokens and of those at or above 2^-5 and 2^-10 of the most likely one, in one pass.
    constexpr int NQ = 3;
    float q[NQ] = {};
#pragma unroll
    for (int i = 0; i < RC; ++i) {
      p[i] = p[i] > -1.0e38f ? expf(p[i] - mx) : 0.f;
      q[0] += p[i];
#pragma unroll
      for (int j = 1; j < NQ; ++j) q[j] += p[i] >= __uint_as_float((127u - 5u * j) << 23) ? p[i] : 0.f;
    }
#pragma unroll
    for (int j = 0; j < NQ; ++j) {
      q[j] = wave_sum_f(q[j]);
      if (lane == 0) mass_at[j][wave] = q[j];
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < NQ; ++j) {
      q[j] = row_sum_f(mass_at[j][lane & 15]);  // added up as the search adds: with top_p 1, target is a sum it can reach
    }
    target = top_p * q[0];
    // the threshold lies at or above the larger of the two bounds whose upper set already has the target mass
    s.lower = left_out(q[0]);
#pragma unroll
    for (int j = NQ - 1; j > 0; --j)
      if (q[j] >= target) s.lower = (127u - 5u * j) << 23;
#pragma unroll
    for (int j = 1; j < NQ; ++j)
      if (q[j] < target) { s.upper = (127u - 5u * j) << 23; s.above = q[j]; }
  }
  s.lower = __builtin_amdgcn_readfirstlane(s.lower);
  s.upper = __builtin_amdgcn_readfirstlane(s.upper);

  // The threshold is found bit by bit on the float bit pattern, from the top; trials outside [lower, upper) need no sum.
  // Before the first round, after the exponent and after three and six more bits the tokens that still matter are counted.
  // If at most 4096 are at or above `lower` they are compacted in index order and one wave (up to 1024) or four finish the
  // row: no more passes over the vocabulary, and sums that need no workgroup barrier, or one of four waves.  Else, if at
  // most 1024 lie in [lower, upper), one wave searches those alone (the mass at or above `upper` is known).  With the
  // first count only, a nucleus of more than the bounds above hold took 30 rounds over the whole row: 50272 tokens, 32
  // rows, top_p 0.95, us of this kernel: logits of standard deviation 4.8 (a nucleus of some hundreds) 76 -> 14, of 1.6
  // 78 -> 57; at temperature 0.3, top_p 0.7 (the paper's setting) and a deviation of 1.6 11.8 -> 10.3.
  unsigned T = 0;
  int set = 0;
  auto wg_sum = [&](float m) {  // the same value in every thread, one barrier: a set is written again two sums later
    m = wave_sum_f(m);
    set ^= 1;
    if (lane == 0) sums[set][wave] = m;
    __syncthreads();
    return row_sum_f(sums[set][lane & 15]);
  };
  int bit = 29, few = -1;  // few: candidates, if they are few enough to be finished by one or four waves
#pragma unroll 1
  for (int stage = 0;; ++stage) {
    int cnt = 0, mid = 0;  // per lane first (a ballot per row here would be kept for the compaction below: 2 SGPRs per row)
    const unsigned below = s.lower - 1u;  // lower >= 1
#pragma unroll
    for (int i = 0; i < RC; ++i) cnt += (__float_as_uint(p[i]) > below) ? 1 : 0;  // non-negative floats order like their bits
    if (stage) {
#pragma unroll
      for (int i = 0; i < RC; ++i) mid += (__float_as_uint(p[i]) >= s.upper) ? 1 : 0;
      mid = cnt - mid;
      __syncthreads();  // wcount has been read
    }
    const int lane_mid = mid;
    cnt = wave_sum_i(cnt);
    mid = wave_sum_i(mid);
    if (lane == 0) {
      wcount[0][wave] = cnt;
      wcount[1][wave] = mid;
    }
    __syncthreads();
    // uniform over the workgroup, and said so: as a divergent branch it would keep the 52-64 probabilities of the
    // other path alive in registers next to this path's candidates
    const int c0 = wcount[0][lane & 15], c1 = wcount[1][lane & 15];
    const int C = __builtin_amdgcn_readfirstlane(row_sum_i(c0)), n = __builtin_amdgcn_readfirstlane(row_sum_i(c1));
    const int wbase = __builtin_amdgcn_readfirstlane(row_sum_i((lane & 15) < wave ? c0 : 0)), nbase = row_sum_i((lane & 15) < wave ? c1 : 0);
    if (C <= SAMPLE_CAND) {
      int pos = wbase, first = base;
      asm volatile("" : "+v"(first));  // the rows' token indices are made here, not kept in registers from before the loop
#pragma unroll
      for (int i = 0; i < RC; ++i) {
        // (the counting loop tests "> lower - 1", this one ">= lower": the same test, but the compiler recomputes it
        // here instead of keeping one lane mask per row from there)
        const bool c = __float_as_uint(p[i]) >= s.lower;
        const unsigned long long m = __ballot(c);
        if (m) {  // most rows have none
          if (c) {
            const int k = pos + __popcll(m & ((1ull << lane) - 1ull));
            cand_p[cand_at(k)] = p[i];
            cand_i[k] = first + 64 * i;
          }
          pos += __popcll(m);
        }
        __builtin_amdgcn_sched_barrier(0);  // row by row: hoisted, the rows' lane masks would need 2 SGPRs each
      }
      few = C;
      break;
    }
    if (stage && n <= SAMPLE_MID) {
      const float above = s.above;
      float *val = cand_p;  // in any order that is the same every time: a lane's values side by side
      int inc = lane_mid;
      for (int off = 1; off < 64; off <<= 1) {
        const int t = __shfl_up(inc, off);
        if (lane >= off) inc += t;
      }
      int pos = nbase + inc - lane_mid;
#pragma unroll
      for (int i = 0; i < RC; ++i) {
        const unsigned v = __float_as_uint(p[i]);
        if (v >= s.lower && v < s.upper) val[pos++] = p[i];
      }
      __syncthreads();
      if (__builtin_amdgcn_readfirstlane(wave) == 0) {
        float v[SAMPLE_MID / 64];
#pragma unroll
        for (int k = 0; k < SAMPLE_MID / 64; ++k) v[k] = lane + 64 * k < n ? val[lane + 64 * k] : 0.f;
#pragma unroll 1
        for (; bit >= 0; --bit) {
          const unsigned cand = T | (1u << bit);
          if (cand >= s.upper) continue;
          if (cand <= s.lower) { T = cand; continue; }
          float m = 0;
#pragma unroll
          for (int k = 0; k < SAMPLE_MID / 64; ++k) m += (__float_as_uint(v[k]) >= cand) ? v[k] : 0.f;
          sample_decide(s, T, cand, above + wave_sum_f(m), target);
        }
        if (lane == 0) threshold = T;
      }
      __syncthreads();
      T = threshold;
      break;
    }
    const int stop = stage < 3 ? 23 - 3 * stage : 0;
#pragma unroll 1
    for (; bit >= stop; --bit) {
      const unsigned cand = T | (1u << bit);
      if (cand >= s.upper) continue;
      if (cand <= s.lower) { T = cand; continue; }
      float m = 0;
#pragma unroll
      for (int i = 0; i < RC; ++i) m += (__float_as_uint(p[i]) >= cand) ? p[i] : 0.f;  // absent tokens hold zeros
      sample_decide(s, T, cand, wg_sum(m), target);
    }
    if (bit < 0) break;
  }
  if (few >= 0) {
    __syncthreads();
    sample_rest(cand_p, cand_i, few, s.lower, s.upper, target, u, b, tokens, tokens2, ex);
    return;
  }
  // nucleus: zero everything else; mass per wave (each wave owns a contiguous index range)
  float loc = 0;
  int last = -1;
#pragma unroll
  for (int i = 0; i < RC; ++i) {
    if (__float_as_uint(p[i]) < T) p[i] = 0.f;
    loc += p[i];
    if (p[i] > 0.f) last = base + 64 * i;
  }
  loc = wave_sum_f(loc);
  if (lane == 0) wmass[wave] = loc;
  if (last >= 0) atomicMax(&last_in, last);
  __syncthreads();
  float mass = 0, before = 0;
  for (int w = 0; w < 16; ++w) {
    if (w < wave) before += wmass[w];
    mass += wmass[w];
  }
  const float goal = u[b] * mass;
  // the wave whose range contains the crossing walks its rows in index order
  const bool mine = before <= goal && before + wmass[wave] > goal;  // at most one wave: the prefix sums are monotone
  if (mine) {
#pragma unroll
    for (int i = 0; i < RC; ++i) rows[i * 64 + lane] = p[i];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    // lane i adds row i up, from its own column on (no bank conflicts); the first row that takes the running sum past the
    // goal, then the first token of that row
    float row = 0;
    if (lane < R)
      for (int k = 0; k < 64; ++k) row += rows[lane * 64 + ((lane + k) & 63)];
    auto prefix = [&](float v) {  // inclusive, over the lanes
      for (int off = 1; off < 64; off <<= 1) {
        const float t = __shfl_up(v, off);
        if (lane >= off) v += t;
      }
      return v;
    };
    const float run = before + prefix(row);
    int tok = -1;
    const unsigned long long past = __ballot(row > 0.f && run > goal);
    if (past) {
      const int i = (int)__builtin_ctzll(past);
      const float start = i ? __shfl(run, i - 1) : before, pi = rows[i * 64 + lane];
      const float in = start + prefix(pi);
      const unsigned long long over = __ballot(pi > 0.f && in > goal), have = __ballot(pi > 0.f);
      // rounding between the two summation orders: the row's last member
      tok = wave * R * 64 + 64 * i + (over ? (int)__builtin_ctzll(over) : 63 - (int)__builtin_clzll(have));
    }
    if (tok < 0) {  // rounding between the two summation orders: the last member of this wave's range
      int wl = last;
      for (int o = 32; o > 0; o >>= 1) wl = max(wl, __shfl_xor(wl, o));
      tok = wl;
    }
    if (lane == 0) hit_tok = tok;
  }
  __syncthreads();
  if (tid == 0) {
    const int tok = hit_tok >= 0 ? hit_tok : last_in;  // rounding at the very end: last member
    tokens[b] = tok;
    if (tokens2) tokens2[b] = tok;
  }
}

// Chunks of the first pass, 0 without one: up to 8192 tokens (8 per thread) a second launch costs more than it saves;
// above 53248 the second pass has no registers left for it.
int sample_chunks(int V) { return V > 8192 && V <= 53248 ? (V + SAMPLE_CHUNK - 1) / SAMPLE_CHUNK : 0; }

int sample_top_p(hipStream_t s, const float *logits, int B, int V, float temperature, float top_p, const float *u,
                 int32_t *tokens, int32_t *tokens2, SampleScratch sc) {
  if (V > 1024 * SAMPLE_C) return -1;
  const int R = (V + 1023) / 1024;
  const float it = 1.0f / temperature;
  // (top_p 1: the nucleus is all the tokens whose mass does not get lost in rounding, more than the first pass lists)
  sc.chunks = sc.z && top_p < 1.0f ? sample_chunks(V) : 0;
  sc.cap = sc.chunks ? SAMPLE_CHUNK_CAND / sc.chunks : 0;
  sc.first = top_p > 0.97f ? 10 : 4;
  // 8 waves per chunk while all of them fit the chip at once (32 waves on each of 256 CUs), else 4: 50272 tokens, 8, 32 and
  // 128 rows, us: 6.6, 7.6, 16.1 with 8 waves, 9.7, 9.7, 15.3 with 4
  if (sc.chunks && sc.chunks * B <= 1024) SKD_LAUNCH(k_sample_chunk<8>, dim3(sc.chunks, B), dim3(512), 0, s, logits, V, it, sc);
  else if (sc.chunks) SKD_LAUNCH(k_sample_chunk<4>, dim3(sc.chunks, B), dim3(256), 0, s, logits, V, it, sc);
  if (R <= 16) SKD_LAUNCH(k_sample_top_p<16>, dim3(B), dim3(1024), 0, s, logits, V, it, top_p, u, tokens, tokens2, sc);
  else if (R <= 32) SKD_LAUNCH(k_sample_top_p<32>, dim3(B), dim3(1024), 0, s, logits, V, it, top_p, u, tokens, tokens2, sc);
  else if (R <= 52) SKD_LAUNCH(k_sample_top_p<52>, dim3(B), dim3(1024), 0, s, logits, V, it, top_p, u, tokens, tokens2, sc);
  else SKD_LAUNCH(k_sample_top_p<SAMPLE_C>, dim3(B), dim3(1024), 0, s, logits, V, it, top_p, u, tokens, tokens2, sc);
  return 0;
}

void f32_embed(hipStream_t s, float *x, const float *tok_emb, const float *pos_emb, const int32_t *tokens,
               const int32_t *start, int t, int B, int d, int V) {
  SKD_LAUNCH(k_f32_embed, dim3(B), dim3(256), 0, s, x, tok_emb, pos_emb, tokens, start, t, d, V);
}
void f32_layernorm(hipStream_t s, const float *x, const float *g, const float *b, float *out, int B, int d) {
  SKD_LAUNCH(k_f32_layernorm, dim3(B), dim3(256), 0, s, x, g, b, out, d);
}
void f32_linear(hipStream_t s, const float *W, const float *bias, const float *in, float *out, int B, int K, int N,
                int relu, int accumulate) {
  SKD_LAUNCH(k_f32_linear, dim3((N + 3) / 4, B), dim3(256), 0, s, W, bias, in, out, K, N, relu, accumulate);
}
void f32_kv_write(hipStream_t s, const float *qkv, float *pool, const int32_t *bt_layer, int t, int B, KvGeom g) {
  SKD_LAUNCH(k_f32_kv_write, dim3(B), dim3(256), 0, s, qkv, pool, bt_layer, t, g);
}
void f32_attention(hipStream_t s, const float *qkv, const float *pool, const int32_t *bt_layer, const int32_t *start,
                   int t, float *o, float *scores, int score_stride, int B, KvGeom g) {
  SKD_LAUNCH(k_f32_attention, dim3(B * g.H), dim3(64), 0, s, qkv, pool, bt_layer, start, t, o, scores,
                     score_stride, g);
}
void f32_argmax(hipStream_t s, const float *logits, int32_t *tokens, int B, int V) {
  SKD_LAUNCH(k_f32_argmax, dim3(B), dim3(256), 0, s, logits, tokens, V);
}

// ------------------------------------------------------------------ KV debug hooks (fp32 pages)
__global__ void k_kv_load_f32(const float *K, const float *V, float *pool, const int32_t *bt_layer, int cols,
                              KvGeom g) {
  const int b = blockIdx.y, j = blockIdx.x, d = g.H * g.dh;
  const int32_t *bt_row = bt_layer + (long)b * g.max_pages;
  float *Kd = pool + f32_kv_off(bt_row, j, 0, g), *Vd = pool + f32_kv_off(bt_row, j, 1, g);
  for (int k = threadIdx.x; k < d; k += blockDim.x) {
    Kd[k] = K ? K[((long)b * cols + j) * d + k] : 0.f;
    Vd[k] = V ? V[((long)b * cols + j) * d + k] : 0.f;
  }
}
__global__ void k_kv_read_f32(const float *pool, const int32_t *bt_row, float *K, float *V, KvGeom g) {
  const int j = blockIdx.x, d = g.H * g.dh;
  for (int k = threadIdx.x; k < d; k += blockDim.x) {
    K[(long)j * d + k] = pool[f32_kv_off(bt_row, j, 0, g) + k];
    V[(long)j * d + k] = pool[f32_kv_off(bt_row, j, 1, g) + k];
  }
}
void kv_load_f32(hipStream_t s, const float *K, const float *V, float *pool, const int32_t *bt_layer, int cols, int B,
                 KvGeom g) {
  if (cols > 0) SKD_LAUNCH(k_kv_load_f32, dim3(cols, B), dim3(256), 0, s, K, V, pool, bt_layer, cols, g);
}
void kv_read_f32(hipStream_t s, const float *pool, const int32_t *bt_row, int len, float *K, float *V, KvGeom g) {
  if (len > 0) SKD_LAUNCH(k_kv_read_f32, dim3(len), dim3(256), 0, s, pool, bt_row, K, V, g);
}

}  // namespace skd
