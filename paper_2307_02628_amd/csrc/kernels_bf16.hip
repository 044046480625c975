// bf16 production kernels for gfx950 (CDNA4, wave64).
//
// Decode at batch sizes 8..128 is a weight- and KV-streaming problem: every
// projection reads its whole weight matrix once per step and every attention
// head reads its whole KV history once per step, with O(batch) flops per byte.
// The kernels are therefore organised around 16-byte-per-lane, fully coalesced
// streams that land directly in the register layout of
// v_mfma_f32_16x16x32_bf16 (no LDS round trip for streamed data):
//   * weights are stored "fragment-major" (see skd_kernels.h) so one
//     wave-wide load = one 16x32 MFMA A-operand;
//   * activations are kept in 16-row x 32-column tiles, row-major inside the
//     tile: one tile is one 1 KiB B-operand load, and a producer that owns a
//     row stores whole 32-byte sectors;
//   * K is stored per 16-key tile as A-operand fragments (keys x head_dim),
//     V per 32-key block as A-operand fragments of V^T (head_dim x keys) with
//     the key order inside a block chosen so that the softmax weights leave
//     the QK^T accumulator already in B-operand position.
#include "bf16_device.h"

namespace skd {

// one barrier: `sh` (16 floats) must not have been read since the last barrier of the block
__device__ inline float block_sum_once(float v, float *sh) {
  v = wave_sum_f(v);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  float r = 0;
  for (unsigned w = 0; w < (blockDim.x >> 6); ++w) r += sh[w];
  return r;
}

// ------------------------------------------------------------------ skinny GEMM
// C[b][n] = sum_k A[b][k] * W[n][k], batch on the MFMA column side.
// Workgroup = 4 or 8 waves that share the same 16*R weight rows and interleave
// the workgroup's K range among themselves; grid.y splits K further across
// workgroups.  Each wave streams R weight-fragment rows and MB activation
// fragments per 32-wide k-step through two register buffers of U k-steps.
// What an epilogue reads from global memory (bias, residual, page index) is
// fetched ahead of the cross-wave reduction, so the end of the kernel is not a
// chain of dependent round trips.
struct EpiPre {
  floatx4 bias, x;
  int page, slot;
};
template <int EPI>
__device__ inline EpiPre epi_prefetch(const GemmArgs &a, int row, int n0) {
  EpiPre p;
  p.bias = p.x = floatx4{0.f, 0.f, 0.f, 0.f};
  p.page = 0;
  p.slot = 0;
  if constexpr (EPI == EPI_QKV || EPI == EPI_RELU || EPI == EPI_QKV_ROWS || EPI == EPI_RESID) {
    if (n0 + 3 < a.N) p.bias = *(const floatx4 *)&a.bias[n0];  // N is a multiple of 4 for these
  }
  if constexpr (EPI == EPI_QKV_ROWS) {
    p.page = -1;
    if (n0 >= a.d && n0 < a.N && row < a.rows) {
      const int b = a.rm.seq[row];
      if (b >= 0) {
        const int slot = row - a.rm.first_row[b];  // = real position: keys are stored by real position
        if (slot < a.rm.P - a.rm.start[b]) {       // else padding of the sequence's last 16-row tile
          p.page = a.bt_layer[(long)b * a.kv.max_pages + slot / a.kv.page_tokens];
          p.slot = slot;
        }
      }
    }
  }
  if constexpr (EPI == EPI_RESID) {
    if (n0 + 3 < a.N && row < a.rows) p.x = *(const floatx4 *)&a.x[(long)row * a.N + n0];
  }
  return p;
}

template <int EPI>
__device__ inline void gemm_epilogue(const GemmArgs &a, int b, int n0, floatx4 v, const EpiPre &pre);

template <>
__device__ inline void gemm_epilogue<EPI_PARTIAL>(const GemmArgs &a, int b, int n0, floatx4 v, const EpiPre &) {
  if (n0 + 3 < a.N) {
    *(floatx4 *)&a.partial[((long)blockIdx.y * a.B_pad + b) * a.N + n0] = v;
  }
}

template <>
__device__ inline void gemm_epilogue<EPI_QKV>(const GemmArgs &a, int b, int n0, floatx4 v, const EpiPre &pre) {
  if (n0 >= a.N) return;
  v += pre.bias;
  const int which = n0 / a.d, within = n0 - which * a.d;
  if (which == 0) {
    uint2 pk = make_uint2(pack2(v[0], v[1]), pack2(v[2], v[3]));
    *(uint2 *)&a.q_out[(long)b * a.d + within] = pk;
    return;
  }
  // k and v of the new position: row-major staging [B][k | v][d]; the attention kernel that follows
  // files them into the KV page while it streams the cache (scattered 2- and 8-byte stores at the end of this
  // kernel cost 3 us per layer)
  if (b >= a.B) return;
  uint2 pk = make_uint2(pack2(v[0], v[1]), pack2(v[2], v[3]));
  *(uint2 *)&a.kv_new[((long)b * 2 + (which - 1)) * a.d + within] = pk;
}

template <>
__device__ inline void gemm_epilogue<EPI_RELU>(const GemmArgs &a, int b, int n0, floatx4 v, const EpiPre &pre) {
  if (n0 >= a.N) return;
  for (int i = 0; i < 4; ++i) v[i] = fmaxf(v[i] + pre.bias[i], 0.f);
  uint2 pk = make_uint2(pack2(v[0], v[1]), pack2(v[2], v[3]));
  *(uint2 *)&a.act_out[d_act_index(b, n0, a.N)] = pk;
}

// tile rows that fit the 64 KiB cross-wave reduction buffer at once (each tile row = WAVES * MB KiB)
constexpr int gemm_stage_rows(int waves, int R, int MB) {
  const int fit = 64 / (waves * MB);
  return fit >= R ? R : (fit > 0 ? fit : 1);
}

template <>
__device__ inline void gemm_epilogue<EPI_QKV_ROWS>(const GemmArgs &a, int row, int n0, floatx4 v, const EpiPre &pre) {
  if (n0 >= a.N || row >= a.rows) return;
  v += pre.bias;
  const int which = n0 / a.d, within = n0 - which * a.d;
  const uint2 pk = make_uint2(pack2(v[0], v[1]), pack2(v[2], v[3]));
  if (which == 0) {
    *(uint2 *)&a.q_out[d_act_index(row, within, a.d)] = pk;
    return;
  }
  if (pre.page < 0) return;  // padding row
  const int h = within / a.kv.dh, e = within - h * a.kv.dh;
  bf16_t *pg = a.kv_pool + (long)pre.page * a.kv.page_elems;
  const int tt = pre.slot % a.kv.page_tokens;
  if (which == 1) {
    *(uint2 *)&pg[kv_k_off(h, tt, e, a.kv)] = pk;
  } else {
    for (int i = 0; i < 4; ++i) pg[kv_v_off(h, tt, e + i, a.kv)] = (bf16_t)f2bf(v[i]);
  }
}

template <>
__device__ inline void gemm_epilogue<EPI_RESID>(const GemmArgs &a, int row, int n0, floatx4 v, const EpiPre &pre) {
  if (n0 + 3 >= a.N || row >= a.rows) return;
  *(floatx4 *)&a.x[(long)row * a.N + n0] = pre.x + (v + pre.bias);
}

// With NB > 0 (decode, at most NB <= 4 rows, 8 waves) the activations are not read: the workgroup makes them itself, in
// LDS, from the residual rows and the partial sums of the projection before: x + bias + sums, then LayerNorm.  Every
// workgroup repeats that, workgroup 0 also stores the new residual rows (to another buffer: the others still read the
// old ones).  The first weights are requested before it, so they arrive under it.  For few rows this costs less than
// the reducer's launch (one row of 4096 with two partial sums: 96 KiB from L2 per workgroup, half of it bias, gain and offset).
constexpr int ln_chunks(int NB) { return NB > 2 ? 1 : 2; }  // float4 chunks per thread: rows of 2048 NC at most
constexpr int ln_row_stride(int K) { return K + 32; }  // bf16 units: rows start 16 banks apart
template <int NB, typename F>
__device__ inline void ln_prologue(const GemmArgs &a, bf16_t *act, float *sh, int wave, int lane, F request_weights) {
  constexpr int NC = ln_chunks(NB);
  const int d4 = a.K >> 2, tid = threadIdx.x;
  auto bar = [&]() {  // bare: __syncthreads() would wait for the weights in flight
    __builtin_amdgcn_s_waitcnt(0xC07F);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  // all loads of the rows, then the first weights, then the sums: what is waited for first is requested first
  floatx4 v[NB][NC], p[NB][NC][4], bias[NC], gv[NC], bv[NC];
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    const int c = tid + 512 * i;
    if (c < d4) {
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        const long at = (long)min(b, a.B - 1) * d4 + c;  // rows past the batch repeat the last one
        v[b][i] = ((const floatx4 *)a.ln_x)[at];
#pragma unroll
        for (int sp = 0; sp < 4; ++sp)
          if (sp < a.ln_split) p[b][i][sp] = ((const floatx4 *)a.ln_partial)[(long)sp * a.B_pad * d4 + at];
      }
      bias[i] = ((const floatx4 *)a.ln_bias)[c];
      gv[i] = ((const floatx4 *)a.ln_g)[c];
      bv[i] = ((const floatx4 *)a.ln_b)[c];
    }
  }
  __builtin_amdgcn_sched_barrier(0);
  request_weights();
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    const int c = tid + 512 * i;
    if (c < d4) {
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        const long at = (long)min(b, a.B - 1) * d4 + c;
        floatx4 acc = p[b][i][0];
#pragma unroll
        for (int sp = 1; sp < 4; ++sp)
          if (sp < a.ln_split) acc += p[b][i][sp];
        for (int sp = 4; sp < a.ln_split; ++sp) acc += ((const floatx4 *)a.ln_partial)[(long)sp * a.B_pad * d4 + at];
        v[b][i] += acc + bias[i];
        if (blockIdx.x == 0 && b < a.B) ((floatx4 *)a.ln_x_out)[at] = v[b][i];
      }
    }
  }
  float mean[NB], rstd[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < NC; ++i)
      if (tid + 512 * i < d4) s += (v[b][i][0] + v[b][i][1]) + (v[b][i][2] + v[b][i][3]);
    s = wave_sum_f(s);
    if (lane == 0) sh[b * 8 + wave] = s;
  }
  bar();
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    float s = 0.f;
#pragma unroll
    for (int w = 0; w < 8; ++w) s += sh[b * 8 + w];
    mean[b] = s / a.K;
    float q = 0.f;
#pragma unroll
    for (int i = 0; i < NC; ++i)
      if (tid + 512 * i < d4) {
        const floatx4 t = v[b][i] - mean[b];
        q += (t[0] * t[0] + t[1] * t[1]) + (t[2] * t[2] + t[3] * t[3]);
      }
    q = wave_sum_f(q);
    if (lane == 0) sh[32 + b * 8 + wave] = q;
  }
  bar();
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    float q = 0.f;
#pragma unroll
    for (int w = 0; w < 8; ++w) q += sh[32 + b * 8 + w];
    rstd[b] = 1.0f / sqrtf(q / a.K + 1e-5f);
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      const int c = tid + 512 * i;
      if (c < d4) {
        const floatx4 y = (v[b][i] - mean[b]) * rstd[b] * gv[i] + bv[i];
        *(uint2 *)&act[b * ln_row_stride(a.K) + 4 * c] = make_uint2(pack2(y[0], y[1]), pack2(y[2], y[3]));
      }
    }
  }
  bar();
}

// With NB > 0 and EPI_PARTIAL (the output projection of one or two rows) the activations are the shares of the keys that the
// attention left behind: the workgroup merges the rows of its own K range into LDS, a float4 chunk per thread and row, while
// its first weights are in flight.  The merge's own launch took 4.8 us of a layer.  us per step, separate -> merged here, 4
// layers of 2048 at 2000 keys: 1 row 179 -> 166, 2 rows 192 -> 185; 2 layers of 4096: 199 -> 191, 208 -> 206; three rows of
// 2048 (64 KiB more in every workgroup) were slower, 223 -> 230, and keep the launch.
constexpr int MERGE_SPLITS = 8;
template <int NB, typename F>
__device__ inline void merge_prologue(const GemmArgs &a, bf16_t *act, int kw0, int kw1, F request_weights) {
  const int c0 = 32 * kw0, n4 = 8 * (kw1 - kw0), dh = a.kv.dh, H = a.K / dh, pairs = a.B * H;
  bool first = true;
  for (int i = threadIdx.x; i < n4 || first; i += 512) {
    floatx4 num[NB][MERGE_SPLITS];
    floatx2 ml[NB][MERGE_SPLITS];
    const int c = c0 + 4 * i, h = c / dh, e = c - h * dh;
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int k = 0; k < MERGE_SPLITS; ++k)
        if (i < n4) {
          const float *p = a.attn_part + ((long)(k < a.attn_splits ? k : 0) * pairs + b * H + h) * (dh + 4);
          num[b][k] = *(const floatx4 *)(p + e);
          ml[b][k] = *(const floatx2 *)(p + dh);
        }
    if (first) {
      __builtin_amdgcn_sched_barrier(0);
      request_weights();
      __builtin_amdgcn_sched_barrier(0);
      first = false;
    }
#pragma unroll
    for (int b = 0; b < NB; ++b)
      if (i < n4) {
        float M = ml[b][0][0], den = 0.f;
#pragma unroll
        for (int k = 1; k < MERGE_SPLITS; ++k) M = fmaxf(M, ml[b][k][0]);
        floatx4 v = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < MERGE_SPLITS; ++k) {
          const float g = k < a.attn_splits ? __expf(ml[b][k][0] - M) : 0.f;
          v += num[b][k] * g;
          den += ml[b][k][1] * g;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = den > 0.f ? v[k] / den : 0.f;
        *(uint2 *)&act[b * ln_row_stride(a.K) + c] = make_uint2(pack2(v[0], v[1]), pack2(v[2], v[3]));
      }
  }
  __builtin_amdgcn_s_waitcnt(0xC07F);  // bare barrier: the weights in flight are not waited for
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

template <int R>
struct RowTiles { static constexpr int value = R; };

// tile0: first of the R weight tiles; group: place of this workgroup's (max, argmax) partials (LM head)
template <int MB, int R, int EPI, int U, int WAVES, int NB>
__device__ __forceinline__ void gemm_body(const GemmArgs &a, int tile0, int group) {
  constexpr int RM = R * MB;
  extern __shared__ floatx4 red[];  // [WAVES][RM][64 lanes]
  // The wave index is the same in all lanes.  Saying so makes the loop conditions that depend on it scalar: as
  // (formally) divergent exits they make the compiler shuttle every accumulator between register files in each
  // iteration to keep the values of lanes that might have left the loop.
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int Kf = a.K >> 5;
  // K range of this workgroup, cut into buffers of U k-steps that are dealt
  // round-robin to the waves: at any moment the workgroup reads WAVES * U KiB
  // of consecutive addresses from each of its R weight-row streams.
  const int kw0 = (int)((long)Kf * blockIdx.y / a.split), kw1 = (int)((long)Kf * (blockIdx.y + 1) / a.split);
  const int nbuf = (kw1 - kw0) / U;  // the launcher picks U so that this is exact
  // weight tile T lives in tile group T / G at slot T % G; the G tiles of a group alternate per k-step
  const bf16x8 *Wl = (const bf16x8 *)a.W + lane;
  const long kstride = (long)a.G * 64;
  long woff[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int T = tile0 + r;
    woff[r] = (((long)(T / a.G) * Kf + kw0) * a.G + T % a.G) * 64;
  }
  const int row0 = blockIdx.z * (MB * 16);  // chunk of activation rows (0 when decoding)
  const bf16x8 *Ab = (const bf16x8 *)a.A + ((long)blockIdx.z * MB * Kf + kw0) * 64 + act_lane(lane);

  floatx4 acc[R][MB];
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int m = 0; m < MB; ++m) acc[r][m] = floatx4{0.f, 0.f, 0.f, 0.f};

  bf16x8 w0[U][R], x0[U][MB], w1[U][R], x1[U][MB];
  auto load = [&](int j, bf16x8(&w)[U][R], bf16x8(&x)[U][MB]) {  // j-th buffer of the workgroup
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int r = 0; r < R; ++r) w[u][r] = __builtin_nontemporal_load(&Wl[woff[r] + (long)(j * U + u) * kstride]);
      if constexpr (NB == 0) {
#pragma unroll
        for (int m = 0; m < MB; ++m) x[u][m] = Ab[((long)m * Kf + j * U + u) * 64];
      }
    }
  };
  // NB > 0: rows of the activations in LDS behind the reduction buffer; lanes of rows that do not exist hold zeros
  bf16_t *act = (bf16_t *)(red + WAVES * gemm_stage_rows(WAVES, R, MB) * MB * 64);
  auto fma = [&](int j, bf16x8(&w)[U][R], bf16x8(&x)[U][MB]) {
    if constexpr (NB > 0) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        x[u][0] = bf16x8{0, 0, 0, 0, 0, 0, 0, 0};
        if ((lane & 15) < NB)
          x[u][0] = *(const bf16x8 *)&act[(lane & 15) * ln_row_stride(a.K) + (kw0 + j * U + u) * 32 + 8 * (lane >> 4)];
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int r = 0; r < R; ++r)
#pragma unroll
        for (int m = 0; m < MB; ++m)
          acc[r][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[u][r], x[u][m], acc[r][m], 0, 0, 0);
  };

  // epilogue operands of the (tile row, batch tile) pairs this wave will finish: fetched now when they are few,
  // else at the start of each reduction stage
  constexpr int RS = gemm_stage_rows(WAVES, R, MB);
  constexpr int NP = (RS * MB + WAVES - 1) / WAVES;
  constexpr bool EARLY = RS == R && NP <= 2;
  EpiPre pre[NP];
  auto fetch_pre = [&](int r0) {
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const int p = wave + i * WAVES;
      const int r = r0 + p / MB, m = p % MB;
      if (p < RS * MB && r < R)
        pre[i] = epi_prefetch<EPI>(a, row0 + m * 16 + (lane & 15), (tile0 + r) * 16 + 4 * (lane >> 4));
    }
  };
  if constexpr (EARLY) fetch_pre(0);

  // two register buffers: the loads of one are in flight while the MFMAs of the other issue
  // A wave beyond the last buffer (short K) streams buffer 0 with its weights zeroed, once: guarding the loop instead
  // makes the compiler keep two copies of the accumulators and move all of them between the copies every iteration.
  const bool idle = wave >= nbuf;
  int j = idle ? 0 : wave;
  if constexpr (NB > 0 && EPI == EPI_PARTIAL) merge_prologue<NB>(a, act, kw0, kw1, [&]() { load(j, w0, x0); });
  else if constexpr (NB > 0) ln_prologue<NB>(a, act, (float *)red, wave, lane, [&]() { load(j, w0, x0); });
  else load(j, w0, x0);
  if (idle) {
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int r = 0; r < R; ++r) w0[u][r] = bf16x8{0, 0, 0, 0, 0, 0, 0, 0};
  }
  // Behind the conditional prefetch the compiler cannot count the loads in flight and makes the first MFMA of a
  // buffer wait for the prefetch as well, so a wave alone does not overlap its loads with its MFMAs: the other
  // waves of the CU do.  Measured with the prefetch made unconditional (exact wait counts, twice the bytes in
  // flight per wave): 2 % slower at 32 rows (8 waves per workgroup), faster only at 128 rows (4 waves).
  while (true) {
    const int j1 = j + WAVES, j2 = j + 2 * WAVES;
    if (j1 < nbuf) load(j1, w1, x1);
    fma(j, w0, x0);
    if (j1 >= nbuf) break;
    if (j2 < nbuf) load(j2, w0, x0);
    fma(j1, w1, x1);
    if (j2 >= nbuf) break;
    j = j2;
  }

  // sum the waves' partial tiles in a fixed order (deterministic).  The LDS buffer holds RS of the R tile rows
  // at a time (64 KiB at most), so wide batches reduce in stages.
  constexpr int NST = (R + RS - 1) / RS;
  float cand_v[NST * NP];  // LM head: lanes 0..15 keep the best logit of each (tile row, batch row) they reduced
  int cand_i[NST * NP];
#pragma unroll
  for (int r0 = 0; r0 < R; r0 += RS) {
    if (r0) __syncthreads();  // the previous stage has been consumed
    if constexpr (!EARLY) fetch_pre(r0);
#pragma unroll
    for (int rr = 0; rr < RS; ++rr)
#pragma unroll
      for (int m = 0; m < MB; ++m)
        if (r0 + rr < R) red[(wave * (RS * MB) + rr * MB + m) * 64 + lane] = acc[r0 + rr < R ? r0 + rr : 0][m];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const int p = wave + i * WAVES;
      const int r = r0 + p / MB, m = p % MB;
      if (p < RS * MB && r < R) {
        floatx4 v = red[p * 64 + lane];
        for (int w = 1; w < WAVES; ++w) v += red[(w * (RS * MB) + p) * 64 + lane];
        const int n0 = (tile0 + r) * 16 + 4 * (lane >> 4);
        if constexpr (EPI != EPI_LOGITS) {
          gemm_epilogue<EPI>(a, row0 + m * 16 + (lane & 15), n0, v, pre[i]);
        } else {
          // optional fp32 logits, and the largest of this tile row per batch row (lowest index on ties)
          const int b = m * 16 + (lane & 15);
          float best = -3.0e38f;
          int bi = 0x7fffffff;
          for (int j = 0; j < 4; ++j) {
            if (n0 + j < a.N) {
              if (a.logits && b < a.B) a.logits[(long)b * a.N + n0 + j] = v[j];
              if (v[j] > best) { best = v[j]; bi = n0 + j; }
            }
          }
          for (int o = 16; o < 64; o <<= 1) {  // across the four 4-row groups of this column
            const float ov = __shfl_xor(best, o);
            const int oi = __shfl_xor(bi, o);
            if (ov > best || (ov == best && oi < bi)) { best = ov; bi = oi; }
          }
          cand_v[(r0 / RS) * NP + i] = best;
          cand_i[(r0 / RS) * NP + i] = bi;
        }
      }
    }
  }
  if constexpr (EPI == EPI_LOGITS) {
    __syncthreads();  // the reduction buffer is free: it now collects the candidates, [R * MB][16] values and indices
    float *cv = (float *)red;
    int *ci = (int *)red + RM * 16;
#pragma unroll
    for (int st = 0; st < NST; ++st)
#pragma unroll
      for (int i = 0; i < NP; ++i) {
        const int p = wave + i * WAVES;
        const int r = st * RS + p / MB, m = p % MB;
        if (p < RS * MB && r < R && lane < 16) {
          cv[(r * MB + m) * 16 + lane] = cand_v[st * NP + i];
          ci[(r * MB + m) * 16 + lane] = cand_i[st * NP + i];
        }
      }
    __syncthreads();
    if (threadIdx.x < MB * 16) {
      const int m = threadIdx.x >> 4, c = threadIdx.x & 15;
      float best = cv[m * 16 + c];
      int bi = ci[m * 16 + c];
      for (int r = 1; r < R; ++r) {
        const float ov = cv[(r * MB + m) * 16 + c];
        const int oi = ci[(r * MB + m) * 16 + c];
        if (ov > best || (ov == best && oi < bi)) { best = ov; bi = oi; }
      }
      a.pmax[(long)group * a.B_pad + m * 16 + c] = best;
      a.pidx[(long)group * a.B_pad + m * 16 + c] = bi;
    }
  }
}

// The LM head is several rounds of workgroups, and 16 R rows of a vocabulary of 50272 are 3.07 workgroups per CU: with equal
// ones the last round keeps a few CUs busy for as long as a full one.  So whole rounds get R tiles, what is left of a round
// one size of fewer, and the remainder single tiles (head_tiles; a logit is the same sum whatever group its tile is in).
// us with the argmax, 50272 x 4096, equal groups -> this, 16, 32, 48, 64, 96 and 128 rows: 75 -> 71, 83 -> 77, 92 -> 84,
// 106 -> 97, 130 -> 122, 146 -> 137; 50272 x 2048: 41 -> 40, 47 -> 45, 53 -> 50, 64 -> 59, 78 -> 71, 90 -> 83; 32000 rows are
// 1.95 rounds either way.
template <int R, typename F>
__device__ __forceinline__ void head_dispatch(const GemmArgs &a, F body) {
  const int id = blockIdx.x, mid = id - a.head_full, rest = mid - a.head_mid;
  if (mid < 0) { body(RowTiles<R>{}, id * R); return; }
  const int mid0 = a.head_full * R;
  if (rest >= 0) { body(RowTiles<1>{}, mid0 + a.head_mid * a.head_mid_r + rest); return; }
  if constexpr (R > 3) if (a.head_mid_r == 3) { body(RowTiles<3>{}, mid0 + mid * 3); return; }
  if constexpr (R > 2) body(RowTiles<2>{}, mid0 + mid * 2);
}

template <int MB, int R, int EPI, int U, int WAVES, int NB = 0>
__global__ __launch_bounds__(WAVES * 64) void k_gemm(GemmArgs a) {
  if constexpr (EPI == EPI_LOGITS)
    head_dispatch<R>(a, [&](auto r, int tile0) { gemm_body<MB, decltype(r)::value, EPI, U, WAVES, NB>(a, tile0, blockIdx.x); });
  else
    gemm_body<MB, R, EPI, U, WAVES, NB>(a, blockIdx.x * R, blockIdx.x);
}

int bf16_gemm_groups(int N, int R) { return (N + 16 * R - 1) / (16 * R); }
// Workgroups of the LM head: a.head_full of R tiles, a.head_mid of a.head_mid_r, the rest of one.  slots: workgroups that run
// at once; 0: equal groups.
int bf16_head_tiles(GemmArgs &a, int R, int slots) {
  const int tiles = (a.N + 15) / 16;
  a.head_full = bf16_gemm_groups(a.N, R);
  a.head_mid = a.head_mid_r = 0;
  if (slots <= 0 || tiles <= R * slots) return a.head_full;
  a.head_full = tiles / (R * slots) * slots;
  int rest = tiles - a.head_full * R;
  int r = rest / slots;
  const bool whole = rest - r * slots <= slots / 2;  // a round of r and a few single tiles, or a round of r + 1 that is not full
  if (!whole) ++r;
  if (r >= R) {
    a.head_full += rest / R;
    rest %= R;
  } else if (r > 1) {  // (one tile each: the last sort)
    a.head_mid_r = r;
    a.head_mid = whole ? slots : rest / r;
    rest -= r * a.head_mid;
  }
  return a.head_full + a.head_mid + rest;
}

template <int MB, int R, int U, int WAVES>
static void launch_gemm_epi(hipStream_t s, const GemmArgs &a, int epi, dim3 grid) {
  const size_t lds = (size_t)WAVES * gemm_stage_rows(WAVES, R, MB) * MB * 64 * sizeof(floatx4);
  const dim3 blk(WAVES * 64);
  switch (epi) {
    case EPI_PARTIAL: SKD_LAUNCH((k_gemm<MB, R, EPI_PARTIAL, U, WAVES>), grid, blk, lds, s, a); break;
    case EPI_QKV: SKD_LAUNCH((k_gemm<MB, R, EPI_QKV, U, WAVES>), grid, blk, lds, s, a); break;
    case EPI_RELU: SKD_LAUNCH((k_gemm<MB, R, EPI_RELU, U, WAVES>), grid, blk, lds, s, a); break;
    case EPI_QKV_ROWS:
      SKD_LAUNCH((k_gemm<MB, R, EPI_QKV_ROWS, U, WAVES>), grid, blk, lds, s, a);
      break;
    case EPI_RESID:
      if constexpr (MB == 8) SKD_LAUNCH((k_gemm<MB, R, EPI_RESID, U, WAVES>), grid, blk, lds, s, a);
      break;
    default: SKD_LAUNCH((k_gemm<MB, R, EPI_LOGITS, U, WAVES>), grid, blk, lds, s, a); break;
  }
}
template <int MB, int R, int U>
static void launch_gemm_w(hipStream_t s, const GemmArgs &a, int epi, int waves, dim3 grid) {
  // 6 and 8 batch tiles need 4-wave workgroups: with 8 waves (2 per SIMD, 256 registers each) the accumulators spill
  if constexpr (MB < 6) {
    if (waves >= 8) { launch_gemm_epi<MB, R, U, 8>(s, a, epi, grid); return; }
  }
  launch_gemm_epi<MB, R, U, 4>(s, a, epi, grid);
}
template <int MB, int R>
static void launch_gemm_u(hipStream_t s, const GemmArgs &a, int epi, int U, int waves, dim3 grid) {
  // register budget: R * MB accumulators plus two buffers of U * (R + MB) fragments, 4 VGPRs each (beyond 44
  // units the 8-wave instantiations spill)
  if constexpr (R * MB + 2 * 4 * (R + MB) <= 44) {
    if (U >= 4) { launch_gemm_w<MB, R, 4>(s, a, epi, waves, grid); return; }
  }
  if constexpr (R * MB + 2 * 2 * (R + MB) <= 44) {
    if (U >= 2) { launch_gemm_w<MB, R, 2>(s, a, epi, waves, grid); return; }
  }
  launch_gemm_w<MB, R, 1>(s, a, epi, waves, grid);
}
template <int MB>
static void launch_gemm_r(hipStream_t s, const GemmArgs &a, int epi, int R, int U, int waves, dim3 grid) {
  if (R == 1) launch_gemm_u<MB, 1>(s, a, epi, U, waves, grid);
  else if (R == 2) launch_gemm_u<MB, 2>(s, a, epi, U, waves, grid);
  else if (R == 3) launch_gemm_u<MB, 3>(s, a, epi, U, waves, grid);
  else launch_gemm_u<MB, 4>(s, a, epi, U, waves, grid);
}

// Decode projections of at most 4 rows with the reducer's work in their prologue (a.ln_*; see k_gemm).
template <int R, int EPI>
static int launch_gemm_ln(hipStream_t s, const GemmArgs &a, dim3 grid) {
  const int NB = a.B <= 1 ? 1 : a.B <= 2 ? 2 : 4;
  const size_t lds = (size_t)8 * R * 64 * sizeof(floatx4) + (size_t)NB * ln_row_stride(a.K) * sizeof(bf16_t);
  const int most = 8 * R * 64 * (int)sizeof(floatx4) + 4 * ln_row_stride(2048) * (int)sizeof(bf16_t);  // more than 2 rows of 4096
  static std::atomic<uint64_t> done{0};
  if (!allow_lds(done, {(const void *)k_gemm<1, R, EPI, 1, 8, 1>,
                        (const void *)k_gemm<1, R, EPI, 1, 8, 2>,
                        (const void *)k_gemm<1, R, EPI, 1, 8, 4>}, most))
    return -1;
  if (NB == 1) SKD_LAUNCH((k_gemm<1, R, EPI, 1, 8, 1>), grid, dim3(512), lds, s, a);
  else if (NB == 2) SKD_LAUNCH((k_gemm<1, R, EPI, 1, 8, 2>), grid, dim3(512), lds, s, a);
  else SKD_LAUNCH((k_gemm<1, R, EPI, 1, 8, 4>), grid, dim3(512), lds, s, a);
  return 0;
}
int bf16_gemm_ln_check(const GemmArgs &a, int epi, int R) {
  if (a.B < 1 || a.B > 4 || a.B_pad != 16 || a.K % 32 || a.K < 32 || a.K > 2048 * ln_chunks(a.B) || a.split != 1 || a.rows != 0)
    return -1;
  if (R < 1 || R > 4 || a.G < 1 || a.G > 4 || a.N < 1 || a.ln_split < 1 || (epi != EPI_QKV && epi != EPI_RELU)) return -1;
  return bf16_gemm_groups(a.N, R);
}
int bf16_gemm_ln(hipStream_t s, const GemmArgs &a, int epi, int R) {
  const int groups = bf16_gemm_ln_check(a, epi, R);
  if (groups < 0) return -1;
  const dim3 grid(groups);
  int rc;
#define SKD_LN(R) (epi == EPI_QKV ? launch_gemm_ln<R, EPI_QKV>(s, a, grid) : launch_gemm_ln<R, EPI_RELU>(s, a, grid))
  if (R == 1) rc = SKD_LN(1);
  else if (R == 2) rc = SKD_LN(2);
  else if (R == 3) rc = SKD_LN(3);
  else rc = SKD_LN(4);
#undef SKD_LN
  return rc < 0 ? -1 : groups;
}

// Every tile of the vocabulary in exactly one group of a size that is compiled; the last group of R may run over the end.
static int bf16_head_groups(const GemmArgs &a) {
  const int tiles = (a.N + 15) / 16, R = a.G;
  const int left = tiles - a.head_full * R - a.head_mid * a.head_mid_r;
  return a.head_full + a.head_mid + (left > 0 ? left : 0);
}
static bool head_shape(const GemmArgs &a, int R) {
  if (a.G != R || a.head_full < 0 || a.head_mid < 0) return false;
  if (a.head_mid && (a.head_mid_r < 2 || a.head_mid_r >= R)) return false;
  const long covered = (long)a.head_full * R + (long)a.head_mid * a.head_mid_r, tiles = (a.N + 15) / 16;
  return covered < tiles + R && (covered <= tiles || a.head_mid == 0);
}

// The output projection of one or two rows with the merge of the attention's shares in its prologue (a.attn_*).
template <int R, int U>
static void launch_gemm_merge(hipStream_t s, const GemmArgs &a, dim3 grid) {
  const size_t lds = (size_t)8 * R * 64 * sizeof(floatx4) + (size_t)a.B * ln_row_stride(a.K) * sizeof(bf16_t);  // 32896 bytes at most: two rows of 4096, two tiles
  if (a.B == 1) SKD_LAUNCH((k_gemm<1, R, EPI_PARTIAL, U, 8, 1>), grid, dim3(512), lds, s, a);
  else SKD_LAUNCH((k_gemm<1, R, EPI_PARTIAL, U, 8, 2>), grid, dim3(512), lds, s, a);
}
int bf16_gemm_merge_check(const GemmArgs &a, int R, int waves) {
  if (a.B < 1 || a.B > 2 || a.B_pad != 16 || a.K % 32 || a.K < 32 || a.K > 4096 || a.rows != 0 || waves != 8) return -1;
  if (R < 1 || R > 2 || a.G < 1 || a.G > 4 || a.N < 1 || a.split < 1 || (a.K / 32) % a.split) return -1;
  if ((a.kv.dh != 64 && a.kv.dh != 128) || a.K % a.kv.dh || a.attn_splits < 2 || a.attn_splits > MERGE_SPLITS) return -1;
  return bf16_gemm_groups(a.N, R);
}
int bf16_gemm_merge(hipStream_t s, const GemmArgs &a, int R, int U, int waves) {
  const int groups = bf16_gemm_merge_check(a, R, waves);
  if (groups < 0) return -1;
  const dim3 grid(groups, a.split);
  if ((a.K / 32 / a.split) % 2) U = 1;  // whole buffers
  if (R == 1) U >= 2 ? launch_gemm_merge<1, 2>(s, a, grid) : launch_gemm_merge<1, 1>(s, a, grid);
  else U >= 2 ? launch_gemm_merge<2, 2>(s, a, grid) : launch_gemm_merge<2, 1>(s, a, grid);
  return groups;
}

// Batch tiles of 16 rows are compiled for B_pad in {16, 32, 48, 64, 96, 128}.
// Launch shape of a skinny GEMM, or false if the kernel cannot run it: nothing is launched here.
static bool gemm_shape(const GemmArgs &a, int epi, int R, int &U, int waves, dim3 &grid, int &groups) {
  const int MB = a.B_pad / 16;
  if (R < 1 || R > 4 || a.G < 1 || a.G > 4 || (waves != 4 && waves != 8)) return false;
  if (a.B_pad % 16 || (MB != 1 && MB != 2 && MB != 3 && MB != 4 && MB != 6 && MB != 8)) return false;
  if (a.K < 32 || a.K % 32 || a.N < 1) return false;
  const int split = epi == EPI_LOGITS ? 1 : a.split;
  const int Kf = a.K / 32;
  if (split < 1 || Kf % split) return false;  // equal K ranges per workgroup
  while (U > 1 && (Kf / split) % U) U >>= 1;  // whole buffers only
  if (U < 1) return false;
  groups = epi == EPI_LOGITS ? bf16_head_groups(a) : bf16_gemm_groups(a.N, R);
  if (epi == EPI_LOGITS && !head_shape(a, R)) return false;
  const bool by_rows = epi == EPI_QKV_ROWS || epi == EPI_RESID || (epi == EPI_RELU && a.rows > 0);
  if (epi == EPI_RESID && MB != 8) return false;
  if ((epi == EPI_QKV_ROWS || epi == EPI_RESID) && a.rows <= 0) return false;
  if (by_rows && (a.rows % a.B_pad || split != 1)) return false;
  grid = dim3(groups, split, by_rows ? a.rows / a.B_pad : 1);
  return true;
}

int bf16_gemm_check(const GemmArgs &a, int epi, int R, int U, int waves) {
  dim3 grid;
  int groups = 0;
  return gemm_shape(a, epi, R, U, waves, grid, groups) ? groups : -1;
}

int bf16_gemm(hipStream_t s, const GemmArgs &a, int epi, int R, int U, int waves) {
  dim3 grid;
  int groups = 0;
  if (!gemm_shape(a, epi, R, U, waves, grid, groups)) return -1;
  switch (a.B_pad / 16) {
    case 1: launch_gemm_r<1>(s, a, epi, R, U, waves, grid); break;
    case 2: launch_gemm_r<2>(s, a, epi, R, U, waves, grid); break;
    case 3: launch_gemm_r<3>(s, a, epi, R, U, waves, grid); break;
    case 4: launch_gemm_r<4>(s, a, epi, R, U, waves, grid); break;
    case 6: launch_gemm_r<6>(s, a, epi, R, U, waves, grid); break;
    default: launch_gemm_r<8>(s, a, epi, R, U, waves, grid); break;
  }
  return groups;
}

// ------------------------------------------------------------------ skinny GEMM for 96 and 128 batch rows
// With 8 batch tiles a workgroup pulls two bytes of activations out of L2 for every byte of weights it streams
// from HBM, and on this part a CU's vector memory path serves the two kinds of request largely one after the
// other: measured per CU with plain streaming waves, 512 KiB of HBM misses take 19.9 us and every further MiB of
// L2 hits adds 7.5 us when separate waves fetch it (12.7 us when the same four waves fetch both in turn, as the
// general kernel above does).  So the work is split by wave role:
//   waves 0..3 (one per SIMD) stream the weights into registers, three k-steps deep, and issue the MFMAs;
//   waves 4..7 fetch the activations with LDS-direct loads (no registers in flight; in the order of staged_piece:
//   in that of act_lane a decode step of the 6.7B shape at 128 rows took 3 % longer) into a ring of four
//   stages; a stage holds the 8 activation fragments of 4 consecutive k-steps; wave 4 + w fetches the k-step
//   that wave w multiplies.  One bare s_barrier per stage orders the ring (as in the tiled prompt GEMM below).
// With a.ws_rot the workgroups start their K range at different stages (and wrap), so that at any moment the
// CUs of an XCD ask its L2 for different lines; the sum over k is then taken in that rotated order: fixed for a
// given launch shape, hence run-to-run deterministic, but not the same order in every workgroup (the caller leaves
// it off for the LM head, where identical vocabulary rows are to give identical logits).
constexpr int WS_NS = 4;  // ring stages
constexpr int WS_CW = 4;  // MFMA waves = loader waves = k-steps per stage
// MB: batch tiles, 6 or 8

template <int MB, int R, int EPI>
__device__ __forceinline__ void gemm_ws_body(const GemmArgs &a, int tile0, int group) {
  constexpr int NS = WS_NS;
  constexpr int STAGE = WS_CW * MB * 64;     // bf16x8 units per stage (24 or 32 KiB)
  extern __shared__ bf16x8 ws_lds[];         // ring [NS][WS_CW][MB][64 lanes]; later the reduction buffer
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int Kf = a.K >> 5;
  const int kw0 = (int)((long)Kf * blockIdx.y / a.split), kw1 = (int)((long)Kf * (blockIdx.y + 1) / a.split);
  const int nchunk = (kw1 - kw0) / WS_CW;  // the launcher makes this exact and >= 1
  const int rot = a.ws_rot ? (int)((blockIdx.x >> 3) * 5u + blockIdx.y * 3u) % nchunk : 0;
  floatx4 *red = (floatx4 *)ws_lds;        // [WS_CW][R * MB][64 lanes] after the main loop
  auto bar = [&]() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };

  if (wave >= WS_CW) {
    // ---- loader of k-step kw0 + 4 * chunk + l of every stage
    const int l = wave - WS_CW;
    const bf16x8 *Ab = (const bf16x8 *)a.A + staged_piece(lane);
    auto issue = [&](int ci) {
      int c = ci + rot;
      if (c >= nchunk) c -= nchunk;
      const long kf = kw0 + c * WS_CW + l;
      bf16x8 *dst = ws_lds + (ci % NS) * STAGE + l * (MB * 64);
#pragma unroll
      for (int m = 0; m < MB; ++m)
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(Ab + ((long)m * Kf + kf) * 64),
                                         (__attribute__((address_space(3))) void *)(dst + m * 64), 16, 0, 0);
    };
#pragma unroll
    for (int i = 0; i < NS - 1; ++i)
      if (i < nchunk) issue(i);
    for (int ci = 0; ci < nchunk; ++ci) {
      // this wave's MB loads of stage ci have landed once only those of the (up to two) later stages in flight
      // are outstanding (vector-memory operations of a wave complete in order)
      const int later = min(nchunk - 1 - ci, NS - 2);
      if (later == 0) wait_vmcnt<0>();
      else if (later == 1) wait_vmcnt<MB>();
      else wait_vmcnt<2 * MB>();
      bar();  // stage ci is complete; every wave has finished reading stage ci - 1
      if (ci + NS - 1 < nchunk) issue(ci + NS - 1);  // into the slot of stage ci - 1
    }
    bar();  // every stage has been read: the ring becomes the reduction buffer
  } else {
    // ---- weight streamer + MFMA: k-step kw0 + 4 * chunk + wave of every stage
    floatx4 acc[R][MB];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int m = 0; m < MB; ++m) acc[r][m] = floatx4{0.f, 0.f, 0.f, 0.f};
    // addresses = wave-uniform base (scalar registers) + the lane's 32-bit offset: no 64-bit vector address
    // arithmetic, no address registers shared with the fragments in flight
    const bf16x8 *Wu = (const bf16x8 *)a.W;
    long wbase[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int T = tile0 + r;
      wbase[r] = (((long)(T / a.G) * Kf + kw0 + wave) * a.G + T % a.G) * 64;
    }
    const long cstride = (long)a.G * 64 * WS_CW;  // one stage further along K
    const unsigned ulane = (unsigned)lane;
    const int xlane = staged_lane(lane);
    auto loadw = [&](int ci, bf16x8(&w)[R]) {
      int c = ci + rot;
      if (c >= nchunk) c -= nchunk;
#pragma unroll
      for (int r = 0; r < R; ++r) w[r] = __builtin_nontemporal_load(&(Wu + (wbase[r] + c * cstride))[ulane]);
    };
    auto step = [&](int ci, bf16x8(&w)[R]) {
      bar();
      const bf16x8 *fs = ws_lds + (ci % NS) * STAGE + wave * (MB * 64) + xlane;
      bf16x8 x[MB];
#pragma unroll
      for (int m = 0; m < MB; ++m) x[m] = fs[m * 64];
#pragma unroll
      for (int r = 0; r < R; ++r)
#pragma unroll
        for (int m = 0; m < MB; ++m) acc[r][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[r], x[m], acc[r][m], 0, 0, 0);
    };
    // three k-steps of weights in flight; the prefetches are unconditional (index clamped to the last stage,
    // which is then fetched again and not used), so that the compiler can count the loads in flight, and fenced
    // so that they stay ahead of the MFMAs they overlap with
    bf16x8 w0[R], w1[R], w2[R];
    const int cl = nchunk - 1;
    loadw(0, w0);
    loadw(min(1, cl), w1);
    // One stage: prefetch the weights two stages ahead into the buffer that came free, then multiply.  Twelve stages
    // per trip of the loop (the three buffers rotate four times): at the loop's head the compiler waits for every
    // load in flight, which costs the prefetch once per trip (measured effect of 12 instead of 3 stages per trip:
    // under 1 %).
#define SKD_WS_STAGE(k, wuse, wload)                     \
  loadw(min(ci + (k) + 2, cl), wload);                   \
  __builtin_amdgcn_sched_barrier(0);                     \
  step(ci + (k), wuse);                                  \
  __builtin_amdgcn_sched_barrier(0);                     \
  if (ci + (k) + 1 >= nchunk) break;
    int ci = 0;
    while (true) {
      SKD_WS_STAGE(0, w0, w2) SKD_WS_STAGE(1, w1, w0) SKD_WS_STAGE(2, w2, w1)
      SKD_WS_STAGE(3, w0, w2) SKD_WS_STAGE(4, w1, w0) SKD_WS_STAGE(5, w2, w1)
      SKD_WS_STAGE(6, w0, w2) SKD_WS_STAGE(7, w1, w0) SKD_WS_STAGE(8, w2, w1)
      SKD_WS_STAGE(9, w0, w2) SKD_WS_STAGE(10, w1, w0) SKD_WS_STAGE(11, w2, w1)
      ci += 12;
    }
#undef SKD_WS_STAGE
    bar();  // all waves are done with the ring
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int m = 0; m < MB; ++m) red[(wave * (R * MB) + r * MB + m) * 64 + lane] = acc[r][m];
  }

  // ---- sum the four MFMA waves' tiles in a fixed order; all eight waves share the epilogue work
  constexpr int NW = 2 * WS_CW;
  constexpr int NP = (R * MB + NW - 1) / NW;
  EpiPre pre[NP];
#pragma unroll
  for (int i = 0; i < NP; ++i) {
    const int p = wave + i * NW;
    if (p < R * MB) pre[i] = epi_prefetch<EPI>(a, (p % MB) * 16 + (lane & 15), (tile0 + p / MB) * 16 + 4 * (lane >> 4));
  }
  __syncthreads();
  float cand_v[NP];
  int cand_i[NP];
#pragma unroll
  for (int i = 0; i < NP; ++i) {
    const int p = wave + i * NW;
    const int r = p / MB, m = p % MB;
    if (p < R * MB) {
      floatx4 v = red[p * 64 + lane];
      for (int w = 1; w < WS_CW; ++w) v += red[(w * (R * MB) + p) * 64 + lane];
      const int n0 = (tile0 + r) * 16 + 4 * (lane >> 4);
      if constexpr (EPI != EPI_LOGITS) {
        gemm_epilogue<EPI>(a, m * 16 + (lane & 15), n0, v, pre[i]);
      } else {
        const int b = m * 16 + (lane & 15);
        float best = -3.0e38f;
        int bi = 0x7fffffff;
        for (int j = 0; j < 4; ++j) {
          if (n0 + j < a.N) {
            if (a.logits && b < a.B) a.logits[(long)b * a.N + n0 + j] = v[j];
            if (v[j] > best) { best = v[j]; bi = n0 + j; }
          }
        }
        for (int o = 16; o < 64; o <<= 1) {
          const float ov = __shfl_xor(best, o);
          const int oi = __shfl_xor(bi, o);
          if (ov > best || (ov == best && oi < bi)) { best = ov; bi = oi; }
        }
        cand_v[i] = best;
        cand_i[i] = bi;
      }
    }
  }
  if constexpr (EPI == EPI_LOGITS) {
    __syncthreads();  // the reduction buffer is free: it now collects the candidates, [R * MB][16] values and indices
    float *cv = (float *)ws_lds;
    int *ci = (int *)ws_lds + R * MB * 16;
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const int p = wave + i * NW;
      if (p < R * MB && lane < 16) {
        cv[p * 16 + lane] = cand_v[i];
        ci[p * 16 + lane] = cand_i[i];
      }
    }
    __syncthreads();
    if (threadIdx.x < MB * 16) {
      const int m = threadIdx.x >> 4, c = threadIdx.x & 15;
      float best = cv[m * 16 + c];
      int bi = ci[m * 16 + c];
      for (int r = 1; r < R; ++r) {
        const float ov = cv[(r * MB + m) * 16 + c];
        const int oi = ci[(r * MB + m) * 16 + c];
        if (ov > best || (ov == best && oi < bi)) { best = ov; bi = oi; }
      }
      a.pmax[(long)group * a.B_pad + m * 16 + c] = best;
      a.pidx[(long)group * a.B_pad + m * 16 + c] = bi;
    }
  }
}

template <int MB, int R, int EPI>
__global__ __launch_bounds__(512) void k_gemm_ws(GemmArgs a) {
  if constexpr (EPI == EPI_LOGITS)
    head_dispatch<R>(a, [&](auto r, int tile0) { gemm_ws_body<MB, decltype(r)::value, EPI>(a, tile0, blockIdx.x); });
  else
    gemm_ws_body<MB, R, EPI>(a, blockIdx.x * R, blockIdx.x);
}

// Decode projections at 96 or 128 (padded) batch rows on the wave-specialised kernel.  Returns the number of row groups,
// or -1 when the shape is not one it handles (the caller then uses bf16_gemm); nothing is launched in that case.
static bool gemm_ws_shape(const GemmArgs &a, int epi, int R, dim3 &grid, int &groups) {
  if ((a.B_pad != 96 && a.B_pad != 128) || a.rows != 0 || R < 1 || R > 4 || a.G < 1 || a.G > 4 || a.K < 32 || a.K % 32 || a.N < 1) return false;
  if (epi != EPI_PARTIAL && epi != EPI_QKV && epi != EPI_RELU && epi != EPI_LOGITS) return false;
  const int split = epi == EPI_LOGITS ? 1 : a.split;
  const int Kf = a.K / 32;
  if (split < 1 || Kf % split || (Kf / split) % WS_CW || Kf / split < WS_CW) return false;
  groups = epi == EPI_LOGITS ? bf16_head_groups(a) : bf16_gemm_groups(a.N, R);
  if (epi == EPI_LOGITS && !head_shape(a, R)) return false;
  grid = dim3(groups, split, 1);
  return true;
}
int bf16_gemm_ws_check(const GemmArgs &a, int epi, int R) {
  dim3 grid;
  int groups = 0;
  return gemm_ws_shape(a, epi, R, grid, groups) ? groups : -1;
}
template <int MB, int R>
static int launch_gemm_ws(hipStream_t s, const GemmArgs &a, int epi, dim3 grid) {
  // the activation ring (4 stages of 4 MB KiB), reused for the cross-wave reduction (4 waves x R x MB KiB): 128 KiB at most
  constexpr size_t ring = (size_t)WS_NS * WS_CW * MB * 64 * sizeof(bf16x8);
  constexpr size_t redb = (size_t)WS_CW * R * MB * 64 * sizeof(floatx4);
  constexpr size_t lds = ring > redb ? ring : redb;
  static std::atomic<uint64_t> done{0};
  if (!allow_lds(done, {(const void *)k_gemm_ws<MB, R, EPI_PARTIAL>,
                        (const void *)k_gemm_ws<MB, R, EPI_QKV>,
                        (const void *)k_gemm_ws<MB, R, EPI_RELU>,
                        (const void *)k_gemm_ws<MB, R, EPI_LOGITS>}, lds))
    return -1;
  const dim3 blk(512);
  switch (epi) {
    case EPI_PARTIAL: SKD_LAUNCH((k_gemm_ws<MB, R, EPI_PARTIAL>), grid, blk, lds, s, a); break;
    case EPI_QKV: SKD_LAUNCH((k_gemm_ws<MB, R, EPI_QKV>), grid, blk, lds, s, a); break;
    case EPI_RELU: SKD_LAUNCH((k_gemm_ws<MB, R, EPI_RELU>), grid, blk, lds, s, a); break;
    default: SKD_LAUNCH((k_gemm_ws<MB, R, EPI_LOGITS>), grid, blk, lds, s, a); break;
  }
  return 0;
}
int bf16_gemm_ws(hipStream_t s, const GemmArgs &a, int epi, int R) {
  dim3 grid;
  int groups = 0;
  if (!gemm_ws_shape(a, epi, R, grid, groups)) return -1;
  int rc;
#define SKD_WS(R) (a.B_pad == 96 ? launch_gemm_ws<6, R>(s, a, epi, grid) : launch_gemm_ws<8, R>(s, a, epi, grid))
  if (R == 1) rc = SKD_WS(1);
  else if (R == 2) rc = SKD_WS(2);
  else if (R == 3) rc = SKD_WS(3);
  else rc = SKD_WS(4);
#undef SKD_WS
  return rc < 0 ? -1 : groups;
}

// ------------------------------------------------------------------ tiled GEMM for the batched prompt
// With thousands of activation rows the projections are compute-bound, and the
// skinny kernel above (every wave fetching its own operands) is limited by
// L2-to-CU traffic.  Here a workgroup of 8 waves owns a 256 x 256 output tile
// (16 weight tiles x 16 activation-row tiles).  The operand fragments of one
// k-step (32 KiB) form a stage; a ring of 4 stages lives in LDS and is filled by
// LDS-direct global loads (each lane supplies a global address, its 16 bytes
// land at the wave's LDS base + 16 * lane: no
// register holds data in flight; weight fragments arrive ready-made, activations
// in the order of staged_piece), three stages ahead of the one being
// multiplied.  Each wave accumulates a 64 x 128 sub-tile (4 x 8 MFMA tiles, 128
// accumulator registers), reading 12 fragments from LDS per 32 MFMAs.
// A k-step takes 1024 cycles of a CU's matrix cores and 1024 of its LDS (96 KiB read, 32 KiB written, 128 bytes a clock),
// so the two waves of a SIMD take turns: while one multiplies the other one reads.  With all 8 waves in phase, each
// reading the next k-step among its MFMAs, a k-step took 0.55 us on an otherwise idle chip, now 0.465 (1116 cycles at
// 2.4 GHz).  With every CU busy it takes 0.72: the power limit lowers the clock (16384 rows x 4096 x 16384, TFLOP/s: 1436
// -> 1541 with normal operands, 1817 -> 1832 with zeros).  Stand-alone, us: 16384 x 4096 x 16384 1553 -> 1470, x 16384 x
// 4096 1531 -> 1427, x 4096 x 12288 1197 -> 1114.  Slower: v_mfma 32x32x16 (1270 TFLOP/s; alone it reaches 1840 against
// 2100 of 16x16x32), four waves of 128 x 128 (1371).
// Sources and ring places advance with the stages; with an address worked out per stage (64-bit products) prompts took, us, 16384
// rows of the 6.7B shape 6217 instead of 6029, 128 ragged sequences 14278 instead of 13674, 32 x 500 of the 1.3B shape 4628
// instead of 4530.
// A workgroup computes one output tile and gives its CU back.  256 workgroups that take several tiles each, the ring running
// on through them, are no faster (the same three: 6036, 13770, 4549), need 212 registers instead of 190, and hold every CU for
// the whole launch: a step of 4 layers of 256 beside prompts of 8192 rows of 4096 took 380 us instead of 170, on the separate
// kernels 690 instead of 450.
constexpr int TILE_NS = 4;   // ring stages
constexpr int TILE_FR = 32;  // fragments per stage: 16 weight tiles, then 16 activation-row tiles

// wait until at most n of this wave's vector-memory operations are outstanding (they complete in order); n: 0, 4 or 8
__device__ inline void wait_vmcnt_le(int n) {
  switch (n) {
    case 0: wait_vmcnt<0>(); break;
    case 4: wait_vmcnt<4>(); break;
    default: wait_vmcnt<8>(); break;
  }
}

// EPI_QKV_ROWS: where the keys and values of a wave's MT activation-row tiles go.  The output rows of a wave lie inside one
// of q | k | v (d is a multiple of 64, a head), and the 16 rows of a tile belong to one sequence, one page and one half of
// a 32-key block of it, so all this is wave-uniform.  The place in the block table and in the page is the same in every
// layer: k_prompt_map writes it once per prompt, so what is left per output tile are two dependent scalar loads, taken under
// the main loop (as vector loads they return behind its stages, 2 us later).
template <int MT>
struct CacheTiles {
  int which;     // 0 = q, 1 = k, 2 = v
  int page[MT];  // -1: nothing to store
  int at[MT];    // CacheTile::at
  __device__ int slot(int m) const { return CacheTile::slot(at[m]); }
  __device__ int valid(int m) const { return CacheTile::valid(at[m]); }
};
template <int MT>
__device__ inline CacheTiles<MT> row_tiles(const GemmArgs &a, int nt0, int mt0) {
  CacheTiles<MT> t;
  t.which = nt0 * 16 / a.d;
#pragma unroll
  for (int m = 0; m < MT; ++m) t.page[m] = -1, t.at[m] = -1;
  if (t.which == 0) return t;
  // no branches: the loads of all tiles are in flight together; scalar ones, which the compiler does not make by itself
  // behind loads to LDS
  const auto tiles = (const CacheTile __attribute__((address_space(4))) *)a.cache_tiles + mt0;
  const auto pages = (const int32_t __attribute__((address_space(4))) *)a.bt_layer;
#pragma unroll
  for (int m = 0; m < MT; ++m) t.page[m] = pages[tiles[m].page], t.at[m] = tiles[m].at;
#pragma unroll
  for (int m = 0; m < MT; ++m)
    if (!CacheTile::any(t.at[m])) t.page[m] = -1;
  return t;
}
struct NoCacheTiles {};
template <int EPI, int MT>
__device__ inline auto row_tiles_for(const GemmArgs &a, int nt0, int mt0) {
  if constexpr (EPI == EPI_QKV_ROWS) return row_tiles<MT>(a, nt0, mt0);
  else return NoCacheTiles{};
}

// Two neighbouring weight tiles of one activation-row tile, four outputs of each per lane (those from 4 (l >> 4) on), as
// bf16: exchanged between 16-lane rows 0 | 1 and 2 | 3, so that a lane gets eight consecutive outputs of one tile, those of
// tile (l >> 4) & 1 from 8 (l >> 5) on, and a wave stores 1 KiB in 16-byte pieces.
__device__ inline uint4 pack_tile_pair(floatx4 v0, floatx4 v1) {
  const auto lo = __builtin_amdgcn_permlane16_swap(pack2(v0[0], v0[1]), pack2(v1[0], v1[1]), false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap(pack2(v0[2], v0[3]), pack2(v1[2], v1[3]), false, false);
  return make_uint4(lo[0], hi[0], lo[1], hi[1]);
}

// Epilogue of the tiled prompt GEMMs: a wave's RT x MT output tiles, weight tiles nt0 .. nt0 + RT - 1 (nt0 even) and
// activation-row tiles mt0 .. mt0 + MT - 1.  acc[r][m]: lane l holds output rows (weight rows) n0 .. n0 + 3 of activation row
// row0(m) + (l & 15), n0 = 16 * (weight tile) + 4 * (l >> 4).
template <int EPI, int RT, int MT, typename T>
__device__ inline void tile_epilogue(const GemmArgs &a, const floatx4 (&acc)[RT][MT], const T &tiles, int nt0, int mt0, int sp, int lane) {
  static_assert(RT % 2 == 0, "weight tiles are stored in pairs");
  const int grp = lane >> 4, j = lane & 15;
  auto n0_of = [&](int r) { return ((nt0 + r) << 4) + 4 * grp; };
  auto pair_n0_of = [&](int r) { return ((nt0 + r + (grp & 1)) << 4) + 8 * (grp >> 1); };  // after pack_tile_pair
  auto row0_of = [&](int m) { return (mt0 + m) << 4; };
  if constexpr (EPI == EPI_PARTIAL) {  // partial sums of K part sp
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int r = 0; r < RT; ++r)
        *(floatx4 *)&a.partial[((long)sp * a.B_pad + row0_of(m) + j) * a.N + n0_of(r)] = acc[r][m];
  } else if constexpr (EPI == EPI_RELU) {
    floatx4 bias[RT];
#pragma unroll
    for (int r = 0; r < RT; ++r) bias[r] = *(const floatx4 *)&a.bias[n0_of(r)];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int r = 0; r < RT; r += 2) {
        floatx4 v0 = acc[r][m] + bias[r], v1 = acc[r + 1][m] + bias[r + 1];
        for (int i = 0; i < 4; ++i) v0[i] = fmaxf(v0[i], 0.f), v1[i] = fmaxf(v1[i], 0.f);
        *(uint4 *)&a.act_out[d_act_index(row0_of(m) + j, pair_n0_of(r), a.N)] = pack_tile_pair(v0, v1);
      }
  } else if constexpr (EPI == EPI_RESID) {
    // the residual values of the next weight tile are requested before the current one is stored: one exposed
    // round trip per workgroup instead of four
    floatx4 xv[2][MT];
    auto fetch = [&](int r, floatx4(&x)[MT]) {
#pragma unroll
      for (int m = 0; m < MT; ++m) x[m] = *(const floatx4 *)&a.x[(long)(row0_of(m) + j) * a.N + n0_of(r)];
    };
    auto store = [&](int r, const floatx4(&x)[MT]) {
      const floatx4 bias = *(const floatx4 *)&a.bias[n0_of(r)];
#pragma unroll
      for (int m = 0; m < MT; ++m) *(floatx4 *)&a.x[(long)(row0_of(m) + j) * a.N + n0_of(r)] = x[m] + (acc[r][m] + bias);
    };
    fetch(0, xv[0]);
    if constexpr (RT > 1) fetch(1, xv[1]);
#pragma unroll
    for (int r = 0; r < RT; ++r) {
      store(r, xv[r & 1]);
      if (r + 2 < RT) fetch(r + 2, xv[r & 1]);
    }
  } else {  // EPI_QKV_ROWS
    // The outputs of a wave lie inside one head, so the place of a value is a 64-bit base per activation tile (page, head,
    // block, half: uniform) and a 32-bit offset inside the block (lane and element): one addition per store.  With the
    // lookups, and the divisions of every store, in here an epilogue took 5.8 us of a launch (128 x 256 tiles, 912 rows of
    // the 1.3B shape) and 7.4 (128 x 128), without them 3.5 and 3.3; those that store partial sums or activations take 2 to
    // 2.6.  Activation tiles outermost: what is uniform per tile is in scalar registers for one of them at a time.  With the
    // weight tiles outermost, and the place of every tile worked out in the kernel, a prompt pass took 573 us (912 rows of the
    // 1.3B shape), 6346 (16384 of the 6.7B shape) and 14683 (128 ragged sequences), then 565, 6267 and 14418.
    static_assert(16 * RT <= 64, "outputs of a wave in one head");
    const int dh = a.kv.dh, head = (nt0 * 16 - tiles.which * a.d) >> (dh == 64 ? 6 : 7), t = j & 3;
    floatx4 bias[RT];
#pragma unroll
    for (int r = 0; r < RT; ++r) bias[r] = *(const floatx4 *)&a.bias[n0_of(r)];
    if (tiles.which == 0) {
#pragma unroll
      for (int m = 0; m < MT; ++m) {
        if (row0_of(m) >= a.rows) continue;
#pragma unroll
        for (int r = 0; r < RT; r += 2)
          *(uint4 *)&a.q_out[d_act_index(row0_of(m) + j, pair_n0_of(r), a.d)] =
              pack_tile_pair(acc[r][m] + bias[r], acc[r + 1][m] + bias[r + 1]);
      }
      return;
    }
    auto block_of = [&](int m) { return a.kv_pool + (long)tiles.page[m] * a.kv.page_elems + kv_block_base(head, tiles.slot(m), a.kv); };
    auto half_of = [&](int m) { return (tiles.slot(m) >> 4) & 1; };  // 16 keys of the block
    if (tiles.which == 1) {  // 16 bytes per position
      int at[RT / 2];
#pragma unroll
      for (int r = 0; r < RT; r += 2) {
        at[r / 2] = kv_k_at(j, (pair_n0_of(r) - a.d) & (dh - 1));
      }
#pragma unroll
      for (int m = 0; m < MT; ++m) {
        if (tiles.page[m] < 0) continue;
        bf16_t *pg = block_of(m) + kv_k_half(half_of(m), dh);
#pragma unroll
        for (int r = 0; r < RT; r += 2) {
          const uint4 pk = pack_tile_pair(acc[r][m] + bias[r], acc[r + 1][m] + bias[r + 1]);
          if (j < tiles.valid(m)) *(uint4 *)&pg[at[r / 2]] = pk;
        }
      }
      return;
    }
    // v: a page holds, for one element e, four consecutive positions of each half side by side.  The four lanes of a quad
    // hold positions 4q .. 4q + 3 for elements e .. e + 3 each: transposed inside the quad (two exchanges,
    // with the lane 1 and the lane 2 away), lane t ends up with element e + t of all four positions, 8 bytes.  Where both
    // halves of a block are whole and in this wave, they are stored together.
    auto transposed = [&](floatx4 v) {
      {
        const float s0 = (t & 1) ? v[0] : v[1], s1 = (t & 1) ? v[2] : v[3];
        const float r0 = __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, s0), 0xB1, 0xF, 0xF, true));
        const float r1 = __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, s1), 0xB1, 0xF, 0xF, true));
        if (t & 1) { v[0] = r0; v[2] = r1; } else { v[1] = r0; v[3] = r1; }
      }
      {
        const float s0 = (t & 2) ? v[0] : v[2], s1 = (t & 2) ? v[1] : v[3];
        const float r0 = __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, s0), 0x4E, 0xF, 0xF, true));
        const float r1 = __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, s1), 0x4E, 0xF, 0xF, true));
        if (t & 2) { v[0] = r0; v[1] = r1; } else { v[2] = r0; v[3] = r1; }
      }
      return v;  // v[s] = element e + t of position 4 * (j / 4) + s
    };
    auto whole_block_at = [&](int m) {
      return m + 1 < MT && half_of(m) == 0 && tiles.valid(m) == 16 && tiles.page[m + 1] == tiles.page[m] &&
             tiles.at[m + 1] == tiles.at[m] + 16;
    };
    int at[RT];
#pragma unroll
    for (int r = 0; r < RT; ++r) {
      at[r] = kv_v_at(j, ((n0_of(r) - 2 * a.d) & (dh - 1)) + t);
    }
#pragma unroll
    for (int m = 0; m < MT; ++m) {
      if (tiles.page[m] < 0 || (m > 0 && whole_block_at(m - 1))) continue;
      bf16_t *pg = block_of(m) + kv_v_half(half_of(m), dh);
      if (whole_block_at(m)) {
        const int m1 = m + 1 < MT ? m + 1 : m;
#pragma unroll
        for (int r = 0; r < RT; ++r) {
          const floatx4 v = transposed(acc[r][m] + bias[r]), u = transposed(acc[r][m1] + bias[r]);
          *(uint4 *)&pg[at[r]] = make_uint4(pack2(v[0], v[1]), pack2(v[2], v[3]), pack2(u[0], u[1]), pack2(u[2], u[3]));
        }
        continue;
      }
      const int nvalid = tiles.valid(m) - (j & ~3);
#pragma unroll
      for (int r = 0; r < RT; ++r) {
        const floatx4 v = transposed(acc[r][m] + bias[r]);
        bf16_t *dst = &pg[at[r]];
        if (nvalid >= 4) {
          *(uint2 *)dst = make_uint2(pack2(v[0], v[1]), pack2(v[2], v[3]));
        } else {
          for (int s_ = 0; s_ < 4; ++s_)
            if (s_ < nvalid) dst[s_] = (bf16_t)f2bf(v[s_]);
        }
      }
    }
  }
}

template <int EPI>
__global__ __launch_bounds__(512) void k_gemm_tile(GemmArgs a) {
  extern __shared__ bf16x8 tile_lds[];  // [TILE_NS stages][TILE_FR][64 lanes]
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int wr = wave >> 1, wc = wave & 1;  // sub-tile: weight tiles 4wr .. 4wr+3, activation tiles 8wc .. 8wc+7
  // workgroup -> output tile.  Workgroups are dealt to the 8 XCDs round-robin; the ones that share an XCD (and
  // its L2) at any moment should share operands, so each XCD walks its own contiguous range of tiles in bands
  // of 4 activation tiles x all weight tiles, weight tile fastest in groups of 4 rows (the last band has the
  // gy % 4 activation tiles that are left; XCD x owns the workgroups with id % 8 == x, one more than the others
  // when x < total % 8).
  int tn, tm, sp;
  {
    const int gx = a.N >> 8, gy = (a.rows + 255) >> 8, tiles = gx * gy, total = tiles * a.split;
    const int id = blockIdx.x;
    const int xcd = id & 7, per = total >> 3, rem = total & 7;
    int logical = xcd * per + min(xcd, rem) + (id >> 3);
    sp = logical / tiles;  // K part
    logical -= sp * tiles;
    const int full = gy >> 2, tail0 = full * 4 * gx;
    if (logical < tail0) {
      const int band = logical / (4 * gx), within = logical - band * 4 * gx;
      tn = within >> 2;
      tm = band * 4 + (within & 3);
    } else {
      const int hb = gy & 3, within = logical - tail0;  // hb > 0 here
      tn = within / hb;
      tm = full * 4 + within % hb;
    }
  }
  const int k0 = (int)((long)(a.K >> 5) * sp / a.split), Kf = (int)((long)(a.K >> 5) * (sp + 1) / a.split) - k0;

  // this wave's share of a stage: 4 fragments; waves 0..3 fetch the weight tiles, waves 4..7 the activation tiles.
  // Fragment bases are wave-uniform (scalar registers); the only per-lane part of an address is the lane's place
  // in the fragment, one 32-bit register.
  const int ld_is_a = wave >> 2, ld_t0 = (wave & 3) * 4;
  const bf16x8 *src[4];  // of the next stage to request
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int T = a.t0 + tn * 16 + ld_t0 + i;
    src[i] = ld_is_a ? (const bf16x8 *)a.A + ((long)(tm * 16 + ld_t0 + i) * (a.K >> 5) + k0) * 64
                     : (const bf16x8 *)a.W + (((long)(T / a.G) * (a.K >> 5) + k0) * a.G + T % a.G) * 64;
  }
  const long sstride = ld_is_a ? 64 : (long)a.G * 64;
  const unsigned vlane = ld_is_a ? staged_piece(lane) : lane;
  const int dfrag = ld_is_a * 16 + ld_t0, xlane = staged_lane(lane);
  int to = 0, from = 0;  // ring slots: of the next stage to request, of the next to multiply
  auto issue = [&]() {  // 4 vector-memory operations per wave and stage
    bf16x8 *dst = tile_lds + (to * TILE_FR + dfrag) * 64;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)&src[i][vlane],
                                       (__attribute__((address_space(3))) void *)(dst + i * 64), 16, 0, 0);
      src[i] += sstride;
    }
    to = (to + 1) % TILE_NS;
  };
  auto bar = [&]() {  // bare: __syncthreads() would also wait for the loads of the later stages
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  floatx4 acc[4][8];
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int m = 0; m < 8; ++m) acc[r][m] = floatx4{0.f, 0.f, 0.f, 0.f};
  // One k-step of a wave: a slot for memory (12 LDS reads of stage st, the requests of stage st + 3), a barrier, a slot
  // for the matrix cores, a barrier.  Waves 4 .. 7 run one barrier behind waves 0 .. 3, so of the two waves on a SIMD one
  // multiplies while the other one reads.
  // Ring: stage st + 3 goes into the slot of stage st - 1, which every wave has read by then (the late group read it
  // in its memory slot before last, with lgkmcnt 0 before the barrier).  Stage st + 1 has landed for every wave that
  // reads it: each wave waits for its own loads of it (all but the `later` stages behind it) in its memory slot st, and
  // at least one barrier lies between the last of these waits and the first read.
  auto k_step = [&](bool more, int later) {
    __builtin_amdgcn_sched_barrier(0);
    bf16x8 wf[4], xf[8];
    const bf16x8 *base = tile_lds + from * (TILE_FR * 64);
#pragma unroll
    for (int r = 0; r < 4; ++r) wf[r] = base[(wr * 4 + r) * 64 + lane];
#pragma unroll
    for (int m = 0; m < 8; ++m) xf[m] = base[(16 + wc * 8 + m) * 64 + xlane];
    from = (from + 1) % TILE_NS;
    if (more) issue();
    __builtin_amdgcn_sched_barrier(0);
    wait_vmcnt_le(4 * later);
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
    bar();
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(1);
    // neighbours share an operand (activation tile outer, weight tiles back and forth): the registers that feed the
    // matrix cores change less, which at this load is clock (1464 -> 1496 TFLOP/s)
#pragma unroll
    for (int m = 0; m < 8; ++m)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int r = (m & 1) ? 3 - i : i;
        acc[r][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[r], xf[m], acc[r][m], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
    __builtin_amdgcn_s_setprio(0);
    bar();
  };

#pragma unroll
  for (int i = 0; i < TILE_NS - 1; ++i)
    if (i < Kf) issue();
  wait_vmcnt_le(4 * min(Kf - 1, TILE_NS - 2));
  bar();  // stage 0 is here
  if (wave >= 4) bar();
  int st = 0;
  for (; st + TILE_NS - 1 < Kf; ++st) k_step(true, TILE_NS - 2);
  const int nt0 = a.t0 + tn * 16 + wr * 4, mt0 = tm * 16 + wc * 8;
  const auto tiles = row_tiles_for<EPI, 8>(a, nt0, mt0);  // arrive under the last k-steps
  for (; st < Kf; ++st) k_step(false, max(Kf - 2 - st, 0));
  if (wave < 4) bar();
  tile_epilogue<EPI, 4, 8>(a, acc, tiles, nt0, mt0, sp, lane);
}

// Batched-prompt projections on 256 x 256 tiles.  Returns 0, or -1 when the shape does not tile.
int bf16_gemm_tile(hipStream_t s, const GemmArgs &a, int epi) {
  if (a.rows <= 0 || a.N % 256 || a.K % 32 || a.G < 1 || a.G > 4 || a.split < 1 || a.split > a.K / 32) return -1;
  if (a.split != 1 && epi != EPI_PARTIAL) return -1;
  const dim3 grid((a.N / 256) * ((a.rows + 255) / 256) * a.split), blk(512);
  const size_t lds = (size_t)TILE_NS * TILE_FR * 64 * sizeof(bf16x8);  // 128 KiB of the CU's 160
  static std::atomic<uint64_t> done{0};
  if (!allow_lds(done, {(const void *)k_gemm_tile<EPI_QKV_ROWS>,
                        (const void *)k_gemm_tile<EPI_RESID>,
                        (const void *)k_gemm_tile<EPI_PARTIAL>,
                        (const void *)k_gemm_tile<EPI_RELU>}, lds))
    return -1;
  switch (epi) {
    case EPI_QKV_ROWS: SKD_LAUNCH(k_gemm_tile<EPI_QKV_ROWS>, grid, blk, lds, s, a); break;
    case EPI_RESID: SKD_LAUNCH(k_gemm_tile<EPI_RESID>, grid, blk, lds, s, a); break;
    case EPI_PARTIAL: SKD_LAUNCH(k_gemm_tile<EPI_PARTIAL>, grid, blk, lds, s, a); break;
    case EPI_RELU: SKD_LAUNCH(k_gemm_tile<EPI_RELU>, grid, blk, lds, s, a); break;
    default: return -1;
  }
  return 0;
}

// ------------------------------------------------------------------ tiled GEMM for prompts of a few hundred rows
// On 256 x 256 tiles a prompt of a few hundred rows gives a handful of workgroups (912 rows at d = 2048: 32 for the
// N = d projections, on 256 CUs).  The same ring and fragment order with WN x WM waves of RT x MT MFMA tiles each: the
// workgroup owns 16 RT WN weight rows x 16 MT WM activation rows, the ring has NS stages, and the K range can be split
// over `a.split` workgroups whose fp32 partial sums the row reducer adds.  With 4 waves two workgroups share a CU, so
// one multiplies while the other waits at its barrier; with 8 waves the two of a SIMD take turns.  What bounds it is how
// many bytes a CU takes in per MFMA: at 912 rows of the 1.3B shape FFN1's 128 x 256 tiles read 11.2 TB/s through L2
// (44 GB/s to each CU) with the matrix cores 37 % busy, whatever the ring depth (64 x 128 tiles: 5 and 6 stages alike,
// 64 x 64: 5 and 9), so the largest tile that still fills the chip wins.
// us per launch, 256 x 256 -> best tile and split: 256 rows of the 6.7B shape QKV 81 -> 43, output 87 -> 17 (split 4),
// FFN1 80 -> 44, FFN2 296 -> 46 (split 4), all 128 x 128; 1024 rows of the 1.3B shape QKV 44 -> 32 and FFN1 45 -> 35
// (128 x 256; 128 x 128: 37 and 41), output 51 -> 15 (128 x 128, split 2), FFN2 153 -> 37 (128 x 256, split 4).
template <int RT, int MT, int WN, int WM, int NS, int EPI>
__global__ __launch_bounds__(WN * WM * 64, 2) void k_gemm_mid(GemmArgs a) {
  constexpr int FW = WN * RT, FA = WM * MT, FR = FW + FA;  // weight and activation fragments per stage
  constexpr int LPW = FR / (WN * WM);                      // loads per wave and stage
  extern __shared__ bf16x8 mid_lds[];                      // [NS][FR][64 lanes]
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int wr = wave / WM, wc = wave % WM;
  const int Kf = a.K >> 5;
  // workgroup -> (K part, output tile), XCD-aware as in k_gemm_tile: every XCD walks a contiguous range, bands of 4
  // activation tiles x all weight tiles
  int tn, tm, sp;
  {
    const int gx = a.N / (16 * FW), gy = (a.rows + 16 * FA - 1) / (16 * FA), tiles = gx * gy, total = tiles * a.split;
    const int id = blockIdx.x, xcd = id & 7;
    int logical = xcd * (total >> 3) + min(xcd, total & 7) + (id >> 3);
    sp = logical / tiles;
    logical -= sp * tiles;
    const int band = logical / (4 * gx), hb = min(4, gy - 4 * band), within = logical - band * 4 * gx;
    tn = within / hb;
    tm = band * 4 + within % hb;
  }
  const int k0 = (int)((long)Kf * sp / a.split), n = (int)((long)Kf * (sp + 1) / a.split) - k0;

  // this wave's fragments of a stage: LPW consecutive ones of [FW weight tiles, FA activation-row tiles]
  const bf16x8 *src[LPW];
  long stride[LPW];
  unsigned vl[LPW];
#pragma unroll
  for (int i = 0; i < LPW; ++i) {
    const int fr = wave * LPW + i;
    if (fr < FW) {
      const int T = a.t0 + tn * FW + fr;
      src[i] = (const bf16x8 *)a.W + (((long)(T / a.G) * Kf + k0) * a.G + T % a.G) * 64;
      stride[i] = (long)a.G * 64;
      vl[i] = lane;
    } else {
      src[i] = (const bf16x8 *)a.A + ((long)(tm * FA + fr - FW) * Kf + k0) * 64;
      stride[i] = 64;
      vl[i] = staged_piece(lane);
    }
  }
  const int xlane = staged_lane(lane);
  floatx4 acc[RT][MT];
#pragma unroll
  for (int r = 0; r < RT; ++r)
#pragma unroll
    for (int m = 0; m < MT; ++m) acc[r][m] = floatx4{0.f, 0.f, 0.f, 0.f};

  auto issue = [&](int st) {
    bf16x8 *dst = mid_lds + ((st % NS) * FR + wave * LPW) * 64;
#pragma unroll
    for (int i = 0; i < LPW; ++i)
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)&(src[i] + (long)st * stride[i])[vl[i]],
                                       (__attribute__((address_space(3))) void *)(dst + i * 64), 16, 0, 0);
  };
  auto read = [&](int st, bf16x8(&wf)[RT], bf16x8(&xf)[MT]) {
    const bf16x8 *base = mid_lds + (st % NS) * (FR * 64);
#pragma unroll
    for (int r = 0; r < RT; ++r) wf[r] = base[(wr * RT + r) * 64 + lane];
#pragma unroll
    for (int m = 0; m < MT; ++m) xf[m] = base[(FW + wc * MT + m) * 64 + xlane];
  };
  auto mma = [&](const bf16x8(&wf)[RT], const bf16x8(&xf)[MT]) {
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
      for (int m = 0; m < MT; ++m) acc[r][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[r], xf[m], acc[r][m], 0, 0, 0);
  };
  auto bar = [&]() {  // this wave's LDS reads are done; bare barrier: __syncthreads() would wait for the loads in flight
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  auto lookups = [&]() { return row_tiles_for<EPI, MT>(a, a.t0 + tn * FW + wr * RT, tm * FA + wc * MT); };
  decltype(lookups()) tiles;
  if constexpr (WN * WM == 8) {
    // The two waves of a SIMD take turns at LDS and matrix cores as in k_gemm_tile, two k-steps (a pair of stages) to a
    // turn: waves 4 .. 7 run one barrier behind waves 0 .. 3.  Ring: pair p + 2 goes into the slots of pair p - 1, which
    // the late group has read in its memory turn before last; pair p + 1 has landed for every reader: each wave waits for
    // its own loads of it in its memory turn p, and at least one barrier lies between the last such wait and the first read.
    // With all waves in phase, LDS reads dealt out among the MFMAs, a k-step took 0.45 us alone and 0.51 with every CU busy;
    // in turns 0.325 with 64 workgroups, 0.38 with 128, 0.44 with 256 (24 KiB to each CU: 14 TB/s).  912 rows of the 1.3B
    // shape, us: QKV 40.4 -> 38.7, FFN1 38.1 -> 35.8, FFN2 39.2 -> 37.2; about 9 us of each lie outside the loop.
    static_assert(NS == 6, "three pairs of stages");
    auto turn = [&](int st, bool two, bool more, int later) {  // later: stages of the pair after next
      __builtin_amdgcn_sched_barrier(0);
      bf16x8 wf[2][RT], xf[2][MT];
      read(st, wf[0], xf[0]);
      if (two) read(st + 1, wf[1], xf[1]);
      if (more || st + 4 < n) issue(st + 4);
      if (more || st + 5 < n) issue(st + 5);
      __builtin_amdgcn_sched_barrier(0);
      if (later == 2) wait_vmcnt<2 * LPW>();
      else if (later == 1) wait_vmcnt<LPW>();
      else wait_vmcnt<0>();
      bar();
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_setprio(1);
#pragma unroll
      for (int h = 0; h < 2; ++h)
        if (h == 0 || two)
#pragma unroll
          for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int i = 0; i < RT; ++i) {  // neighbours share an operand
              const int r = (m & 1) ? RT - 1 - i : i;
              acc[r][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[h][r], xf[h][m], acc[r][m], 0, 0, 0);
              __builtin_amdgcn_sched_barrier(0);
            }
      __builtin_amdgcn_s_setprio(0);
      bar();
    };
#pragma unroll
    for (int i = 0; i < NS - 2; ++i)
      if (i < n) issue(i);
    tiles = lookups();
    if (n >= 4) wait_vmcnt<2 * LPW>();
    else if (n == 3) wait_vmcnt<LPW>();
    else wait_vmcnt<0>();
    bar();  // pair 0 is here
    if (wave >= 4) bar();
    int st = 0;
    for (; st + NS <= n; st += 2) turn(st, true, true, 2);
    for (; st < n; st += 2) turn(st, st + 1 < n, false, min(max(n - 4 - st, 0), 2));
    if (wave < 4) bar();
  } else {
    // stage st becomes readable, the slot of stage st - 1 is refilled (see k_gemm_tile)
    auto open_stage = [&](int st) {
      const int later = min(n - 1 - st, NS - 2);
      if (later == 0) wait_vmcnt<0>();
      else if (later == 1) wait_vmcnt<LPW>();
      else if (later == 2) wait_vmcnt<2 * LPW>();
      else if (later == 3) wait_vmcnt<3 * LPW>();
      else wait_vmcnt<(NS - 2) * LPW>();
      bar();
      if (st + NS - 1 < n) issue(st + NS - 1);
    };
#pragma unroll
    for (int i = 0; i < NS - 1; ++i)
      if (i < n) issue(i);
    tiles = lookups();
    bf16x8 wfA[RT], xfA[MT], wfB[RT], xfB[MT];
    open_stage(0);
    read(0, wfA, xfA);
    // steady state: the LDS reads of the next stage are dealt out among the MFMAs of the current one
    auto steady = [&](int nx, bf16x8(&wn)[RT], bf16x8(&xn)[MT], const bf16x8(&wc_)[RT], const bf16x8(&xc)[MT]) {
      wait_vmcnt<(NS - 2) * LPW>();
      bar();
      issue(nx + NS - 1);
      read(nx, wn, xn);
      mma(wc_, xc);
      __builtin_amdgcn_sched_group_barrier(0x020, LPW, 0);
#pragma unroll
      for (int i = 0; i < RT + MT; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      }
      __builtin_amdgcn_sched_group_barrier(0x008, RT * MT - (RT + MT), 0);
    };
    int st = 0;
    for (; st + NS + 1 < n; st += 2) {
      steady(st + 1, wfB, xfB, wfA, xfA);
      steady(st + 2, wfA, xfA, wfB, xfB);
    }
    for (; st < n; st += 2) {  // the last stages
      if (st + 1 < n) {
        open_stage(st + 1);
        read(st + 1, wfB, xfB);
      }
      __builtin_amdgcn_sched_barrier(0);
      mma(wfA, xfA);
      if (st + 1 < n) {
        if (st + 2 < n) {
          open_stage(st + 2);
          read(st + 2, wfA, xfA);
        }
        __builtin_amdgcn_sched_barrier(0);
        mma(wfB, xfB);
      }
    }
  }
  tile_epilogue<EPI, RT, MT>(a, acc, tiles, a.t0 + tn * FW + wr * RT, tm * FA + wc * MT, sp, lane);
}

template <int RT, int MT, int WN, int WM, int NS>
static int launch_gemm_mid(hipStream_t s, const GemmArgs &a, int epi) {
  constexpr int BN = 16 * RT * WN, BM = 16 * MT * WM;
  constexpr size_t lds = (size_t)NS * (BN + BM) * 4 * sizeof(bf16x8);
  if (a.N % BN) return -1;
  static std::atomic<uint64_t> done{0};
  if (!allow_lds(done, {(const void *)k_gemm_mid<RT, MT, WN, WM, NS, EPI_QKV_ROWS>,
                        (const void *)k_gemm_mid<RT, MT, WN, WM, NS, EPI_RESID>,
                        (const void *)k_gemm_mid<RT, MT, WN, WM, NS, EPI_PARTIAL>,
                        (const void *)k_gemm_mid<RT, MT, WN, WM, NS, EPI_RELU>}, lds))
    return -1;
  const dim3 grid((a.N / BN) * ((a.rows + BM - 1) / BM) * a.split), blk(WN * WM * 64);
  switch (epi) {
    case EPI_QKV_ROWS: SKD_LAUNCH((k_gemm_mid<RT, MT, WN, WM, NS, EPI_QKV_ROWS>), grid, blk, lds, s, a); break;
    case EPI_RESID: SKD_LAUNCH((k_gemm_mid<RT, MT, WN, WM, NS, EPI_RESID>), grid, blk, lds, s, a); break;
    case EPI_PARTIAL: SKD_LAUNCH((k_gemm_mid<RT, MT, WN, WM, NS, EPI_PARTIAL>), grid, blk, lds, s, a); break;
    case EPI_RELU: SKD_LAUNCH((k_gemm_mid<RT, MT, WN, WM, NS, EPI_RELU>), grid, blk, lds, s, a); break;
    default: return -1;
  }
  return 0;
}
// weight_rows x act_rows per workgroup: 256 x 128, 128 x 256, 128 x 128, 64 x 128, 128 x 64 or 64 x 64.  Returns 0, or -1 when the shape does
// not tile (nothing launched).
int bf16_gemm_mid(hipStream_t s, const GemmArgs &a, int epi, int weight_rows, int act_rows) {
  const int Kf = a.K >> 5;
  if (a.rows <= 0 || a.N < 1 || a.K < 32 || a.K % 32 || a.G < 1 || a.G > 4 || a.split < 1 || a.split > Kf) return -1;
  if (a.split != 1 && epi != EPI_PARTIAL) return -1;
  if (weight_rows == 256 && act_rows == 128) return launch_gemm_mid<4, 4, 4, 2, 6>(s, a, epi);
  if (weight_rows == 128 && act_rows == 256) return launch_gemm_mid<4, 4, 2, 4, 6>(s, a, epi);
  if (weight_rows == 128 && act_rows == 128) return launch_gemm_mid<4, 4, 2, 2, 5>(s, a, epi);
  if (weight_rows == 64 && act_rows == 128) return launch_gemm_mid<2, 4, 2, 2, 5>(s, a, epi);
  if (weight_rows == 128 && act_rows == 64) return launch_gemm_mid<4, 2, 2, 2, 5>(s, a, epi);
  if (weight_rows == 64 && act_rows == 64) return launch_gemm_mid<2, 2, 2, 2, 5>(s, a, epi);
  return -1;
}

// ------------------------------------------------------------------ row kernels: embedding / split-K reduce, + LayerNorm
// One workgroup per batch row, one thread per float4 chunk up to 1024 threads.  These kernels move < 5 MB and are
// pure latency chains, so each thread keeps its share of the row in registers
// (float4 chunk c = threadIdx.x + blockDim.x * i, rows up to 16384 wide), issues
// every global load it will ever need up front, and the row never touches LDS.
constexpr int LN_NC = 4;

// v[i] = elements 4c .. 4c+3 of row b.  LayerNorm (mean, biased variance, eps 1e-5) -> bf16 row of the activation tiles.
template <int LN_NC>
__device__ inline void ln_finish_row(const floatx4 (&v)[LN_NC], const floatx4 (&gv)[LN_NC], const floatx4 (&bv)[LN_NC],
                                     int d, int b, bf16_t *a_out, float *sh) {
  const int d4 = d >> 2;
  float s = 0;
#pragma unroll
  for (int i = 0; i < LN_NC; ++i)
    if ((int)(threadIdx.x + blockDim.x * i) < d4) s += (v[i][0] + v[i][1]) + (v[i][2] + v[i][3]);
  const float mean = block_sum_once(s, sh) / d;  // sh: 32 floats, one half per reduction, so two barriers in all
  float q = 0;
#pragma unroll
  for (int i = 0; i < LN_NC; ++i)
    if ((int)(threadIdx.x + blockDim.x * i) < d4) {
      const floatx4 t = v[i] - mean;
      q += (t[0] * t[0] + t[1] * t[1]) + (t[2] * t[2] + t[3] * t[3]);
    }
  const float rstd = 1.0f / sqrtf(block_sum_once(q, sh + 16) / d + 1e-5f);
#pragma unroll
  for (int i = 0; i < LN_NC; ++i) {
    const int c = (int)(threadIdx.x + blockDim.x * i);
    if (c < d4) {
      const floatx4 y = (v[i] - mean) * rstd * gv[i] + bv[i];
      *(uint2 *)&a_out[d_act_index(b, 4 * c, d)] = make_uint2(pack2(y[0], y[1]), pack2(y[2], y[3]));
    }
  }
}

// threads of a row workgroup: one per float4 chunk, whole waves, at most 1024 (narrow rows: fewer waves at the barriers)
static int row_threads(int d) { return d / 4 >= 1024 ? 1024 : (d / 4 + 63) / 64 * 64; }

__global__ __launch_bounds__(1024) void k_embed_ln(const int32_t *tokens, const int32_t *start, int t,
                                                   const bf16_t *tok_emb, const bf16_t *pos_emb, const float *g,
                                                   const float *bt, float *x, bf16_t *a_out, int d, int V) {
  __shared__ float sh[32];
  const int b = blockIdx.x, d4 = d >> 2;
  int tok = tokens[b];
  tok = tok < 0 ? 0 : (tok >= V ? V - 1 : tok);
  int pos = t - start[b];  // number of real tokens before this column
  if (pos < 0) pos = 0;    // padding column, never attended to
  const uint2 *te = (const uint2 *)(tok_emb + (long)tok * d), *pe = (const uint2 *)(pos_emb + (long)pos * d);
  floatx4 v[LN_NC], gv[LN_NC], bv[LN_NC];
#pragma unroll
  for (int i = 0; i < LN_NC; ++i) {
    const int c = (int)(threadIdx.x + blockDim.x * i);
    if (c < d4) {
      const uint2 a = te[c], p = pe[c];
      gv[i] = ((const floatx4 *)g)[c];
      bv[i] = ((const floatx4 *)bt)[c];
      v[i] = floatx4{bf2f(a.x & 0xffffu) + bf2f(p.x & 0xffffu), bf2f(a.x >> 16) + bf2f(p.x >> 16),
                     bf2f(a.y & 0xffffu) + bf2f(p.y & 0xffffu), bf2f(a.y >> 16) + bf2f(p.y >> 16)};
      ((floatx4 *)x)[(long)b * d4 + c] = v[i];
    }
  }
  ln_finish_row(v, gv, bv, d, b, a_out, sh);
}

void bf16_embed_ln(hipStream_t s, const int32_t *tokens, const int32_t *start, int t, const bf16_t *tok_emb,
                   const bf16_t *pos_emb, const float *g, const float *b, float *x, bf16_t *a_out, int B, int d,
                   int V) {
  SKD_LAUNCH(k_embed_ln, dim3(B), dim3(row_threads(d)), 0, s, tokens, start, t, tok_emb, pos_emb, g, b, x, a_out, d, V);
}

// x[b][:] = x_in[b][:] + bias + sum_s partial[s][b][:] (fixed order), then LayerNorm; x_in may be x.  A latency chain: S is the number of partial
// sums (0 = any, `split` of them), so that all loads are in flight together; as a loop of unknown length the loads
// of the second and later sums waited for one another.
template <int S, int NC>
__global__ __launch_bounds__(1024) void k_reduce_ln(const float *partial, int split, int B_pad, const float *bias,
                                                    const float *x_in, float *x, const float *g, const float *bt, bf16_t *a_out, int d) {
  __shared__ float sh[32];
  const int b = blockIdx.x, d4 = d >> 2;
  const floatx4 *p4 = (const floatx4 *)partial;
  floatx4 *x4 = (floatx4 *)x + (long)b * d4;
  const floatx4 *xi4 = (const floatx4 *)x_in + (long)b * d4;
  floatx4 v[NC], gv[NC], bv[NC];
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    const int c = (int)(threadIdx.x + blockDim.x * i);
    if (c < d4) {
      const floatx4 xv = xi4[c], bias4 = ((const floatx4 *)bias)[c];
      gv[i] = ((const floatx4 *)g)[c];
      bv[i] = ((const floatx4 *)bt)[c];
      floatx4 acc = p4[(long)b * d4 + c];
      if constexpr (S > 0) {
        floatx4 p[S];
#pragma unroll
        for (int sp = 1; sp < S; ++sp) p[sp] = p4[((long)sp * B_pad + b) * d4 + c];
#pragma unroll
        for (int sp = 1; sp < S; ++sp) acc += p[sp];
      } else {
        for (int sp = 1; sp < split; ++sp) acc += p4[((long)sp * B_pad + b) * d4 + c];
      }
      v[i] = xv + (acc + bias4);
      x4[c] = v[i];
    }
  }
  ln_finish_row<NC>(v, gv, bv, d, b, a_out, sh);
}

void bf16_reduce_ln(hipStream_t s, const float *partial, int split, int B_pad, const float *bias, const float *x_in,
                    float *x, const float *g, const float *b, bf16_t *a_out, int B, int d) {
  const dim3 grid(B), blk(row_threads(d));
#define SKD_RED(S, NC) SKD_LAUNCH((k_reduce_ln<S, NC>), grid, blk, 0, s, partial, split, B_pad, bias, x_in, x, g, b, a_out, d)
  if (d > 4096) SKD_RED(0, LN_NC);
  else if (split == 1) SKD_RED(1, 1);
  else if (split == 2) SKD_RED(2, 1);
  else if (split == 3) SKD_RED(3, 1);
  else if (split == 4) SKD_RED(4, 1);
  else if (split == 6) SKD_RED(6, 1);
  else if (split == 8) SKD_RED(8, 1);
  else SKD_RED(0, 1);
#undef SKD_RED
}

// ------------------------------------------------------------------ decode attention over the paged KV cache
// One workgroup of NW waves (1, 2, 4, 8 or 16) per (row, head, split).  Wave w takes
// 32-key blocks first + w, first + w + NW, ...; each block is 2 K tiles (QK^T:
// 2 * DH/32 MFMAs, q replicated over the 16 MFMA columns) and one V block
// (DH/16 MFMAs).  Online softmax per wave in fp32; the waves (and, with
// splits > 1, the workgroups of one head) are merged with the usual max / sum
// rescaling.  Batches with few (row, head) pairs get their 16 waves per CU from
// wider workgroups rather than from splits, which need a second kernel.
// Four waves per SIMD are required: with three the kernel is 13 % slower.
template <int DH, int NW>
__global__ __launch_bounds__(NW * 64, 4) void k_attention(AttnArgs a) {  // 4 waves per SIMD whatever the workgroup width
  constexpr int QC = DH / 32, VM = DH / 16;
  __shared__ float sm_m[NW], sm_l[NW], sm_dot[NW];
  __shared__ float sm_o[NW][DH];
  // uniform wave index: block numbers, page lookups and block addresses become scalar work
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, grp = lane >> 4;
  const int H = a.kv.H, h = blockIdx.x % H, d = H * DH;
  // longest rows are dispatched first, so that the last workgroups to start are the short ones
  const int b = a.order ? a.order[blockIdx.x / H] : (int)(blockIdx.x / H);
  const int j0 = a.start[b], t = a.t;
  // a row's keys are stored by real position: column j sits in slot j - j0, so neither end of the row's first
  // block is padding.  Slots 0 .. len-1 are cached; slot len (column t) arrives in kv_new.
  const int len = t - j0;  // cached keys of this row (negative: column t is still padding for it)
  const int blk_lo = 0, blk_hi = (len + 31) >> 5;
  const int nblk = blk_hi - blk_lo;
  const int per = (nblk + a.splits - 1) / a.splits;
  const int my_lo = blk_lo + (int)blockIdx.y * per;
  const int my_hi = min(my_lo + per, blk_hi);
  const int bpp = a.kv.page_tokens >> 5;  // blocks per page
  const int32_t *bt_row = a.bt_layer + (long)b * a.kv.max_pages;
  const float scale = 1.0f / sqrtf((float)DH);

  bf16x8 qf[QC];
#pragma unroll
  for (int c = 0; c < QC; ++c)
    qf[c] = *(const bf16x8 *)&a.q[(long)b * d + h * DH + 32 * c + 8 * grp];

  // Position t itself is not in the cache yet: its k and v arrive in the projection's staging rows.  Thread e
  // takes element e of q, k_t and v_t; the token joins the softmax as one more partial state when the waves
  // are merged, and is filed into its page slot at the very end, when the lines around it have just been read
  // and are resident in L2 (the same stores from the projection's epilogue or from a later kernel cost about
  // 3 us per layer).  When len is not a multiple of 32 the 32-key block that contains slot len IS loaded above,
  // with several splits possibly by another workgroup while this one stores: the result does not depend on
  // what that load sees, because keys >= len get weight 0 and every slot of the pool holds finite bits at all
  // times (the pool is zeroed when it is created and only finite k and v are ever filed), so 0 x slot = 0.
  // (a one-wave workgroup has 64 threads for 128 elements: EPT elements per thread, e = threadIdx.x + i * NW * 64)
  constexpr int EPT = (DH + NW * 64 - 1) / (NW * 64);
  const bool with_new = blockIdx.y == gridDim.y - 1 && len >= 0;
  float q_e[EPT], k_e[EPT], v_e[EPT];
  bf16_t k_bits[EPT], v_bits[EPT];
  int page_t = 0;
#pragma unroll
  for (int i = 0; i < EPT; ++i) {
    q_e[i] = k_e[i] = v_e[i] = 0.f;
    k_bits[i] = v_bits[i] = 0;
    const int e = (int)threadIdx.x + i * NW * 64;
    if (with_new && e < DH) {
      const bf16_t *kr = a.kv_new + ((long)b * 2) * d + h * DH;
      k_bits[i] = kr[e];
      v_bits[i] = kr[d + e];
      q_e[i] = bf2f(a.q[(long)b * d + h * DH + e]);
      k_e[i] = bf2f(k_bits[i]);
      v_e[i] = bf2f(v_bits[i]);
      page_t = bt_row[len / a.kv.page_tokens];
    }
  }

  floatx4 O[VM];
#pragma unroll
  for (int m = 0; m < VM; ++m) O[m] = floatx4{0.f, 0.f, 0.f, 0.f};
  float m_run = -1.0e30f, l_run = 0.f;  // l_run: this lane group's share of the denominator

  auto load_blk = [&](int blk, bf16x8(&kf)[2][QC], bf16x8(&vf)[VM]) {
    const int page = bt_row[blk / bpp];
    const bf16x8 *kp = (const bf16x8 *)(a.pool + (long)page * a.kv.page_elems + (long)h * a.kv.page_tokens * (DH * 2) +
                                        (long)(blk % bpp) * (64 * DH)) + lane;
#pragma unroll
    for (int tl = 0; tl < 2; ++tl)
#pragma unroll
      for (int c = 0; c < QC; ++c) kf[tl][c] = __builtin_nontemporal_load(&kp[(tl * QC + c) * 64]);
#pragma unroll
    for (int m = 0; m < VM; ++m) vf[m] = __builtin_nontemporal_load(&kp[4 * DH + m * 64]);
  };
  auto use_blk = [&](int blk, bf16x8(&kf)[2][QC], bf16x8(&vf)[VM]) {
    floatx4 S[2];
#pragma unroll
    for (int tl = 0; tl < 2; ++tl) {
      S[tl] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int c = 0; c < QC; ++c) S[tl] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[tl][c], qf[c], S[tl], 0, 0, 0);
    }
    // S[tl][i] = q . k of key  blk*32 + 16*tl + 4*grp + i
    float sv[8];
    bool ok[8];
    float bm = -1.0e30f;
#pragma unroll
    for (int tl = 0; tl < 2; ++tl)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int key = blk * 32 + 16 * tl + 4 * grp + i;
        ok[tl * 4 + i] = key < len;
        sv[tl * 4 + i] = S[tl][i] * scale;
        if (ok[tl * 4 + i]) bm = fmaxf(bm, sv[tl * 4 + i]);
      }
    bm = fmaxf(bm, __shfl_xor(bm, 16));
    bm = fmaxf(bm, __shfl_xor(bm, 32));
    const float m_new = fmaxf(m_run, bm);
    const float alpha = __expf(m_run - m_new);
    float p[8], ps = 0.f;
    uint32_t pk[4];
#pragma unroll
    for (int j = 0; j < 8; ++j) p[j] = ok[j] ? __expf(sv[j] - m_new) : 0.f;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      pk[j] = pack2(p[2 * j], p[2 * j + 1]);
      ps += bf2f(pk[j] & 0xffffu) + bf2f(pk[j] >> 16);  // the denominator uses the rounded weights
    }
    l_run = l_run * alpha + ps;
    m_run = m_new;
    const uint32x4 pku = uint32x4{pk[0], pk[1], pk[2], pk[3]};
    const bf16x8 pv = __builtin_bit_cast(bf16x8, pku);
#pragma unroll
    for (int m = 0; m < VM; ++m) {
      O[m] *= alpha;
      O[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[m], pv, O[m], 0, 0, 0);
    }
  };
  // With 64-wide heads a second block fits in the registers (four waves per SIMD leave 128), so the next block's
  // loads are in flight while this one is used: rows of a few blocks per wave are otherwise one full memory
  // latency per block.  128-wide heads would need 64 more registers than four waves per SIMD allow.
  if constexpr (DH == 64) {
    bf16x8 kf0[2][QC], vf0[VM], kf1[2][QC], vf1[VM];
    int blk = my_lo + wave;
    if (blk < my_hi) {
      load_blk(blk, kf0, vf0);
      while (true) {
        if (blk + NW < my_hi) load_blk(blk + NW, kf1, vf1);
        use_blk(blk, kf0, vf0);
        if (blk + NW >= my_hi) break;
        if (blk + 2 * NW < my_hi) load_blk(blk + 2 * NW, kf0, vf0);
        use_blk(blk + NW, kf1, vf1);
        if (blk + 2 * NW >= my_hi) break;
        blk += 2 * NW;
      }
    }
  } else {
    for (int blk = my_lo + wave; blk < my_hi; blk += NW) {
      bf16x8 kf[2][QC], vf[VM];
      load_blk(blk, kf, vf);
      use_blk(blk, kf, vf);
    }
  }
  // O[m][i] = sum_key p * v[key][16*m + 4*grp + i]   (same in all 16 columns)
  l_run += __shfl_xor(l_run, 16);
  l_run += __shfl_xor(l_run, 32);
  if (lane == 0) { sm_m[wave] = m_run; sm_l[wave] = l_run; }
  if ((lane & 15) == 0) {
#pragma unroll
    for (int m = 0; m < VM; ++m)
#pragma unroll
      for (int i = 0; i < 4; ++i) sm_o[wave][16 * m + 4 * grp + i] = O[m][i];
  }
  {  // q . k_t: the first waves (the threads below DH) hold the products
    float dot = 0.f;
#pragma unroll
    for (int i = 0; i < EPT; ++i) dot += q_e[i] * k_e[i];
    for (int o = 32; o > 0; o >>= 1) dot += __shfl_xor(dot, o);
    if (lane == 0) sm_dot[wave] = dot;
  }
  __syncthreads();
  constexpr int NDW = NW < DH / 64 ? NW : DH / 64;  // waves whose sm_dot holds products
#pragma unroll
  for (int i = 0; i < EPT; ++i) {
    const int e = (int)threadIdx.x + i * NW * 64;
    if (e >= DH) continue;
    float M = sm_m[0];
    for (int w = 1; w < NW; ++w) M = fmaxf(M, sm_m[w]);
    float s_t = 0.f;
    if (with_new) {
      for (int w = 0; w < NDW; ++w) s_t += sm_dot[w];
      s_t *= scale;
      M = fmaxf(M, s_t);
    }
    float num = 0.f, den = 0.f;
    for (int w = 0; w < NW; ++w) {
      const float f = __expf(sm_m[w] - M);
      num += f * sm_o[w][e];
      den += f * sm_l[w];
    }
    if (with_new) {
      const float f = __expf(s_t - M);
      num += f * v_e[i];
      den += f;
    }
    if (a.splits == 1) {
      const float r = den > 0.f ? num / den : 0.f;
      a.o[d_act_index(b, h * DH + e, d)] = (bf16_t)f2bf(r);
    } else {
      float *pp = a.part + ((long)blockIdx.y * gridDim.x + (long)b * H + h) * (DH + 4);
      pp[e] = num;
      if (e == 0) { pp[DH] = M; pp[DH + 1] = den; }
    }
    if (with_new) {
      bf16_t *pg = a.pool + (long)page_t * a.kv.page_elems;
      const int tt = len % a.kv.page_tokens;
      pg[kv_k_off(h, tt, e, a.kv)] = k_bits[i];
      pg[kv_v_off(h, tt, e, a.kv)] = v_bits[i];
    }
  }
}

// merges the splits of a (row, head); at most 16, all of them requested together
template <int DH>
__global__ __launch_bounds__(DH) void k_attn_merge(AttnArgs a) {
  const int H = a.kv.H, b = blockIdx.x / H, h = blockIdx.x % H, d = H * DH, e = threadIdx.x;
  float m[16], n[16], l[16];
#pragma unroll
  for (int s = 0; s < 16; ++s)
    if (s < a.splits) {
      const float *pp = a.part + ((long)s * gridDim.x + blockIdx.x) * (DH + 4);
      m[s] = pp[DH];
      l[s] = pp[DH + 1];
      n[s] = pp[e];
    }
  float M = -1.0e30f;
#pragma unroll
  for (int s = 0; s < 16; ++s)
    if (s < a.splits) M = fmaxf(M, m[s]);
  float num = 0.f, den = 0.f;
#pragma unroll
  for (int s = 0; s < 16; ++s)
    if (s < a.splits) {
      const float f = __expf(m[s] - M);
      num += f * n[s];
      den += f * l[s];
    }
  a.o[d_act_index(b, h * DH + e, d)] = (bf16_t)f2bf(den > 0.f ? num / den : 0.f);
}

void bf16_attention(hipStream_t s, const AttnArgs &a) {
  const dim3 grid(a.B * a.kv.H, a.splits);
  const int nw = a.waves >= 16 ? 16 : a.waves >= 8 ? 8 : a.waves >= 4 ? 4 : a.waves >= 2 ? 2 : 1;
  if (a.kv.dh == 64) {
    if (nw == 1) SKD_LAUNCH((k_attention<64, 1>), grid, dim3(64), 0, s, a);
    else if (nw == 16) SKD_LAUNCH((k_attention<64, 16>), grid, dim3(1024), 0, s, a);
    else if (nw == 8) SKD_LAUNCH((k_attention<64, 8>), grid, dim3(512), 0, s, a);
    else if (nw == 2) SKD_LAUNCH((k_attention<64, 2>), grid, dim3(128), 0, s, a);
    else SKD_LAUNCH((k_attention<64, 4>), grid, dim3(256), 0, s, a);
    if (a.splits > 1 && a.merge) SKD_LAUNCH(k_attn_merge<64>, dim3(a.B * a.kv.H), dim3(64), 0, s, a);
  } else {
    if (nw == 1) SKD_LAUNCH((k_attention<128, 1>), grid, dim3(64), 0, s, a);
    else if (nw == 16) SKD_LAUNCH((k_attention<128, 16>), grid, dim3(1024), 0, s, a);
    else if (nw == 8) SKD_LAUNCH((k_attention<128, 8>), grid, dim3(512), 0, s, a);
    else if (nw == 2) SKD_LAUNCH((k_attention<128, 2>), grid, dim3(128), 0, s, a);
    else SKD_LAUNCH((k_attention<128, 4>), grid, dim3(256), 0, s, a);
    if (a.splits > 1 && a.merge) SKD_LAUNCH(k_attn_merge<128>, dim3(a.B * a.kv.H), dim3(128), 0, s, a);
  }
}

// ------------------------------------------------------------------ causal attention over a whole prompt
// Same fragments as k_attention, but the 16 MFMA columns carry 16 different queries (consecutive positions of one
// sequence).  A workgroup is NW waves on 32 NW consecutive positions of one sequence and one head, a wave two 16-query
// tiles.  The waves share the K and V blocks: a ring of NS stages (32 keys, K and V, one contiguous piece of a page)
// is filled by LDS-direct loads ahead of their use, one bare barrier per stage; each wave loading its own fragments
// asked four times as much of the CU's memory path (64 bytes per clock).
// Four waves, and a ring of three stages; where no sequence has more than 32 or 64 positions one or two, and a stage for
// each of their blocks.  As workgroups of four with waves that have nothing to do, 128 prompts of 16 tokens (32 heads of
// 128) took 24.5 us instead of 17.4, of 48 tokens (32 heads of 64) 24.0 instead of 20.9.
// Positions of a wave start at a multiple of 32, so exactly one block, its last, needs the causal mask.
// The softmax works in units of log2 and against a reference m that is raised only when a score exceeds it by more than
// 8 (weights up to 2^8: bf16 and fp32 keep their relative precision), so that most blocks need no cross-lane maximum
// and no rescaling of the 64 accumulators; the denominator comes from the matrix cores (a row of ones), summed over the
// rounded weights as the numerator is.
constexpr int att_stages(int NW) { return NW == 4 ? 3 : NW; }

template <int DH, int NW>
__global__ __launch_bounds__(NW * 64, 3) void k_attention_rows(AttnRowsArgs a) {
  constexpr int QC = DH / 32, VM = DH / 16, NT = 2;
  constexpr int NS = att_stages(NW), AHEAD = NW == 4 ? NS - 1 : NS;  // stages requested before the first is used
  constexpr int FR = 2 * QC + VM, LPW = FR / NW;  // fragments per stage, loads per wave and stage
  extern __shared__ bf16x8 ring[];                // [NS][FR][64 lanes]
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int grp = lane >> 4, col = lane & 15;
  const int h = blockIdx.x, b = blockIdx.y % a.B;
  const int g0 = (int)(gridDim.y / a.B - 1 - blockIdx.y / a.B) * (32 * NW);  // longest key ranges are dispatched first
  const int len = a.rm.P - a.rm.start[b];                                    // real positions of this sequence
  if (g0 >= len) return;
  const int d = a.kv.H * DH;
  const int nblk = (min(g0 + 32 * NW - 1, len - 1) >> 5) + 1;  // blocks the workgroup walks (NW < 4: at most NW, g0 is 0)
  const int p0 = g0 + 32 * wave;                       // first position of this wave
  const int mine = p0 < len ? p0 >> 5 : -1;            // this wave's last block
  const long row0 = (long)a.rm.first_row[b] + p0;
  const int bpp = a.kv.page_tokens >> 5;
  const int32_t *bt_row = a.bt_layer + (long)b * a.kv.max_pages;
  const float c = 1.4426950408889634f / sqrtf((float)DH);  // scores -> log2 of the weights

  floatx4 O[NT][VM], L[NT];
  float m_ref[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    m_ref[t] = -1.0e30f;
    L[t] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int m = 0; m < VM; ++m) O[t][m] = floatx4{0.f, 0.f, 0.f, 0.f};
  }
  bf16x8 ones;
#pragma unroll
  for (int i = 0; i < 8; ++i) ones[i] = (__bf16)1.0f;

  bf16x8 qf[NT][QC];
  auto load_q = [&]() {
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int k = 0; k < QC; ++k) {
        qf[t][k] = bf16x8{0, 0, 0, 0, 0, 0, 0, 0};
        if (p0 + 16 * t < len)  // the tile exists
          qf[t][k] = ((const bf16x8 *)a.q)[(((row0 >> 4) + t) * (d >> 5) + ((h * DH) >> 5) + k) * 64 + act_lane(lane)];
      }
  };
  if constexpr (NW < 4) load_q();  // (four waves: behind the ring, 5 % faster for one sequence of 1024 positions)

  // blocks are issued in order: block ib of page ip comes next.  Lane l holds page 64 w + l of the row for the window w
  // of 64 pages that ip is in; a window is waited for where it is loaded (waited for at its use, in the loop, the
  // compiler would wait for the ring's loads as well).
  // With one or two blocks the pages are scalar loads.
  int ip = 0, ib = 0, pages = 0;
  const int page0 = NW < 4 ? bt_row[0] : 0, page1 = NW < 4 ? bt_row[min(1, a.kv.max_pages - 1)] : 0;
  auto issue = [&](int blk) {
    int page = ip ? page1 : page0;
    if constexpr (NW == 4) {
      if (ib == 0 && (ip & 63) == 0) {
        pages = ip + lane < a.kv.max_pages ? bt_row[ip + lane] : 0;
        asm volatile("" : "+v"(pages));
      }
      page = __builtin_amdgcn_readlane(pages, ip & 63);
    }
    const bf16x8 *src = (const bf16x8 *)(a.pool + (long)page * a.kv.page_elems + (long)h * a.kv.page_tokens * (DH * 2) +
                                         (long)ib * (64 * DH)) + wave * LPW * 64;
    bf16x8 *dst = ring + ((blk % NS) * FR + wave * LPW) * 64;
#pragma unroll
    for (int i = 0; i < LPW; ++i) {
      if (NW == 1 && i >= QC && i < 2 * QC && len <= 16) continue;  // keys 16 .. 31: the mask covers them whatever LDS holds
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)&(src + i * 64)[lane],
                                       (__attribute__((address_space(3))) void *)(dst + i * 64), 16, 0, 0);
    }
    if (++ib == bpp) { ib = 0; ++ip; }
  };
#pragma unroll
  for (int i = 0; i < AHEAD; ++i)
    if (i < nblk) issue(i);
  if constexpr (NW == 4) load_q();
  // the queries arrive before the loop: waited for inside it, they would make the compiler wait for every load in flight
  wait_vmcnt<0>();
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int k = 0; k < QC; ++k) asm volatile("" : "+v"(qf[t][k]));
  auto use = [&](int blk, bool diagonal) {
    const bf16x8 *kv = ring + (blk % NS) * (FR * 64) + lane;
    floatx4 S[NT][2];
#pragma unroll
    for (int tl = 0; tl < 2; ++tl) {
      bf16x8 kf[QC];
#pragma unroll
      for (int k = 0; k < QC; ++k) kf[k] = kv[(tl * QC + k) * 64];
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        S[t][tl] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < QC; ++k) S[t][tl] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[k], qf[t][k], S[t][tl], 0, 0, 0);
      }
    }
    // S[t][tl][i] = query 16 t + col of this wave . key 32 blk + 16 tl + 4 grp + i
    bf16x8 pv[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      if (diagonal) {
#pragma unroll
        for (int tl = 0; tl < 2; ++tl)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (16 * tl + 4 * grp + i > 16 * t + col) S[t][tl][i] = -1.0e30f;
      }
      float bm = fmaxf(fmaxf(fmaxf(S[t][0][0], S[t][0][1]), fmaxf(S[t][0][2], S[t][0][3])),
                       fmaxf(fmaxf(S[t][1][0], S[t][1][1]), fmaxf(S[t][1][2], S[t][1][3]))) * c;
      if (__any(bm > m_ref[t] + 8.0f)) {
        bm = fmaxf(bm, __shfl_xor(bm, 16));  // lanes 16 and 32 apart hold the same query
        bm = fmaxf(bm, __shfl_xor(bm, 32));
        const float m_new = fmaxf(m_ref[t], bm);
        const float alpha = __builtin_amdgcn_exp2f(m_ref[t] - m_new);
        m_ref[t] = m_new;
        L[t] *= alpha;
#pragma unroll
        for (int m = 0; m < VM; ++m) O[t][m] *= alpha;
      }
      uint32_t pk[4];
#pragma unroll
      for (int tl = 0; tl < 2; ++tl)
#pragma unroll
        for (int i = 0; i < 4; i += 2)
          pk[tl * 2 + i / 2] = pack2(__builtin_amdgcn_exp2f(__builtin_fmaf(S[t][tl][i], c, -m_ref[t])),
                                     __builtin_amdgcn_exp2f(__builtin_fmaf(S[t][tl][i + 1], c, -m_ref[t])));
      pv[t] = __builtin_bit_cast(bf16x8, (uint32x4{pk[0], pk[1], pk[2], pk[3]}));
      L[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, pv[t], L[t], 0, 0, 0);
    }
#pragma unroll
    for (int m = 0; m < VM; ++m) {
      const bf16x8 vf = kv[(2 * QC + m) * 64];
#pragma unroll
      for (int t = 0; t < NT; ++t) O[t][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, pv[t], O[t][m], 0, 0, 0);
    }
  };
  auto open = [&](int blk) {
    // this wave's loads of stage blk have landed once only those of the later stages in flight are outstanding
    if (blk + 1 < nblk) wait_vmcnt<LPW>();
    else wait_vmcnt<0>();
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): this wave's reads of stage blk - 1
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if constexpr (NW == 4)
      if (blk + AHEAD < nblk) issue(blk + AHEAD);  // into the slot of stage blk - 1
  };
  int blk = 0;
  for (; blk <= mine; ++blk) {
    open(blk);
    use(blk, blk == mine);
  }
  for (; blk < nblk; ++blk) open(blk);  // blocks that only the other waves need
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    if (p0 + 16 * t >= len) continue;
    // O[t][m][i] = numerator of query `col` of tile t, head-dim element 16m + 4grp + i; L[t]: its denominator
    const float inv = L[t][0] > 0.f ? 1.0f / L[t][0] : 0.f;
#pragma unroll
    for (int m = 0; m < VM; ++m) {
      const uint2 pk = make_uint2(pack2(O[t][m][0] * inv, O[t][m][1] * inv), pack2(O[t][m][2] * inv, O[t][m][3] * inv));
      *(uint2 *)&a.o[d_act_index(row0 + 16 * t + col, h * DH + 16 * m + 4 * grp, d)] = pk;
    }
  }
}

template <int DH, int NW>
static void launch_attention_rows(hipStream_t s, const AttnRowsArgs &a) {
  const dim3 grid(a.kv.H, a.B * ((a.max_len + 32 * NW - 1) / (32 * NW)));
  const size_t lds = (size_t)att_stages(NW) * 32 * DH * 2 * sizeof(bf16_t);  // 8 or 16 KiB a stage
  SKD_LAUNCH((k_attention_rows<DH, NW>), grid, dim3(64 * NW), lds, s, a);
}
void bf16_attention_rows(hipStream_t s, const AttnRowsArgs &a) {
#define SKD_ATT(DH) (a.max_len <= 32 ? launch_attention_rows<DH, 1>(s, a) : a.max_len <= 64 ? launch_attention_rows<DH, 2>(s, a) : launch_attention_rows<DH, 4>(s, a))
  if (a.kv.dh == 64) SKD_ATT(64);
  else SKD_ATT(128);
#undef SKD_ATT
}

// ------------------------------------------------------------------ row kernels of the batched prompt
// The row map of a prompt from by-value kernel arguments (at most 128 sequences): workgroup b fills the rows of
// sequence b, the last one the rows past the last sequence.  Replaces four pageable copies and two host waits.
__global__ __launch_bounds__(256) void k_prompt_map(PromptMap pm, int B, int rows, int rows_pad, int P, KvGeom kv,
                                                    int32_t *start, int32_t *order, int32_t *first, int32_t *seq,
                                                    CacheTile *tiles) {
  const int b = blockIdx.x;
  int lo = rows, n = rows_pad - rows, val = -1;
  if (b < B) {
    lo = pm.first[b];
    n = ((P - pm.start[b]) + 15) / 16 * 16;
    val = b;
    if (threadIdx.x == 0) {
      start[b] = pm.start[b];
      order[b] = pm.order[b];
      first[b] = lo;
    }
  }
  for (int i = threadIdx.x; i < n; i += 256) seq[lo + i] = val;
  for (int i = threadIdx.x; i < n >> 4; i += 256) {
    const int pos = i * 16, page = pos / kv.page_tokens;  // real position of the tile's first row
    tiles[(lo >> 4) + i] = val < 0 ? CacheTile::none()
                                   : CacheTile::of(b * kv.max_pages + page, pos - page * kv.page_tokens, min(16, P - pm.start[b] - pos));
  }
}
void bf16_prompt_map(hipStream_t s, const PromptMap &pm, int B, int rows, int rows_pad, int P, const KvGeom &kv, int32_t *start,
                     int32_t *order, int32_t *first, int32_t *seq, CacheTile *tiles) {
  SKD_LAUNCH(k_prompt_map, dim3(B + 1), dim3(256), 0, s, pm, B, rows, rows_pad, P, kv, start, order, first, seq, tiles);
}

__global__ __launch_bounds__(1024) void k_embed_ln_rows_wide(const int32_t *tokens, RowMap rm, const bf16_t *tok_emb,
                                                        const bf16_t *pos_emb, const float *g, const float *bt, float *x,
                                                        bf16_t *a_out, int B, int d, int V) {
  __shared__ float sh[32];
  const int row = blockIdx.x, d4 = d >> 2;
  const int b = rm.seq[row];
  if (b < 0) return;
  const int pos = row - rm.first_row[b];  // real position = position id
  if (pos >= rm.P - rm.start[b]) {  // padding of the sequence's last 16-row tile: zero (no other row ever depends on it)
    for (int c = threadIdx.x; c < d4; c += blockDim.x) {
      ((floatx4 *)x)[(long)row * d4 + c] = floatx4{0.f, 0.f, 0.f, 0.f};
      *(uint2 *)&a_out[d_act_index(row, 4 * c, d)] = make_uint2(0, 0);
    }
    return;
  }
  int tok = tokens[(long)(rm.start[b] + pos) * B + b];
  tok = tok < 0 ? 0 : (tok >= V ? V - 1 : tok);
  const uint2 *te = (const uint2 *)(tok_emb + (long)tok * d), *pe = (const uint2 *)(pos_emb + (long)pos * d);
  floatx4 v[LN_NC], gv[LN_NC], bv[LN_NC];
#pragma unroll
  for (int i = 0; i < LN_NC; ++i) {
    const int c = (int)(threadIdx.x + blockDim.x * i);
    if (c < d4) {
      const uint2 aa = te[c], p = pe[c];
      gv[i] = ((const floatx4 *)g)[c];
      bv[i] = ((const floatx4 *)bt)[c];
      v[i] = floatx4{bf2f(aa.x & 0xffffu) + bf2f(p.x & 0xffffu), bf2f(aa.x >> 16) + bf2f(p.x >> 16),
                     bf2f(aa.y & 0xffffu) + bf2f(p.y & 0xffffu), bf2f(aa.y >> 16) + bf2f(p.y >> 16)};
      ((floatx4 *)x)[(long)row * d4 + c] = v[i];
    }
  }
  ln_finish_row(v, gv, bv, d, row, a_out, sh);
}

__global__ __launch_bounds__(1024) void k_ln_rows_wide(const float *x, const float *g, const float *bt, bf16_t *a_out, int d) {
  __shared__ float sh[32];
  const int row = blockIdx.x, d4 = d >> 2;
  floatx4 v[LN_NC], gv[LN_NC], bv[LN_NC];
#pragma unroll
  for (int i = 0; i < LN_NC; ++i) {
    const int c = (int)(threadIdx.x + blockDim.x * i);
    if (c < d4) {
      v[i] = ((const floatx4 *)x)[(long)row * d4 + c];
      gv[i] = ((const floatx4 *)g)[c];
      bv[i] = ((const floatx4 *)bt)[c];
    }
  }
  ln_finish_row(v, gv, bv, d, row, a_out, sh);
}

// LayerNorm of the prompt rows, one wave per row: the row stays in registers (NC chunks of 256 columns), and so do gain and
// offset, requested with it; the statistics need no barrier.  A row's 64-byte pieces of the 16 x 32 tiles are stored
// directly: two neighbouring rows share a 128-byte line and leave their workgroup at about the same time.  EMBED: the row
// is the sum of its token and position embeddings (zero in the padding of a sequence's last tile) and is stored to x.
// Memory-bound where the rows fill the chip, else one latency chain per row.  NC is exact: with the next of 4, 8 or 16 and
// a test per chunk, and gain and offset loaded behind the statistics, 16384 rows of 2048 took 93 us instead of 63 (a
// workgroup of 16 waves that put whole tiles together in LDS: 75), 64 rows of 4096 with the embedding 15 instead of 8.
template <int NC, bool EMBED>
__global__ __launch_bounds__(512) void k_ln_rows(const int32_t *tokens, RowMap rm, const bf16_t *tok_emb, const bf16_t *pos_emb,
                                                  float *x, const float *g, const float *bt, bf16_t *a_out, int B, int V) {
  constexpr int d = 256 * NC;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const long row = (long)blockIdx.x * (blockDim.x >> 6) + wave;
  floatx4 *xr = (floatx4 *)x + row * (d >> 2) + lane;
  uint2 *out = (uint2 *)(a_out + (row >> 4) * 16 * d) + (lane >> 3) * 128 + (row & 15) * 8 + (lane & 7);
  floatx4 v[NC], gv[NC], bv[NC];
  if constexpr (EMBED) {
    const int b = rm.seq[row];
    if (b < 0) return;
    const int pos = (int)row - rm.first_row[b];  // real position = position id
    if (pos >= rm.P - rm.start[b]) {
#pragma unroll
      for (int i = 0; i < NC; ++i) {
        xr[64 * i] = floatx4{0.f, 0.f, 0.f, 0.f};
        out[(long)i * 1024] = make_uint2(0, 0);
      }
      return;
    }
    int tok = tokens[(long)(rm.start[b] + pos) * B + b];
    tok = tok < 0 ? 0 : (tok >= V ? V - 1 : tok);
    const uint2 *te = (const uint2 *)(tok_emb + (long)tok * d) + lane, *pe = (const uint2 *)(pos_emb + (long)pos * d) + lane;
    uint2 tv[NC], pv[NC];
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      tv[i] = te[64 * i];
      pv[i] = pe[64 * i];
    }
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      v[i] = floatx4{bf2f(tv[i].x & 0xffffu) + bf2f(pv[i].x & 0xffffu), bf2f(tv[i].x >> 16) + bf2f(pv[i].x >> 16),
                     bf2f(tv[i].y & 0xffffu) + bf2f(pv[i].y & 0xffffu), bf2f(tv[i].y >> 16) + bf2f(pv[i].y >> 16)};
      xr[64 * i] = v[i];
    }
  } else {
#pragma unroll
    for (int i = 0; i < NC; ++i) v[i] = xr[64 * i];
  }
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    gv[i] = ((const floatx4 *)g)[lane + 64 * i];
    bv[i] = ((const floatx4 *)bt)[lane + 64 * i];
  }
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < NC; ++i) s += (v[i][0] + v[i][1]) + (v[i][2] + v[i][3]);
  const float mean = wave_sum_f(s) / d;
  float q = 0.f;
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    const floatx4 t = v[i] - mean;
    q += (t[0] * t[0] + t[1] * t[1]) + (t[2] * t[2] + t[3] * t[3]);
  }
  const float rstd = 1.0f / sqrtf(wave_sum_f(q) / d + 1e-5f);
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    const floatx4 y = (v[i] - mean) * rstd * gv[i] + bv[i];
    out[(long)i * 1024] = make_uint2(pack2(y[0], y[1]), pack2(y[2], y[3]));
  }
}
// Up to 1024 rows one row per workgroup (every CU gets rows: 64, 512, 1024 rows of 4096 with the embedding 6.6, 9.6, 13.9 us
// against 8.3, 10.3, 15.3 with four), beyond four, or eight rows of 3072 and more (16384 rows of 4096 with the embedding:
// 173 us with one, 145 with four, 127 with eight; of 2048: 88, 81, 82).
template <bool EMBED>
static bool launch_ln_rows(hipStream_t s, const int32_t *tokens, RowMap rm, int rows, const bf16_t *tok_emb, const bf16_t *pos_emb,
                            float *x, const float *g, const float *b, bf16_t *a_out, int B, int d, int V) {
  if (rows % 16 || d % 256 || d < 256 || d > 4096) return false;  // other widths: one workgroup per row
  const int per = rows <= 1024 ? 1 : d >= 3072 ? 8 : 4;
  const dim3 grid(rows / per), blk(64 * per);
  switch (d / 256) {
#define SKD_NC(NC) \
  case NC: SKD_LAUNCH((k_ln_rows<NC, EMBED>), grid, blk, 0, s, tokens, rm, tok_emb, pos_emb, x, g, b, a_out, B, V); break;
    SKD_NC(1) SKD_NC(2) SKD_NC(3) SKD_NC(4) SKD_NC(5) SKD_NC(6) SKD_NC(7) SKD_NC(8)
    SKD_NC(9) SKD_NC(10) SKD_NC(11) SKD_NC(12) SKD_NC(13) SKD_NC(14) SKD_NC(15) SKD_NC(16)
#undef SKD_NC
  }
  return true;
}

// Hidden state of each sequence's last prompt position: x_out[b] = its row of x_rows (+ bias + the partial sums of the
// last projection when split > 0), and its LayerNorm.
__global__ __launch_bounds__(1024) void k_last_rows_ln(const float *x_rows, RowMap rm, const float *partial, int split,
                                                       int stride, const float *bias, const float *g, const float *bt,
                                                       float *x_out, bf16_t *a_out, int d) {
  __shared__ float sh[32];
  const int b = blockIdx.x, d4 = d >> 2;
  const long row = (long)rm.first_row[b] + (rm.P - rm.start[b]) - 1;
  floatx4 v[LN_NC], gv[LN_NC], bv[LN_NC];
#pragma unroll
  for (int i = 0; i < LN_NC; ++i) {
    const int c = (int)(threadIdx.x + blockDim.x * i);
    if (c < d4) {
      v[i] = ((const floatx4 *)x_rows)[row * d4 + c];
      gv[i] = ((const floatx4 *)g)[c];
      bv[i] = ((const floatx4 *)bt)[c];
      if (split) {
        floatx4 acc = ((const floatx4 *)partial)[row * d4 + c];
        for (int sp = 1; sp < split; ++sp) acc += ((const floatx4 *)partial)[((long)sp * stride + row) * d4 + c];
        v[i] += acc + ((const floatx4 *)bias)[c];
      }
      ((floatx4 *)x_out)[(long)b * d4 + c] = v[i];
    }
  }
  ln_finish_row(v, gv, bv, d, b, a_out, sh);
}

void bf16_embed_ln_rows(hipStream_t s, const int32_t *tokens, RowMap rm, int rows, const bf16_t *tok_emb,
                        const bf16_t *pos_emb, const float *g, const float *b, float *x, bf16_t *a_out, int B, int d,
                        int V) {
  if (launch_ln_rows<true>(s, tokens, rm, rows, tok_emb, pos_emb, x, g, b, a_out, B, d, V)) return;
  SKD_LAUNCH(k_embed_ln_rows_wide, dim3(rows), dim3(row_threads(d)), 0, s, tokens, rm, tok_emb, pos_emb, g, b, x, a_out, B, d, V);
}
void bf16_ln_rows(hipStream_t s, float *x, const float *g, const float *b, bf16_t *a_out, int rows, int d) {
  if (launch_ln_rows<false>(s, nullptr, RowMap{}, rows, nullptr, nullptr, x, g, b, a_out, 0, d, 0)) return;
  SKD_LAUNCH(k_ln_rows_wide, dim3(rows), dim3(row_threads(d)), 0, s, x, g, b, a_out, d);
}
void bf16_last_rows_ln(hipStream_t s, const float *x_rows, RowMap rm, const float *partial, int split, int stride,
                       const float *bias, const float *g, const float *b, float *x_out, bf16_t *a_out, int B, int d) {
  SKD_LAUNCH(k_last_rows_ln, dim3(B), dim3(row_threads(d)), 0, s, x_rows, rm, partial, split, stride, bias, g, b, x_out, a_out, d);
}

// ------------------------------------------------------------------ argmax over workgroup partials
// One workgroup per row; the token goes to both destinations (tokens2 may be null).  A wave reduces without barriers, the
// four results meet in LDS once.
__global__ __launch_bounds__(256) void k_argmax_final(const float *pmax, const int32_t *pidx, int groups, int B_pad,
                                                      int32_t *tokens, int32_t *tokens2) {
  __shared__ float sv[4];
  __shared__ int si[4];
  const int b = blockIdx.x;
  float best = -3.0e38f;
  int bi = 0x7fffffff;
  auto take = [&](float v, int i) {  // larger value, lower index on ties
    if (v > best || (v == best && i < bi)) { best = v; bi = i; }
  };
#pragma unroll 4
  for (int g = threadIdx.x; g < groups; g += 256) take(pmax[(long)g * B_pad + b], pidx[(long)g * B_pad + b]);
  for (int o = 32; o > 0; o >>= 1) take(__shfl_xor(best, o), __shfl_xor(bi, o));
  if ((threadIdx.x & 63) == 0) {
    sv[threadIdx.x >> 6] = best;
    si[threadIdx.x >> 6] = bi;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 4; ++w) take(sv[w], si[w]);
    tokens[b] = bi;
    if (tokens2) tokens2[b] = bi;
  }
}
void bf16_argmax_final(hipStream_t s, const float *pmax, const int32_t *pidx, int groups, int B_pad, int32_t *tokens,
                       int32_t *tokens2, int B) {
  SKD_LAUNCH(k_argmax_final, dim3(B), dim3(256), 0, s, pmax, pidx, groups, B_pad, tokens, tokens2);
}

// Logits from partial sums along K ([split][B_pad][N], N = whole 16-row tiles; added in order) and the greedy token, one
// workgroup per row: the end of an LM head whose tiles would leave most CUs without a workgroup.  Logits and tokens are
// optional, as in k_argmax_final; `whole`: rows of logits can be written 16 bytes at a time.
__global__ __launch_bounds__(256) void k_logits_sum(const float *partial, int split, int B_pad, int N, int V, float *logits,
                                                    bool whole, int32_t *tokens, int32_t *tokens2) {
  __shared__ float sv[4];
  __shared__ int si[4];
  const int b = blockIdx.x, n4 = N >> 2;
  const long part = (long)B_pad * n4;
  const floatx4 *p4 = (const floatx4 *)partial + (long)b * n4;
  float best = -3.0e38f;
  int bi = 0x7fffffff;
  auto take = [&](float v, int i) {  // larger value, lower index on ties
    if (v > best || (v == best && i < bi)) { best = v; bi = i; }
  };
  for (int c = threadIdx.x; c < n4; c += 256) {
    floatx4 p[LOGITS_SPLIT];
#pragma unroll
    for (int k = 0; k < LOGITS_SPLIT; ++k)
      if (k < split) p[k] = p4[k * part + c];
    floatx4 v = p[0];
#pragma unroll
    for (int k = 1; k < LOGITS_SPLIT; ++k)
      if (k < split) v += p[k];
    float *to = logits ? logits + (long)b * V + 4 * c : nullptr;
    if (to && whole && 4 * c < V) *(floatx4 *)to = v;
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (4 * c + k < V) {
        if (to && !whole) to[k] = v[k];
        take(v[k], 4 * c + k);
      }
  }
  if (!tokens) return;
  for (int o = 32; o > 0; o >>= 1) take(__shfl_xor(best, o), __shfl_xor(bi, o));
  if ((threadIdx.x & 63) == 0) {
    sv[threadIdx.x >> 6] = best;
    si[threadIdx.x >> 6] = bi;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 4; ++w) take(sv[w], si[w]);
    tokens[b] = bi;
    if (tokens2) tokens2[b] = bi;
  }
}
void bf16_logits_sum(hipStream_t s, const float *partial, int split, int B_pad, int N, int V, float *logits, int32_t *tokens,
                     int32_t *tokens2, int B) {
  const bool whole = V % 4 == 0 && ((uintptr_t)logits & 15) == 0;
  SKD_LAUNCH(k_logits_sum, dim3(B), dim3(256), 0, s, partial, split, B_pad, N, V, logits, whole, tokens, tokens2);
}

// ------------------------------------------------------------------ weight preparation
template <typename T>
__device__ inline float src_to_f(const T *p, long i);
template <>
__device__ inline float src_to_f<float>(const float *p, long i) { return p[i]; }
template <>
__device__ inline float src_to_f<bf16_t>(const bf16_t *p, long i) { return bf2f(p[i]); }

// one thread per 8-element lane slot of the destination
template <typename T>
__global__ void k_prep_frag(const T *src, bf16_t *dst, long N, long K, long N_pad, int G) {
  const long slot = (long)blockIdx.x * blockDim.x + threadIdx.x;
  const long Kf = K >> 5;
  if (slot >= (N_pad >> 4) * Kf * 64) return;
  const int lane = slot & 63;
  const long frag = slot >> 6, kf = (frag / G) % Kf, nt = frag / (G * Kf) * G + frag % G;
  const long row = nt * 16 + (lane & 15), col = kf * 32 + (lane >> 4) * 8;
  uint32_t pk[4] = {0, 0, 0, 0};
  if (row < N)
    for (int j = 0; j < 4; ++j) pk[j] = pack2(src_to_f<T>(src, row * K + col + 2 * j), src_to_f<T>(src, row * K + col + 2 * j + 1));
  *(uint32x4 *)&dst[slot * 8] = uint32x4{pk[0], pk[1], pk[2], pk[3]};
}
template <typename T>
__global__ void k_prep_rm(const T *src, bf16_t *dst, long n) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = (bf16_t)f2bf(src_to_f<T>(src, i));
}
template <typename T>
__global__ void k_prep_f32(const T *src, float *dst, long n) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = src_to_f<T>(src, i);
}
void prep_matrix_frag(hipStream_t s, const void *src, int src_is_bf16, bf16_t *dst, long N, long K, long N_pad,
                      int G) {
  const long slots = (N_pad / 16) * (K / 32) * 64;
  const dim3 grid((unsigned)((slots + 255) / 256));
  if (src_is_bf16) SKD_LAUNCH(k_prep_frag<bf16_t>, grid, dim3(256), 0, s, (const bf16_t *)src, dst, N, K, N_pad, G);
  else SKD_LAUNCH(k_prep_frag<float>, grid, dim3(256), 0, s, (const float *)src, dst, N, K, N_pad, G);
}
void prep_matrix_rm_bf16(hipStream_t s, const void *src, int src_is_bf16, bf16_t *dst, long n) {
  const dim3 grid((unsigned)((n + 255) / 256));
  if (src_is_bf16) SKD_LAUNCH(k_prep_rm<bf16_t>, grid, dim3(256), 0, s, (const bf16_t *)src, dst, n);
  else SKD_LAUNCH(k_prep_rm<float>, grid, dim3(256), 0, s, (const float *)src, dst, n);
}
void prep_to_f32(hipStream_t s, const void *src, int src_is_bf16, float *dst, long n) {
  const dim3 grid((unsigned)((n + 255) / 256));
  if (src_is_bf16) SKD_LAUNCH(k_prep_f32<bf16_t>, grid, dim3(256), 0, s, (const bf16_t *)src, dst, n);
  else SKD_LAUNCH(k_prep_f32<float>, grid, dim3(256), 0, s, (const float *)src, dst, n);
}

// ------------------------------------------------------------------ KV debug hooks (bf16 pages)
__global__ void k_kv_load_bf16(const float *K, const float *V, bf16_t *pool, const int32_t *bt_layer,
                               const int32_t *start, int cols, KvGeom g) {
  const int b = blockIdx.y, j = blockIdx.x, d = g.H * g.dh;
  const int slot = j - start[b];  // stored by real position
  if (slot < 0) return;
  const int page = bt_layer[(long)b * g.max_pages + slot / g.page_tokens];
  bf16_t *pg = pool + (long)page * g.page_elems;
  const int tt = slot % g.page_tokens;
  for (int k = threadIdx.x; k < d; k += blockDim.x) {
    const int h = k / g.dh, e = k % g.dh;
    pg[kv_k_off(h, tt, e, g)] = (bf16_t)f2bf(K ? K[((long)b * cols + j) * d + k] : 0.f);
    pg[kv_v_off(h, tt, e, g)] = (bf16_t)f2bf(V ? V[((long)b * cols + j) * d + k] : 0.f);
  }
}
__global__ void k_kv_read_bf16(const bf16_t *pool, const int32_t *bt_row, int start, float *K, float *V, KvGeom g) {
  const int j = blockIdx.x, d = g.H * g.dh, slot = j - start;
  if (slot < 0) {  // padding column: nothing is stored for it
    for (int k = threadIdx.x; k < d; k += blockDim.x) K[(long)j * d + k] = V[(long)j * d + k] = 0.f;
    return;
  }
  const bf16_t *pg = pool + (long)bt_row[slot / g.page_tokens] * g.page_elems;
  const int tt = slot % g.page_tokens;
  for (int k = threadIdx.x; k < d; k += blockDim.x) {
    const int h = k / g.dh, e = k % g.dh;
    K[(long)j * d + k] = bf2f(pg[kv_k_off(h, tt, e, g)]);
    V[(long)j * d + k] = bf2f(pg[kv_v_off(h, tt, e, g)]);
  }
}
void kv_load_bf16(hipStream_t s, const float *K, const float *V, bf16_t *pool, const int32_t *bt_layer,
                  const int32_t *start, int cols, int B, KvGeom g) {
  if (cols > 0) SKD_LAUNCH(k_kv_load_bf16, dim3(cols, B), dim3(256), 0, s, K, V, pool, bt_layer, start, cols, g);
}
void kv_read_bf16(hipStream_t s, const bf16_t *pool, const int32_t *bt_row, int start, int len, float *K, float *V,
                  KvGeom g) {
  if (len > 0) SKD_LAUNCH(k_kv_read_bf16, dim3(len), dim3(256), 0, s, pool, bt_row, start, K, V, g);
}

}  // namespace skd
