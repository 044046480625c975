// One decode column of a narrow model in ONE launch.
//
// Narrow models (a layer of a few MiB) spend a decode step on launches: five to seven kernels of 3 to 5 us per layer, each
// of which moves its bytes in well under one.  Batch rows are independent, and the 32 CUs of an XCD share an L2, so here
// every XCD takes its own share of the rows through all active layers: the workgroups that run on one XCD form a team,
// hand their results to each other through that L2 and meet at barriers whose counters live in it.  A barrier of 32
// workgroups of one XCD takes 0.83 us (of 16: 0.63; of 256 on all XCDs: 3.6 and results past the L2), a kernel boundary
// 2.5 to 3.3.  Every XCD streams all the weights, which is what limits this to narrow models (bf16_team_ok).
//
// Who is in a team is settled by the workgroups that run, not assumed from the dispatch order: each one reads its XCD's
// number and registers; the first of an XCD claims a group of rows, waits (bounded) for the expected number to register,
// closes the team and publishes its size.  Later ones leave.  So every member is running when the team is formed, and the
// barriers, which wait for members only, always end, whatever else occupies the GPU; a team may be a single workgroup, and
// an XCD that is done claims the next group that nobody has taken.  (The polls are bounded all the same.)
//
// Per layer, with a barrier behind each: q | k | v, attention, output projection, FFN1, FFN2.  Every member keeps the
// residual rows (fp32) of its group in LDS and adds the projection's output and applies LayerNorm itself, so the row
// reducers need no phase of their own.  A phase's first weights, and a wave's first K and V block, are requested between
// arrival at the barrier before it and its end.  What a phase takes (256 wide, 2 rows at 16 keys, us): q | k | v 0.6,
// attention 1.7, output projection 0.7, LayerNorm and FFN1 1.2, FFN2 1.3, LayerNorm 0.6, and 0.8 to 1.4 for each barrier
// with the stores before it; 5 to 7 for a launch's start, embeddings and end.
// Tried: workgroups beside the team that pull the coming weights into the L2 (slower by 3 to 10 %), a ninth wave that only
// polls (registers), K and V two barriers ahead (the loads behind them wait for them: slower).
// Ordering: a wave's stores have been acknowledged by the L2 (vmcnt 0) before its workgroup arrives; what other members
// have written is read with agent-scope loads, which do not look into the L1.
#include "bf16_device.h"

namespace skd {

constexpr int TEAM_WAVES = 8;
constexpr int TEAM_THREADS = 64 * TEAM_WAVES;
constexpr int TEAM_ROWS = 16;    // rows of a group: one batch tile
constexpr int TEAM_MAX_D = 512;  // 16 k-steps: the weight tile of a wave, and the K and V of a 32-key block, fit 16 fragments
constexpr int TEAM_MAX_F = 2048; // 8 waves x 8 k-steps
constexpr int TEAM_SPLITS = 4, TEAM_PARTS = 32;  // shares of one pair's keys, of all pairs (one per workgroup of the team)
constexpr int TEAM_REG_POLLS = 400;       // about 100 us: how long a leader waits for workgroups that have not started
constexpr int TEAM_MAX_POLLS = 1 << 22;   // over a second; never reached: members run until they arrive

// 16 bytes that another CU of this XCD may have written in this launch: a buffer load with sc1 (agent scope), which the L1
// does not answer.  (As two 8-byte atomic loads: 1.8 instead of 1.3 us for FFN2's phase at d = 256, f = 1024.)
__device__ inline bf16x8 load_shared16(const void *p, int byte_offset) {
  const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void *)p, 0, 0x7fffffff, 0x00027000);
  return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(r, byte_offset, 0, 16));
}
__device__ inline uint32_t ctl_load(const uint32_t *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ inline void ctl_store(uint32_t *p, uint32_t v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ inline uint32_t ctl_add(uint32_t *p, uint32_t v) { return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

typedef const TeamArgs __attribute__((address_space(4))) *ArgsPtr;
typedef const TeamLayer __attribute__((address_space(4))) *LayerPtr;

template <int N>
struct Parts { static constexpr int value = N; };  // k-steps of a wave

struct TeamLds {
  float x[TEAM_ROWS][TEAM_MAX_D];             // residual rows
  bf16_t act[TEAM_ROWS][TEAM_MAX_D + 32];     // their LayerNorm (rows 16 banks apart)
  floatx4 red[2][TEAM_WAVES][64];             // cross-wave sums, two sets in turn
  float m[TEAM_WAVES], l[TEAM_WAVES], dot[TEAM_WAVES], o[TEAM_WAVES][128];
  int row[TEAM_ROWS], start[TEAM_ROWS], tok[TEAM_ROWS];
  int all_tok[128], all_start[128], all_order[128];
  int rank, size, group;
};

template <int DH, int KD>
__global__ __launch_bounds__(TEAM_THREADS) void k_team_column(TeamArgs by_value) {
  constexpr int QC = DH / 32, VM = DH / 16, d = 32 * KD, d4 = d / 4, NC = (d4 + 63) / 64, Kd = KD, H = d / DH;
  constexpr int NW = KD > 8 ? KD : 8;  // weight fragments in registers: a tile over all of d, or an eighth of one over f
  extern __shared__ __align__(16) unsigned char team_lds[];
  TeamLds &s = *(TeamLds *)team_lds;
  int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int lane = threadIdx.x & 63, grp = lane >> 4, col = lane & 15;
  // at the start of a phase: what is derived from the lane is computed anew, not kept in registers over all phases
  // (and what comes from the arguments is loaded anew: 60 pointers and sizes do not stay in scalar registers)
  ArgsPtr ap = (ArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
  (void)by_value;
  auto anew = [](int &x) __attribute__((always_inline)) { asm volatile("" : "+s"(x)); };  // the same for uniform values
  auto phase = [&]() __attribute__((always_inline)) {
    anew(wave);
    asm volatile("" : "+v"(lane));
    asm volatile("" : "+s"(ap));
    grp = lane >> 4;
    col = lane & 15;
  };
  TeamSlot *slot = &ap->ctl->slot[__builtin_amdgcn_s_getreg(20 | (31 << 11)) & (TEAM_SLOTS - 1)];  // HW_REG_XCC_ID
  const int f = ap->f, Kf = f >> 5;

  // ---- the team
  if ((int)threadIdx.x >= 64 && (int)threadIdx.x < 64 + ap->B) {  // (while it forms: every row's token and start)
    const int b = (int)threadIdx.x - 64;
    s.all_tok[b] = ap->tokens[b];
    s.all_start[b] = ap->start[b];
    s.all_order[b] = ap->order ? ap->order[b] : b;
  }
  if (threadIdx.x == 0) {
    const int rank = (int)ctl_add(&slot->registered, 1u);
    uint32_t t = 0;
    if (rank == 0) {
      const int group = (int)ctl_add(&ap->ctl->next_group, 1u);
      int n = 1;
      if (group < ap->groups)
        for (int i = 0; i < TEAM_REG_POLLS && (n = (int)ctl_load(&slot->registered)) < ap->members; ++i) {}
      t = (uint32_t)((group + 1) << 16 | min(n, ap->members));
      ctl_store(&slot->team, t);
    } else {
      for (int i = 0; i < TEAM_MAX_POLLS && !(t = ctl_load(&slot->team)); ++i) {}
    }
    s.rank = rank;
    s.size = (int)(t & 0xffffu);
    s.group = (int)(t >> 16) - 1;
  }
  __syncthreads();
  int rank = __builtin_amdgcn_readfirstlane(s.rank), T = __builtin_amdgcn_readfirstlane(s.size);
  int group = __builtin_amdgcn_readfirstlane(s.group);
  if (rank >= T) group = ap->groups;  // more than the team needs, or late

  auto bar = [&]() __attribute__((always_inline)) {  // of the workgroup; bare: weights in flight are not waited for
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  uint32_t arrived = 0;  // by the team, once this workgroup may go on
  // of the team; what the waves do meanwhile: requests for the next phase
  auto team_bar = [&](auto meanwhile) __attribute__((always_inline)) {
    wait_vmcnt<0>();  // stores
    bar();
    arrived += (uint32_t)T;
    const bool polls = wave == TEAM_WAVES - 1 && lane == 0;  // the wave with the least to request
    if (polls) (void)ctl_add(&slot->arrived, 1u);
    meanwhile();
    if (polls)
      for (int i = 0; i < TEAM_MAX_POLLS && (int)(ctl_load(&slot->arrived) - arrived) < 0; ++i) {}
    bar();
  };

  while (group < ap->groups) {
    // ---- rows of this group: every groups-th one, from the longest down where they differ
    int R = (ap->B - group + ap->groups - 1) / ap->groups;
    if ((int)threadIdx.x < R) {
      const int b = s.all_order[group + ap->groups * (int)threadIdx.x];
      int tok = s.all_tok[b];
      s.tok[threadIdx.x] = tok < 0 ? 0 : (tok >= ap->V ? ap->V - 1 : tok);
      s.row[threadIdx.x] = b;
      s.start[threadIdx.x] = s.all_start[b];
    }
    // buffers of this group
    auto wk_q = [&]() __attribute__((always_inline)) { return ap->work.q + (long)group * TEAM_ROWS * d; };
    auto wk_kv = [&]() __attribute__((always_inline)) { return ap->work.kv + (long)group * TEAM_ROWS * 2 * d; };
    auto wk_o = [&]() __attribute__((always_inline)) { return ap->work.o + (long)group * TEAM_ROWS * d; };
    auto wk_u = [&]() __attribute__((always_inline)) { return ap->work.u + (long)group * TEAM_ROWS * f; };
    auto wk_part = [&]() __attribute__((always_inline)) { return ap->work.part + (long)group * TEAM_PARTS * (128 + 4); };
    auto wk_y = [&]() __attribute__((always_inline)) { return ap->work.y + (long)group * TEAM_ROWS * d; };

    constexpr int wg_tiles = d / 16;
    bf16x8 w[NW];  // the phase's first weight tile of this wave, or its first K and V block, requested ahead of the barrier
    bf16x8 kv[2 * QC + VM];  // K and V of 32 keys: fragments 0 .. 2 QC - 1, and those behind them
    floatx4 bias;
    // fragment (tile, k) of a layout in groups of G is base + 1024 k G bytes + 16 lane: a scalar base and a 32-bit offset
    auto tile_base = [&](const bf16_t *W, int G, int Kt, int tile, int k) __attribute__((always_inline)) {
      return (const char *)W + ((long)(tile / G) * Kt * G + (long)k * G + tile % G) * 1024;
    };
    // what a conditional load leaves as it was is not wanted any more: without this it would stay in registers
    auto forget_w = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int k = 0; k < NW; ++k) asm volatile("" : "=v"(w[k]));
    };
    auto forget_kv = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int k = 0; k < 2 * QC + VM; ++k) asm volatile("" : "=v"(kv[k]));
    };
    // a wave's own tile over all of K (q | k | v, FFN1)
    auto load_tile = [&](const bf16_t *W, int G, const float *b, int tile) __attribute__((always_inline)) {
      const char *base = tile_base(W, G, Kd, tile, 0);
      uint32_t off = 16 * lane;
#pragma unroll
      for (int k = 0; k < Kd; ++k) { w[k] = *(const bf16x8 *)(base + off); off += 1024 * G; }
      bias = *(const floatx4 *)&b[tile * 16 + 4 * grp];
    };
    // a workgroup's tile, K shared out among the waves (output projection, FFN2)
    auto load_part = [&](auto np, const bf16_t *W, int G, int Kt, const float *b, int tile) __attribute__((always_inline)) {
      constexpr int NP = decltype(np)::value;
      const char *base = tile_base(W, G, Kt, tile, wave);
      const uint32_t off = 16 * lane;
#pragma unroll
      for (int i = 0; i < NP; ++i)
        if (wave + TEAM_WAVES * i < Kt) w[i] = *(const bf16x8 *)(base + (off + 1024 * TEAM_WAVES * i * G));
      if (wave == 0) bias = *(const floatx4 *)&b[tile * 16 + 4 * grp];
    };
    int tile0 = wave * T + rank;  // spread over the workgroups first

    // x += y (not at the start); act = LayerNorm(x).  Wave w: rows w and w + 8.
    floatx4 gv[NC], bv[NC];
    auto load_ln = [&](const float *g, const float *b) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < NC; ++i) {
        const int c = lane + 64 * i;
        if (c < d4) { gv[i] = ((const floatx4 *)g)[c]; bv[i] = ((const floatx4 *)b)[c]; }
      }
    };
    auto row_ln = [&](floatx4(&v)[NC], floatx4(&y)[NC]) __attribute__((always_inline)) {  // LayerNorm of the row in v
      float sum = 0.f;
#pragma unroll
      for (int i = 0; i < NC; ++i)
        if (lane + 64 * i < d4) sum += (v[i][0] + v[i][1]) + (v[i][2] + v[i][3]);
      const float mean = wave_sum_f(sum) / d;
      float q = 0.f;
#pragma unroll
      for (int i = 0; i < NC; ++i)
        if (lane + 64 * i < d4) {
          const floatx4 t = v[i] - mean;
          q += (t[0] * t[0] + t[1] * t[1]) + (t[2] * t[2] + t[3] * t[3]);
        }
      const float rstd = 1.0f / sqrtf(wave_sum_f(q) / d + 1e-5f);
#pragma unroll
      for (int i = 0; i < NC; ++i)
        if (lane + 64 * i < d4) y[i] = (v[i] - mean) * rstd * gv[i] + bv[i];
    };
    auto make_act = [&](bool add) __attribute__((always_inline)) {
      floatx4 v[2][NC], y[2][NC];
#pragma unroll
      for (int jj = 0; jj < 2; ++jj)
#pragma unroll
        for (int i = 0; i < NC; ++i) {
          const int j = wave + 8 * jj, c = lane + 64 * i;
          if (add && j < R && c < d4) y[jj][i] = __builtin_bit_cast(floatx4, load_shared16(wk_y(), (j * d + 4 * c) * 4));
        }
#pragma unroll
      for (int jj = 0; jj < 2; ++jj) {
        const int j = wave + 8 * jj;
        if (j >= R) continue;
#pragma unroll
        for (int i = 0; i < NC; ++i) {
          const int c = lane + 64 * i;
          if (c < d4) {
            v[jj][i] = *(floatx4 *)&s.x[j][4 * c];
            if (add) {
              v[jj][i] += y[jj][i];
              *(floatx4 *)&s.x[j][4 * c] = v[jj][i];
            }
          }
        }
        row_ln(v[jj], y[jj]);
#pragma unroll
        for (int i = 0; i < NC; ++i) {
          const int c = lane + 64 * i;
          if (c < d4)
            *(uint2 *)&s.act[j][4 * c] = make_uint2(pack2(y[jj][i][0], y[jj][i][1]), pack2(y[jj][i][2], y[jj][i][3]));
        }
      }
    };
    auto mul_tile = [&]() __attribute__((always_inline)) {  // w x act: rows 4 grp .. + 3 of the tile, batch row col
      floatx4 acc[2] = {bias, floatx4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
      for (int k = 0; k < Kd; ++k) {
          const bf16x8 x = *(const bf16x8 *)&s.act[col][32 * k + 8 * grp];  // rows past R: columns that nobody reads
          acc[k & 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[k], x, acc[k & 1], 0, 0, 0);
          if ((k & 3) == 3) __builtin_amdgcn_sched_barrier(0);  // four LDS reads in flight: registers
        }
      return acc[0] + acc[1];
    };
    // the splits of all pairs -> s.act, a float4 chunk per thread (at most TEAM_PARTS / 2 pairs of 128)
    auto merge_splits = [&](int splits, int pairs) __attribute__((always_inline)) {
      const int at = 4 * (int)threadIdx.x, j = at / d, c = at - j * d, p = j * H + c / DH, e = c % DH;
      if (j < R) {
        floatx4 num[TEAM_SPLITS], ml[TEAM_SPLITS];
#pragma unroll
        for (int k = 0; k < TEAM_SPLITS; ++k) {
          const int part = ((k < splits ? k : 0) * pairs + p) * (DH + 4);
          num[k] = __builtin_bit_cast(floatx4, load_shared16(wk_part(), (part + e) * 4));
          ml[k] = __builtin_bit_cast(floatx4, load_shared16(wk_part(), (part + DH) * 4));
        }
        float M = ml[0][0], den = 0.f;
#pragma unroll
        for (int k = 1; k < TEAM_SPLITS; ++k) M = fmaxf(M, ml[k][0]);
        floatx4 v = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < TEAM_SPLITS; ++k) {
          const float g = k < splits ? __expf(ml[k][0] - M) : 0.f;
          v += num[k] * g;
          den += ml[k][1] * g;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = den > 0.f ? v[k] / den : 0.f;
        *(uint2 *)&s.act[j][c] = make_uint2(pack2(v[0], v[1]), pack2(v[2], v[3]));
      }
      bar();
    };
    int set = 0;
    // the d / 16 tiles of in (activation tiles of Kt k-steps) x W + b -> y; the first tile's weights are in w
    auto project = [&](auto np, const bf16_t *W, int G, int Kt, const float *b, const bf16_t *in, bool from_lds) __attribute__((always_inline)) {
      constexpr int NP = decltype(np)::value;
      anew(rank), anew(T);
      for (int tile = rank; tile - rank < wg_tiles; tile += T) {
        if (tile < wg_tiles) {
          bf16x8 x[NP];
#pragma unroll
          for (int i = 0; i < NP; ++i)
            if (!from_lds && wave + TEAM_WAVES * i < Kt) x[i] = load_shared16(in, (wave + TEAM_WAVES * i) * 1024 + act_lane(lane) * 16);
          if (from_lds)
#pragma unroll
            for (int i = 0; i < NP; ++i)
              if (wave + TEAM_WAVES * i < Kt) x[i] = *(const bf16x8 *)&s.act[col][32 * (wave + TEAM_WAVES * i) % TEAM_MAX_D + 8 * grp];
          if (tile != rank) load_part(np, W, G, Kt, b, tile);
          floatx4 acc = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int i = 0; i < NP; ++i)
            if (wave + TEAM_WAVES * i < Kt) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[i], x[i], acc, 0, 0, 0);
          s.red[set][wave][lane] = acc;
        }
        bar();
        if (wave == 0 && tile < wg_tiles) {
          floatx4 v = bias;
#pragma unroll
          for (int k = 0; k < TEAM_WAVES; ++k) v += s.red[set][k][lane];
          if (col < R) *(floatx4 *)&wk_y()[(long)col * d + tile * 16 + 4 * grp] = v;
        }
        set ^= 1;  // (two iterations on, a barrier lies between these reads and the next writes)
      }
    };

    // attention: W waves share a (row, head) pair
    int pairs = R * H;
    int wpp = TEAM_WAVES;
    while (wpp > 1 && (pairs * wpp > T * TEAM_WAVES || wpp / 2 * 32 >= ap->longest)) wpp >>= 1;
    // long rows of few pairs: workgroups that would have no pair take a share of the keys of one (att_iters is 1 then)
    int splits = 1;
    if (wpp == TEAM_WAVES)
      while (2 * splits * pairs <= T && splits < TEAM_SPLITS && 32 * TEAM_WAVES * splits < ap->longest) splits *= 2;
    int stride = wpp * splits;  // blocks between two of a wave
    int sub = wave / wpp, ws0 = wave % wpp;
    const int teams = TEAM_WAVES / wpp, att_iters = (pairs + T * teams - 1) / (T * teams);
    int split = splits > 1 ? rank / pairs : 0, pair0 = splits > 1 ? (split < splits ? rank - split * pairs : pairs) : sub * T + rank;
    int ws = ws0 + wpp * split;  // the wave's first block
    const int bpp = ap->kv.page_tokens >> 5;
    const KvGeom kvg{ap->kv.page_tokens, ap->kv.max_pages, H, DH, ap->kv.page_elems};
    int first_page = -1;  // of the wave's first block, looked up before it is needed; -1: it has none
    auto page_of = [&](const int32_t *bt, int p, int blk) __attribute__((always_inline)) {
      return bt[(long)__builtin_amdgcn_readfirstlane(s.row[p / H]) * ap->kv.max_pages + blk / bpp];
    };
    auto load_block = [&](int page, int p, int blk) __attribute__((always_inline)) {
      const bf16x8 *kp = (const bf16x8 *)(ap->pool + (long)page * ap->kv.page_elems + (long)(p % H) * (ap->kv.page_tokens * DH * 2) +
                                          (long)(blk % bpp) * (64 * DH)) + lane;
#pragma unroll
      for (int i = 0; i < 2 * QC + VM; ++i) kv[i] = kp[i * 64];
    };
    auto find_first = [&](const int32_t *bt, int p) __attribute__((always_inline)) {
      first_page = -1;
      if (p < pairs && 32 * ws < ap->t - __builtin_amdgcn_readfirstlane(s.start[p / H])) first_page = page_of(bt, p, ws);
    };
    auto first_block = [&](int p) __attribute__((always_inline)) {
      forget_kv();
      if (first_page >= 0) load_block(first_page, p, ws);
    };
    const float scale = 1.0f / sqrtf((float)DH);
    auto attend = [&](const int32_t *bt) __attribute__((always_inline)) {
      anew(ws), anew(ws0), anew(sub), anew(wpp), anew(stride), anew(pair0), anew(split), anew(pairs);
      for (int it = 0; it < att_iters; ++it) {
        const int p = pair0 + it * teams * T;
        const bool live = p < pairs;
        const int j = live ? p / H : 0, h = live ? p - j * H : 0;
        const int len = ap->t - __builtin_amdgcn_readfirstlane(s.start[j]);  // cached keys (negative: column t is still padding for this row)
        const int nblk = (len + 31) >> 5;
        const int te = ws0 * 64 + lane;     // this thread's element of the new position (and te + 64 for a wave alone on 128)
        constexpr int EPT = DH / 64;
        bf16_t q_bits[EPT], k_bits[EPT], v_bits[EPT];
        const bool with_new = live && len >= 0 && split == 0;
        int page_t = 0;
        if (live) {
          bf16x8 qf[QC];
#pragma unroll
          for (int c = 0; c < QC; ++c) qf[c] = load_shared16(wk_q(), (j * d + h * DH + 32 * c + 8 * grp) * 2);
#pragma unroll
          for (int i = 0; i < EPT; ++i) {
            const int e = te + i * wpp * 64;
            q_bits[i] = k_bits[i] = v_bits[i] = 0;
            if (with_new && e < DH) {
              const bf16_t *kr = wk_kv() + (long)j * 2 * d + h * DH + e;
              k_bits[i] = __hip_atomic_load(kr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
              v_bits[i] = __hip_atomic_load(kr + d, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
              q_bits[i] = __hip_atomic_load(wk_q() + (long)j * d + h * DH + e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
          }
          if (with_new) page_t = bt[(long)__builtin_amdgcn_readfirstlane(s.row[j]) * ap->kv.max_pages + len / ap->kv.page_tokens];
          floatx4 O[VM];
#pragma unroll
          for (int m = 0; m < VM; ++m) O[m] = floatx4{0.f, 0.f, 0.f, 0.f};
          float m_run = -1.0e30f, l_run = 0.f;
          auto use_block = [&](int blk) __attribute__((always_inline)) {
            floatx4 S[2];
#pragma unroll
            for (int tl = 0; tl < 2; ++tl) {
              S[tl] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
              for (int c = 0; c < QC; ++c) S[tl] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kv[tl * QC + c], qf[c], S[tl], 0, 0, 0);
            }
            float sv[8], bm = -1.0e30f;
            bool ok[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
              ok[i] = blk * 32 + 16 * (i >> 2) + 4 * grp + (i & 3) < len;
              sv[i] = S[i >> 2][i & 3] * scale;
              if (ok[i]) bm = fmaxf(bm, sv[i]);
            }
            bm = fmaxf(bm, __shfl_xor(bm, 16));
            bm = fmaxf(bm, __shfl_xor(bm, 32));
            const float m_new = fmaxf(m_run, bm), alpha = __expf(m_run - m_new);
            float ps = 0.f;
            uint32_t pk[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              pk[i] = pack2(ok[2 * i] ? __expf(sv[2 * i] - m_new) : 0.f, ok[2 * i + 1] ? __expf(sv[2 * i + 1] - m_new) : 0.f);
              ps += bf2f(pk[i] & 0xffffu) + bf2f(pk[i] >> 16);  // the denominator uses the rounded weights
            }
            l_run = l_run * alpha + ps;
            m_run = m_new;
            const bf16x8 pv = __builtin_bit_cast(bf16x8, (uint32x4{pk[0], pk[1], pk[2], pk[3]}));
#pragma unroll
            for (int m = 0; m < VM; ++m) {
              O[m] *= alpha;
              O[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kv[2 * QC + m], pv, O[m], 0, 0, 0);
            }
          };
          if (ws < nblk) {
            if (it) load_block(page_of(bt, p, ws), p, ws);
            use_block(ws);
          }
          for (int blk = ws + stride; blk < nblk; blk += stride) {
            load_block(page_of(bt, p, blk), p, blk);
            use_block(blk);
          }
          __builtin_amdgcn_sched_barrier(0);
          l_run += __shfl_xor(l_run, 16);
          l_run += __shfl_xor(l_run, 32);
          float dot = 0.f;
#pragma unroll
          for (int i = 0; i < EPT; ++i) dot += bf2f(q_bits[i]) * bf2f(k_bits[i]);
          dot = wave_sum_f(dot);
          if (lane == 0) { s.m[wave] = m_run; s.l[wave] = l_run; s.dot[wave] = dot; }
          if (col == 0) {
#pragma unroll
            for (int m = 0; m < VM; ++m)
#pragma unroll
              for (int i = 0; i < 4; ++i) s.o[wave][16 * m + 4 * grp + i] = O[m][i];
          }
        }
        if (wpp > 1) bar();
        else __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        if (live) {
          const int w0 = sub * wpp;
          float pm[TEAM_WAVES], pl[TEAM_WAVES], M = -1.0e30f, s_t = 0.f;  // all partial results requested together
#pragma unroll
          for (int k = 0; k < TEAM_WAVES; ++k) {
            const int at = w0 + (k < wpp ? k : 0);
            pm[k] = s.m[at];
            pl[k] = s.l[at];
          }
#pragma unroll
          for (int k = 0; k < TEAM_WAVES; ++k) M = fmaxf(M, pm[k]);
          if (with_new) {
            for (int k = 0; k < wpp && k < EPT; ++k) s_t += s.dot[w0 + k];
            s_t *= scale;
            M = fmaxf(M, s_t);
          }
#pragma unroll
          for (int k = 0; k < TEAM_WAVES; ++k) pm[k] = k < wpp ? __expf(pm[k] - M) : 0.f;
#pragma unroll
          for (int i = 0; i < EPT; ++i) {
            const int e = te + i * wpp * 64;
            if (e >= DH) continue;
            float num = 0.f, den = 0.f;
#pragma unroll
            for (int k = 0; k < TEAM_WAVES; ++k) {
              num += pm[k] * s.o[w0 + (k < wpp ? k : 0)][e];
              den += pm[k] * pl[k];
            }
            if (with_new) {
              const float g = __expf(s_t - M);
              num += g * bf2f(v_bits[i]);
              den += g;
            }
            if (splits == 1) {
              wk_o()[d_act_index(j, h * DH + e, d)] = (bf16_t)f2bf(den > 0.f ? num / den : 0.f);
            } else {
              float *part = wk_part() + (long)(split * pairs + p) * (DH + 4);
              part[e] = num;
              if (e < 2) part[DH + e] = e ? den : M;
            }
            if (with_new) {
              bf16_t *pg = ap->pool + (long)page_t * ap->kv.page_elems;
              const int tt = len % ap->kv.page_tokens;
              pg[kv_k_off(h, tt, e, kvg)] = k_bits[i];
              pg[kv_v_off(h, tt, e, kvg)] = v_bits[i];
            }
          }
        }
        if (wpp > 1 && it + 1 < att_iters) bar();  // the partial results have been read
      }
    };
    auto layer_of = [&](int i) __attribute__((always_inline)) -> LayerPtr { return (LayerPtr)ap->layers + (i < ap->warmup ? i : ap->L - ap->n + i); };

    // ---- embeddings of the group's rows
    bar();  // s.row, s.start, s.tok
    {
      LayerPtr L0 = layer_of(0);
      uint2 tv[2][NC], pv[2][NC];
#pragma unroll
      for (int jj = 0; jj < 2; ++jj) {
        const int j = wave + 8 * jj;
        if (j >= R) continue;
        int pos = ap->t - __builtin_amdgcn_readfirstlane(s.start[j]);
        if (pos < 0) pos = 0;
        const uint2 *te = (const uint2 *)(ap->tok_emb + (long)__builtin_amdgcn_readfirstlane(s.tok[j]) * d), *pe = (const uint2 *)(ap->pos_emb + (long)pos * d);
#pragma unroll
        for (int i = 0; i < NC; ++i) {
          const int c = lane + 64 * i;
          if (c < d4) { tv[jj][i] = te[c]; pv[jj][i] = pe[c]; }
        }
      }
      load_ln(L0->ln1_g, L0->ln1_b);
      forget_w();
          if (tile0 < 3 * wg_tiles) load_tile(L0->wqkv, ap->G_qkv, L0->bqkv, tile0);
#pragma unroll
      for (int jj = 0; jj < 2; ++jj) {
        const int j = wave + 8 * jj;
        if (j >= R) continue;
#pragma unroll
        for (int i = 0; i < NC; ++i) {
          const int c = lane + 64 * i;
          if (c < d4)
            *(floatx4 *)&s.x[j][4 * c] = floatx4{bf2f(tv[jj][i].x & 0xffffu) + bf2f(pv[jj][i].x & 0xffffu), bf2f(tv[jj][i].x >> 16) + bf2f(pv[jj][i].x >> 16),
                                                 bf2f(tv[jj][i].y & 0xffffu) + bf2f(pv[jj][i].y & 0xffffu), bf2f(tv[jj][i].y >> 16) + bf2f(pv[jj][i].y >> 16)};
        }
      }
      make_act(false);
    }
    for (int i = 0; i < ap->n; ++i) {
      LayerPtr L = layer_of(i);
      // ---- q | k | v
      phase();
      anew(R), anew(group);
      anew(tile0);
      find_first(L->bt, pair0);
      bar();  // act
      {
        for (int tile = tile0; tile < 3 * wg_tiles; tile += TEAM_WAVES * T) {
          if (tile != tile0) load_tile(L->wqkv, ap->G_qkv, L->bqkv, tile);
          const floatx4 v = mul_tile();
          const int n0 = tile * 16 + 4 * grp, which = n0 / d, within = n0 - which * d;
          const uint2 pk = make_uint2(pack2(v[0], v[1]), pack2(v[2], v[3]));
          if (col < R) {
            if (which == 0) *(uint2 *)&wk_q()[(long)col * d + within] = pk;
            else *(uint2 *)&wk_kv()[((long)col * 2 + which - 1) * d + within] = pk;
          }
        }
      }
      team_bar([&]() __attribute__((always_inline)) { forget_w(); first_block(pair0); });
      // ---- attention
      phase();
      anew(R), anew(group);
      attend(L->bt);
      team_bar([&]() __attribute__((always_inline)) {
        forget_w();
        if (rank < wg_tiles) load_part(Parts<(Kd + TEAM_WAVES - 1) / TEAM_WAVES>{}, L->wo, ap->G_out, Kd, L->bo, rank);
      });
      // ---- output projection
      phase();
      anew(R), anew(group);
      if (splits > 1) merge_splits(splits, pairs);
      project(Parts<(Kd + TEAM_WAVES - 1) / TEAM_WAVES>{}, L->wo, ap->G_out, Kd, L->bo, wk_o(), splits > 1);
      team_bar([&]() __attribute__((always_inline)) {
        load_ln(L->ln2_g, L->ln2_b);
        forget_w();
        if (tile0 < Kf * 2) load_tile(L->w1, ap->G_ffn1, L->b1, tile0);
      });
      // ---- FFN1
      phase();
      anew(R), anew(group);
      anew(tile0);
      make_act(true);
      bar();
      {
        for (int tile = tile0; tile < Kf * 2; tile += TEAM_WAVES * T) {
          if (tile != tile0) load_tile(L->w1, ap->G_ffn1, L->b1, tile);
          floatx4 v = mul_tile();
          for (int k = 0; k < 4; ++k) v[k] = fmaxf(v[k], 0.f);
          if (col < R) *(uint2 *)&wk_u()[d_act_index(col, tile * 16 + 4 * grp, f)] = make_uint2(pack2(v[0], v[1]), pack2(v[2], v[3]));
        }
      }
      team_bar([&]() __attribute__((always_inline)) {
        forget_w();
        if (rank < wg_tiles) load_part(Parts<(TEAM_MAX_F / 32 + TEAM_WAVES - 1) / TEAM_WAVES>{}, L->w2, ap->G_ffn2, Kf, L->b2, rank);
      });
      // ---- FFN2
      phase();
      anew(R), anew(group);
      project(Parts<(TEAM_MAX_F / 32 + TEAM_WAVES - 1) / TEAM_WAVES>{}, L->w2, ap->G_ffn2, Kf, L->b2, wk_u(), false);
      if (i + 1 == ap->n && rank == 0 && threadIdx.x == 64 * (TEAM_WAVES - 1))  // another group that no team has taken
        ctl_store(&slot->next, ctl_add(&ap->ctl->next_group, 1u));
      team_bar([&]() __attribute__((always_inline)) {
        if (i + 1 < ap->n) {
          LayerPtr N = layer_of(i + 1);
          load_ln(N->ln1_g, N->ln1_b);
          forget_w();
          if (tile0 < 3 * wg_tiles) load_tile(N->wqkv, ap->G_qkv, N->bqkv, tile0);
        } else {
          load_ln(ap->lnf_g, ap->lnf_b);
        }
      });
      if (i + 1 < ap->n) make_act(true);
    }
    // ---- final LayerNorm: a row per wave of the team
    if (threadIdx.x == 0) s.group = (int)ctl_load(&slot->next);
    {
      for (int j = tile0; j < R; j += TEAM_WAVES * T) {
        floatx4 v[NC], y[NC];
        const long b = __builtin_amdgcn_readfirstlane(s.row[j]);
#pragma unroll
        for (int i = 0; i < NC; ++i) {
          const int c = lane + 64 * i;
          if (c < d4) {
            v[i] = *(floatx4 *)&s.x[j][4 * c] + __builtin_bit_cast(floatx4, load_shared16(wk_y(), (j * d + 4 * c) * 4));
            ((floatx4 *)ap->x_out)[b * d4 + c] = v[i];
          }
        }
        row_ln(v, y);
#pragma unroll
        for (int i = 0; i < NC; ++i) {
          const int c = lane + 64 * i;
          if (c < d4) *(uint2 *)&ap->a_out[d_act_index(b, 4 * c, d)] = make_uint2(pack2(y[i][0], y[i][1]), pack2(y[i][2], y[i][3]));
        }
      }
    }
    __syncthreads();
    group = __builtin_amdgcn_readfirstlane(s.group);
    __syncthreads();
  }
  // ---- the last workgroup to leave clears the control words for the next launch
  if (threadIdx.x == 0 && ctl_add(&ap->ctl->left, 1u) == gridDim.x - 1) {
    for (int i = 0; i < TEAM_SLOTS; ++i) {
      TeamSlot *t = &ap->ctl->slot[i];
      ctl_store(&t->registered, 0);
      ctl_store(&t->team, 0);
      ctl_store(&t->arrived, 0);
      ctl_store(&t->next, 0);
    }
    ctl_store(&ap->ctl->next_group, 0);
    ctl_store(&ap->ctl->left, 0);
  }
}

// Every XCD reads all the weights: at the widest model taken here 6 to 8 MiB a layer at about 1.0 TB/s for each of eight
// XCDs, 6 to 8 us, and the rest of a layer takes 9 to 12.  us per step of 4 layers, separate kernels -> this: (256, ffn 1024)
// 1 row at 16 keys 69 -> 52, 16 rows at 200 keys 90 -> 57, at 2000 keys 116 -> 75, 128 rows at 200 keys 125 -> 80;
// (384, 1024) 77 -> 61, 96 -> 67, 140 -> 90, 147 -> 96; (512, 1536) 82 -> 68, 102 -> 80, 145 -> 112, 159 -> 115.
bool bf16_team_ok(int d, int f, int B) {
  return d <= TEAM_MAX_D && f <= TEAM_MAX_F && d % 64 == 0 && f % 32 == 0 && B >= 1 && B <= 128;
}
// As many as the output projection and FFN2 have tiles (at most TEAM_PARTS): a larger team only makes the barriers longer
// (256 wide, 16 rows at 16 keys: 53, 59, 65 us per step of 4 layers with 16, 24, 32), a smaller one has two rounds.
int bf16_team_members(int cus, int d) { return cus < d / 16 ? (cus > 1 ? cus : 1) : d / 16; }
int bf16_team_groups(int B) { return B < 8 ? B : 8; }
size_t bf16_team_rows() { return 8 * TEAM_ROWS; }
size_t bf16_team_part() { return 8 * TEAM_PARTS * (128 + 4); }

bool bf16_team_column(hipStream_t s, const TeamArgs &a) {
  static_assert(sizeof(TeamLds) <= 96 * 1024, "LDS of a workgroup");
  if (!bf16_team_ok(a.d, a.f, a.B) || a.n < 1 || a.workgroups < 1 || a.members < 1 || a.members > TEAM_PARTS) return false;
  const dim3 grid(a.workgroups), blk(TEAM_THREADS);
#define SKD_TEAM(DH, KD)                                                                                \
  {                                                                                                     \
    static std::atomic<uint64_t> done{0};                                                               \
    if (!allow_lds(done, {(const void *)k_team_column<DH, KD>}, sizeof(TeamLds))) return false;         \
    SKD_LAUNCH((k_team_column<DH, KD>), grid, blk, sizeof(TeamLds), s, a);                              \
    break;                                                                                              \
  }
  if (a.kv.dh == 64) switch (a.d / 64) {
    case 1: SKD_TEAM(64, 2) case 2: SKD_TEAM(64, 4) case 3: SKD_TEAM(64, 6) case 4: SKD_TEAM(64, 8)
    case 5: SKD_TEAM(64, 10) case 6: SKD_TEAM(64, 12) case 7: SKD_TEAM(64, 14) case 8: SKD_TEAM(64, 16)
  } else switch (a.d / 128) {
    case 1: SKD_TEAM(128, 4) case 2: SKD_TEAM(128, 8) case 3: SKD_TEAM(128, 12) case 4: SKD_TEAM(128, 16)
  }
#undef SKD_TEAM
  return true;
}

}  // namespace skd
