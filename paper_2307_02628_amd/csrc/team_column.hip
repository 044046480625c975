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
// arrival at the barrier before it and its end.
//
// A column gives the same bits as the separate kernels, whatever the size of the teams that form: every sum is taken in the
// order in which those take it (NV, TeamStep, attn_waves and attn_splits below), and a team only shares out the work.  So a
// state may change between the two, and nothing depends on what else is on the GPU.  For the order of the attention's sums a
// wave carries up to four softmax states; at 2000 keys that is 5 to 12 % of a step.
// Tried: workgroups beside the team that pull the coming weights into the L2 (slower by 3 to 10 %), a ninth wave that only
// polls (registers), K and V two barriers ahead (the loads behind them wait for them: slower).
// Ordering: a wave's stores have been acknowledged by the L2 (vmcnt 0) before its workgroup arrives; what other members
// have written is read with agent-scope loads, which do not look into the L1.
#include <algorithm>

#include "bf16_device.h"

namespace skd {

constexpr int TEAM_WAVES = 8;
constexpr int TEAM_THREADS = 64 * TEAM_WAVES;
constexpr int TEAM_ROWS = 16;    // rows of a group: one batch tile
constexpr int TEAM_MAX_D = 512;  // 16 k-steps: the weight tile of a wave, and the K and V of a 32-key block, fit 16 fragments
constexpr int TEAM_MAX_F = 2048; // 8 waves x 8 k-steps
constexpr int TEAM_SPLITS = 8, TEAM_PARTS = 128;  // shares of one pair's keys, of all pairs of a group
constexpr int TEAM_SUMS = 32;    // partial sums of a tile along K, and softmax states of the pairs that a workgroup has at a time
// k-steps of a wave; with more than 64 rows, an odd number of k-steps above 32 (FFN2 without a split, by four waves) takes more
// and keeps the separate kernels
constexpr int TEAM_OUT_STEPS = 2, TEAM_OUT_STEPS_WIDE = 4, TEAM_FFN2_STEPS = 8;
// an entry of TeamStep: k-step in bits 0 .. 5, whether there is one, whether the sum ends here, which sum (and not zero)
constexpr uint32_t TEAM_STEP_K = 1 << 6, TEAM_STEP_LAST = 1 << 7, TEAM_STEP_USED = 1 << 8;
constexpr int TEAM_STEP_SUM = 9;
constexpr int TEAM_REG_POLLS = 400;       // about 100 us: how long a leader waits for workgroups that have not started
constexpr int TEAM_MAX_POLLS = 1 << 22;   // over a second; members run until they arrive, so a wait that long is an error (GaveUp)

// 16 bytes that another CU of this XCD may have written in this launch: a buffer load with sc1 (agent scope), which the L1
// does not answer.  (As two 8-byte atomic loads: 1.8 instead of 1.3 us for FFN2's phase at d = 256, f = 1024.)
__device__ inline bf16x8 load_shared16(const void *p, int byte_offset) {
  const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void *)p, 0, 0x7fffffff, 0x00027000);
  return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(r, byte_offset, 0, 16));
}
__device__ inline floatx2 load_shared8(const void *p, int byte_offset) {
  const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void *)p, 0, 0x7fffffff, 0x00027000);
  return __builtin_bit_cast(floatx2, __builtin_amdgcn_raw_buffer_load_b64(r, byte_offset, 0, 16));
}
__device__ inline uint32_t ctl_load(const uint32_t *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ inline void ctl_store(uint32_t *p, uint32_t v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ inline void give_up(uint32_t *word) { __hip_atomic_store(word, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM); }
__device__ inline uint32_t ctl_add(uint32_t *p, uint32_t v) { return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

typedef const TeamArgs __attribute__((address_space(4))) *ArgsPtr;
typedef const TeamLayer __attribute__((address_space(4))) *LayerPtr;

typedef const uint32_t __attribute__((address_space(4))) *WordPtr;

__device__ inline float row_sum(float v) {  // over 16 lanes, the pairs of a butterfly of 8, 4, 2, 1
#define SKD_ROR(n) v += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x120 + n, 0xF, 0xF, true))
  SKD_ROR(8);
  SKD_ROR(4);
  SKD_ROR(2);
  SKD_ROR(1);
#undef SKD_ROR
  return v;
}

template <int N>
struct Parts { static constexpr int value = N; };

// A wave's k-steps of a tile (TeamSteps), at most N of them: f(place, step).
template <int N, int I = 0, typename F>
__device__ __forceinline__ void walk_steps(const uint32x4 &steps, F f) {
  if constexpr (I < N) {
    const uint32_t e = (steps[I >> 1] >> (16 * (I & 1))) & 0xffffu;
    if (e) {
      f(I, e);
      walk_steps<N, I + 1>(steps, f);
    }
  }
}

struct TeamLds {
  float x[TEAM_ROWS][TEAM_MAX_D];             // residual rows
  bf16_t act[TEAM_ROWS][TEAM_MAX_D + 32];     // their LayerNorm (rows 16 banks apart)
  union {
    floatx4 red[TEAM_SUMS][64];               // of a tile along K
    float o[TEAM_SUMS][128];                  // numerators of the softmax states
  };
  float m[TEAM_SUMS], l[TEAM_SUMS], dot[2 * TEAM_WAVES];
  int row[TEAM_ROWS], start[TEAM_ROWS], tok[TEAM_ROWS];
  int all_tok[128], all_start[128], all_order[128];
  int rank, size, group;
};

// NV: waves of the separate kernels' projections (8, or 4 from 65 rows on), see the sums below
template <int DH, int KD, int NV>
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
      if (!t) give_up(ap->gave_up);
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
  int patience = TEAM_MAX_POLLS;  // of the wave that polls; none left once it had to go on without the others
  // of the team; what the waves do meanwhile: requests for the next phase
  auto team_bar = [&](auto meanwhile) __attribute__((always_inline)) {
    wait_vmcnt<0>();  // stores
    bar();
    arrived += (uint32_t)T;
    const bool polls = wave == TEAM_WAVES - 1;  // the wave with the least to request
    if (polls && lane == 0) (void)ctl_add(&slot->arrived, 1u);
    meanwhile();
    if (polls)
      for (int i = 0; __builtin_amdgcn_readfirstlane((int)(ctl_load(&slot->arrived) - arrived)) < 0; ++i)
        if (i >= patience) {
          give_up(ap->gave_up);
          patience = 0;
          break;
        }
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
    typedef Parts<NV == 8 ? TEAM_OUT_STEPS : TEAM_OUT_STEPS_WIDE> OutSteps;
    bf16x8 w[NW];  // the phase's first weight tile of this wave, or its first K and V block, requested ahead of the barrier
    bf16x8 kv[2 * QC + VM];  // K and V of 32 keys: fragments 0 .. 2 QC - 1, and those behind them
    floatx4 bias;
    // fragment (tile, k) of a layout in groups of one tile is base + 1024 k bytes + 16 lane: a scalar base and a 32-bit offset
    auto tile_base = [&](const bf16_t *W, int Kt, int tile) __attribute__((always_inline)) { return (const char *)W + (long)tile * Kt * 1024; };
    // what a conditional load leaves as it was is not wanted any more: without this it would stay in registers
    auto forget_w = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int k = 0; k < NW; ++k) asm volatile("" : "=v"(w[k]));
    };
    auto forget_kv = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int k = 0; k < 2 * QC + VM; ++k) asm volatile("" : "=v"(kv[k]));
    };
    // Sums along K are taken as the separate kernels take them: one per wave of theirs (NV of them, which have the k-steps
    // in turn, one or two at a time), added in wave order, then the sums of their K parts in order, then the bias.  With 96
    // and 128 padded rows a wave begins at a step that depends on the tile and the part (rotated).
    constexpr bool ROT = NV == 4;
    constexpr int CH = KD % 4 == 0 ? KD / 4 : 1;  // steps of a wave where they may be rotated
    int rot = 0;  // of the tile in w
    auto k_of = [&](int j) __attribute__((always_inline)) {  // k-step of w[j] in load_tile
      if constexpr (!ROT || KD % 4) return j;
      const int c = (j >> 2) + rot;
      return 4 * (c >= CH ? c - CH : c) + (j & 3);
    };
    // a wave's own tile over all of K (q | k | v, FFN1)
    auto load_tile = [&](const bf16_t *W, int rotate, const float *b, int tile) __attribute__((always_inline)) {
      const char *base = tile_base(W, Kd, tile);
      if constexpr (ROT) rot = rotate ? (tile >> 3) * 5 % CH : 0;
#pragma unroll
      for (int j = 0; j < Kd; ++j) w[j] = *(const bf16x8 *)(base + (uint32_t)(16 * lane + 1024 * k_of(j)));
      bias = *(const floatx4 *)&b[tile * 16 + 4 * grp];
    };
    // a workgroup's tile, K shared out among the waves (output projection, FFN2)
    uint32x4 steps;  // of the tile in w
    auto load_part = [&](auto np, const bf16_t *W, const TeamStep *table, int Kt, const float *b, int tile) __attribute__((always_inline)) {
      const char *base = tile_base(W, Kt, tile);
      const WordPtr at = (WordPtr)table + (tile * TEAM_WAVES + wave) * (sizeof(TeamStep) / 4);
#pragma unroll
      for (int i = 0; i < 4; ++i) steps[i] = at[i];
      walk_steps<decltype(np)::value>(steps, [&](int i, uint32_t e) __attribute__((always_inline)) {
        if (e & TEAM_STEP_K) w[i] = *(const bf16x8 *)(base + (uint32_t)(16 * lane + 1024 * (e & 63)));
      });
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
      float sum = 0.f, sq = 0.f;  // 256 columns at a time, as the row kernels' waves
#pragma unroll
      for (int i = 0; i < NC; ++i) {
        float s = 0.f;
        if (lane + 64 * i < d4) s += (v[i][0] + v[i][1]) + (v[i][2] + v[i][3]);
        sum += wave_sum_f(s);
      }
      const float mean = sum / d;
#pragma unroll
      for (int i = 0; i < NC; ++i) {
        float q = 0.f;
        if (lane + 64 * i < d4) {
          const floatx4 t = v[i] - mean;
          q += (t[0] * t[0] + t[1] * t[1]) + (t[2] * t[2] + t[3] * t[3]);
        }
        sq += wave_sum_f(q);
      }
      const float rstd = 1.0f / sqrtf(sq / d + 1e-5f);
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
      constexpr int NA = KD < NV ? KD : NV;
      floatx4 acc[NA];
#pragma unroll
      for (int j = 0; j < Kd; ++j) {
        const bf16x8 x = *(const bf16x8 *)&s.act[col][32 * k_of(j) + 8 * grp];  // rows past R: columns that nobody reads
        acc[j % NV] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[j], x, j < NV ? floatx4{0.f, 0.f, 0.f, 0.f} : acc[j % NV], 0, 0, 0);
        if ((j & 3) == 3) __builtin_amdgcn_sched_barrier(0);  // four LDS reads in flight: registers
      }
      floatx4 v = acc[0];
#pragma unroll
      for (int j = 1; j < NA; ++j) v += acc[j];
      return v + bias;
    };
    // the splits of all pairs -> s.act, a float4 chunk per thread at a time
    auto merge_splits = [&](int splits, int pairs) __attribute__((always_inline)) {
      for (int at = 4 * (int)threadIdx.x; at < R * d; at += 4 * TEAM_THREADS) {
        const int j = at / d, c = at - j * d, p = j * H + c / DH, e = c % DH;
        floatx4 num[TEAM_SPLITS];
        floatx2 ml[TEAM_SPLITS];
#pragma unroll
        for (int k = 0; k < TEAM_SPLITS; ++k) {
          const int part = ((k < splits ? k : 0) * pairs + p) * (DH + 4);
          num[k] = __builtin_bit_cast(floatx4, load_shared16(wk_part(), (part + e) * 4));
          ml[k] = load_shared8(wk_part(), (part + DH) * 4);
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
    // the d / 16 tiles of in (activation tiles of Kt k-steps) x W + b -> y; the first tile's weights are in w
    auto project = [&](auto np, const bf16_t *W, const TeamStep *table, int parts, int Kt, const float *b, const bf16_t *in, bool from_lds) __attribute__((always_inline)) {
      constexpr int NP = decltype(np)::value;
      anew(rank), anew(T);
      for (int tile = rank; tile < wg_tiles; tile += T) {
        if (tile != rank) {
          load_part(np, W, table, Kt, b, tile);
          bar();  // the sums of the tile before have been read
        }
        bf16x8 x[NP];
        if (from_lds)
          walk_steps<NP>(steps, [&](int i, uint32_t e) __attribute__((always_inline)) {
            if (e & TEAM_STEP_K) x[i] = *(const bf16x8 *)&s.act[col][32 * (e & 63) % TEAM_MAX_D + 8 * grp];
          });
        else
          walk_steps<NP>(steps, [&](int i, uint32_t e) __attribute__((always_inline)) {
            if (e & TEAM_STEP_K) x[i] = load_shared16(in, (e & 63) * 1024 + act_lane(lane) * 16);
          });
        floatx4 acc = floatx4{0.f, 0.f, 0.f, 0.f};
        walk_steps<NP>(steps, [&](int i, uint32_t e) __attribute__((always_inline)) {
          if (e & TEAM_STEP_K) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[i], x[i], acc, 0, 0, 0);
          if (e & TEAM_STEP_LAST) {
            s.red[e >> TEAM_STEP_SUM][lane] = acc;
            acc = floatx4{0.f, 0.f, 0.f, 0.f};
          }
        });
        bar();
        if (wave == 0) {
          auto part_sum = [&](int part) __attribute__((always_inline)) {
            floatx4 p = s.red[part * NV][lane];
#pragma unroll
            for (int k = 1; k < NV; ++k) p += s.red[part * NV + k][lane];
            return p;
          };
          floatx4 v;
          if (parts == 2) {  // (both requested together)
            const floatx4 v0 = part_sum(0), v1 = part_sum(1);
            v = v0 + v1;
          } else {
            v = part_sum(0);
            for (int part = 1; part < parts; ++part) v += part_sum(part);
          }
          v += bias;
          if (col < R) *(floatx4 *)&wk_y()[(long)col * d + tile * 16 + 4 * grp] = v;
        }
      }
    };

    // Attention: the keys of a (row, head) pair are shared out over `splits` x `states` softmax states, every states-th
    // block of a split each, as the separate kernels share them out over workgroups and waves; they say how the sums are taken.
    // rw waves of a workgroup have the states of one (pair, split) between them: what a team of another size changes.
    auto splits_of = [&]() __attribute__((always_inline)) { return ap->attn_splits; };
    int lrw = 3;  // log2 of rw
    while (lrw > 0 && ((1 << lrw) > ap->attn_waves || (4 << lrw > ap->attn_waves &&  // (at most four states a wave: TEAM_SUMS)
                                                       ((R * H * ap->attn_splits << lrw) > T * TEAM_WAVES || 16 << lrw >= ap->longest))))
      --lrw;
    // page of a block; block / blocks per page, exact below 2^20 blocks: the quotient is half a block from the next integer
    auto page_at = [&](WordPtr pages, int blk) __attribute__((always_inline)) {
      return (int)pages[__builtin_amdgcn_readfirstlane((int)(((float)blk + 0.5f) * __builtin_amdgcn_rcpf((float)(ap->kv.page_tokens >> 5))))];
    };
    const KvGeom kvg{ap->kv.page_tokens, ap->kv.max_pages, H, DH, ap->kv.page_elems};
    int first_page = -1;  // of the wave's first block, looked up before it is needed; -1: it has none
    auto split_len = [](int splits, int nblk) __attribute__((always_inline)) { return splits > 1 ? (nblk + splits - 1) / splits : nblk; };  // blocks
    auto pages_of = [&](const int32_t *bt, int p) __attribute__((always_inline)) {
      return (WordPtr)bt + (long)__builtin_amdgcn_readfirstlane(s.row[p / H]) * ap->kv.max_pages;
    };
    auto load_block = [&](bf16x8(&kv)[2 * QC + VM], int page, int p, int blk) __attribute__((always_inline)) {
      const bf16x8 *kp = (const bf16x8 *)(ap->pool + (long)page * ap->kv.page_elems + (long)(p % H) * ap->kv.page_tokens * (DH * 2) +
                                          (long)(blk % (ap->kv.page_tokens >> 5)) * (64 * DH)) + lane;
#pragma unroll
      for (int i = 0; i < 2 * QC + VM; ++i) kv[i] = kp[i * 64];
    };
    auto first_block = [&](const int32_t *bt, bool load) __attribute__((always_inline)) {
      const int splits = splits_of(), pairs = R * H, item = (wave >> lrw) * T + rank, sp = splits > 1 ? item / pairs : 0, p = item - sp * pairs;
      const int nblk = sp < splits && p < pairs ? (ap->t - __builtin_amdgcn_readfirstlane(s.start[p / H]) + 31) >> 5 : 0;
      const int per = split_len(splits, nblk), blk = sp * per + (wave & ((1 << lrw) - 1));
      if (load) {
        forget_kv();
        if (first_page >= 0) load_block(kv, first_page, p, blk);
      } else {
        first_page = blk < min(sp * per + per, nblk) ? page_at(pages_of(bt, p), blk) : -1;
      }
    };
    const float scale = 1.0f / sqrtf((float)DH);
    auto attend = [&](const int32_t *bt) __attribute__((always_inline)) {
      anew(lrw), anew(rank), anew(T);
      const int states = ap->attn_waves, splits = splits_of(), pairs = R * H, rw = 1 << lrw, sub = wave >> lrw, ws0 = wave & (rw - 1);
      const int at_once = T * (TEAM_WAVES >> lrw), items = pairs * splits, item0 = sub * T + rank;
      for (int it = 0; it == 0 || it * at_once < items; ++it) {
        const int item = item0 + it * at_once;
        const bool live = item < items;
        const int sp = live && splits > 1 ? item / pairs : 0, p = live ? item - sp * pairs : 0;
        const int j = p / H, h = p - j * H;
        const int len = ap->t - __builtin_amdgcn_readfirstlane(s.start[j]);  // cached keys (negative: column t is still padding for this row)
        const int nblk = (len + 31) >> 5, per = split_len(splits, nblk), lo = sp * per, hi = min(lo + per, nblk);
        constexpr int EPT = DH / 64;        // this thread's elements of the new position: te + 64 rw i, below DH
        const int te = ws0 * 64 + lane;
        bf16_t q_bits[EPT], k_bits[EPT], v_bits[EPT];
        const bool with_new = live && len >= 0 && sp + 1 == splits;
        int page_t = 0;
        if (live) {
          bf16x8 qf[QC];
#pragma unroll
          for (int c = 0; c < QC; ++c) qf[c] = load_shared16(wk_q(), (j * d + h * DH + 32 * c + 8 * grp) * 2);
#pragma unroll
          for (int i = 0; i < EPT; ++i) {
            const int e = te + i * rw * 64;
            q_bits[i] = k_bits[i] = v_bits[i] = 0;
            if (with_new && e < DH) {
              const bf16_t *kr = wk_kv() + (long)j * 2 * d + h * DH + e;
              k_bits[i] = __hip_atomic_load(kr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
              v_bits[i] = __hip_atomic_load(kr + d, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
              q_bits[i] = __hip_atomic_load(wk_q() + (long)j * d + h * DH + e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
          }
          const WordPtr pages = pages_of(bt, p);
          if (with_new) page_t = (int)pages[len / ap->kv.page_tokens];
          floatx4 O[VM];
          float m_run, l_run;
          auto fresh = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int m = 0; m < VM; ++m) O[m] = floatx4{0.f, 0.f, 0.f, 0.f};
            m_run = -1.0e30f;
            l_run = 0.f;
          };
          auto leave = [&](int st) __attribute__((always_inline)) {  // the state to LDS
            const int at = sub * states + st;
            if (lane == 0) { s.m[at] = m_run; s.l[at] = l_run; }
            if (col == 0) {
#pragma unroll
              for (int m = 0; m < VM; ++m)
#pragma unroll
                for (int i = 0; i < 4; ++i) s.o[at][16 * m + 4 * grp + i] = O[m][i];
            }
          };
          auto use_block = [&](bf16x8(&kv)[2 * QC + VM], int blk) __attribute__((always_inline)) {
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
          const int filled = min(hi - lo, states);  // states with a block; the others are left as they begin
          fresh();
          for (int st = ws0; st < states; st += rw)
            if (st >= filled) leave(st);
          int st = ws0, blk = lo + ws0, st1 = st, blk1 = blk, page1 = 0;
          auto advance = [&]() __attribute__((always_inline)) {  // to the wave's next block
            blk1 += states;
            if (blk1 >= hi) {
              st1 += rw;
              blk1 = lo + st1;
            }
            if (st1 < filled) page1 = page_at(pages, blk1);
          };
          // one block, and the request for the next one (64-wide heads: ahead of it)
          auto step = [&](bf16x8(&kv)[2 * QC + VM], bf16x8(&next)[2 * QC + VM]) __attribute__((always_inline)) {
            const bool more = st1 < filled;
            const int st_next = st1, blk_next = blk1, page_next = page1;
            if constexpr (DH == 64) if (more) load_block(next, page_next, p, blk_next);
            advance();
            use_block(kv, blk);
            if (st_next != st) {
              __builtin_amdgcn_sched_barrier(0);
              l_run += __shfl_xor(l_run, 16);
              l_run += __shfl_xor(l_run, 32);
              leave(st);
              fresh();
            }
            if constexpr (DH != 64) if (more) load_block(next, page_next, p, blk_next);
            st = st_next;
            blk = blk_next;
            return more;
          };
          if (st < filled) {
            if (it) load_block(kv, page_at(pages, blk), p, blk);
            advance();
            if constexpr (DH == 64) {
              bf16x8 kv1[2 * QC + VM];
              while (step(kv, kv1) && step(kv1, kv)) {}
            } else {
              while (step(kv, kv)) {}
            }
          }
#pragma unroll
          for (int i = 0; i < EPT; ++i) {  // q . k of the new position, 64 elements at a time
            float dot = bf2f(q_bits[i]) * bf2f(k_bits[i]);
            dot += __shfl_xor(dot, 32);
            dot += __shfl_xor(dot, 16);
            dot = row_sum(dot);
            if (lane == 0 && ws0 + i * rw < EPT) s.dot[sub * 2 + ws0 + i * rw] = dot;
          }
        }
        if (rw > 1) bar();
        else __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        auto merge = [&](auto chunk) __attribute__((always_inline)) {  // states requested together
          constexpr int N = decltype(chunk)::value;
          const int w0 = sub * states;
          float pm[N], pl[N], M = -1.0e30f, s_t = 0.f;
          auto request = [&](int k0) __attribute__((always_inline)) {
#pragma unroll
            for (int k = 0; k < N; ++k) {
              const int at = w0 + (k0 + k < states ? k0 + k : 0);
              pm[k] = s.m[at];
              pl[k] = s.l[at];
            }
          };
          request(0);
          float dots[EPT];
#pragma unroll
          for (int k = 0; k < EPT; ++k) dots[k] = s.dot[sub * 2 + k];
          for (int k0 = 0;;) {
#pragma unroll
            for (int k = 0; k < N; ++k) M = fmaxf(M, pm[k]);
            if ((k0 += N) >= states) break;
            request(k0);
          }
          if (with_new) {
#pragma unroll
            for (int k = 0; k < EPT; ++k) s_t += dots[k];
            s_t *= scale;
            M = fmaxf(M, s_t);
          }
#pragma unroll
          for (int i = 0; i < EPT; ++i) {
            const int e = te + i * rw * 64;
            if (e >= DH) continue;
            float num = 0.f, den = 0.f;
            for (int k0 = 0; k0 < states; k0 += N) {
              float po[N];
              if (states > N) request(k0);
#pragma unroll
              for (int k = 0; k < N; ++k) po[k] = s.o[w0 + (k0 + k < states ? k0 + k : 0)][e];
#pragma unroll
              for (int k = 0; k < N; ++k) {
                const float g = k0 + k < states ? __expf(pm[k] - M) : 0.f;
                num += g * po[k];
                den += g * pl[k];
              }
            }
            if (with_new) {
              const float g = __expf(s_t - M);
              num += g * bf2f(v_bits[i]);
              den += g;
            }
            if (splits == 1) {
              wk_o()[d_act_index(j, h * DH + e, d)] = (bf16_t)f2bf(den > 0.f ? num / den : 0.f);
            } else {
              float *part = wk_part() + (long)item * (DH + 4);
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
        };
        if (live) {
          if (states <= 2) merge(Parts<2>{});
          else merge(Parts<DH == 64 ? 8 : 4>{});
        }
        if (rw > 1 && (it + 1) * at_once < items) bar();  // the partial results have been read
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
      if (tile0 < 3 * wg_tiles) load_tile(L0->wqkv, ap->rot_qkv, L0->bqkv, tile0);
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
      first_block(L->bt, false);
      bar();  // act
      {
        for (int tile = tile0; tile < 3 * wg_tiles; tile += TEAM_WAVES * T) {
          if (tile != tile0) load_tile(L->wqkv, ap->rot_qkv, L->bqkv, tile);
          const floatx4 v = mul_tile();
          const int n0 = tile * 16 + 4 * grp, which = n0 / d, within = n0 - which * d;
          const uint2 pk = make_uint2(pack2(v[0], v[1]), pack2(v[2], v[3]));
          if (col < R) {
            if (which == 0) *(uint2 *)&wk_q()[(long)col * d + within] = pk;
            else *(uint2 *)&wk_kv()[((long)col * 2 + which - 1) * d + within] = pk;
          }
        }
      }
      team_bar([&]() __attribute__((always_inline)) { forget_w(); first_block(L->bt, true); });
      // ---- attention
      phase();
      anew(R), anew(group);
      attend(L->bt);
      team_bar([&]() __attribute__((always_inline)) {
        forget_w();
        if (rank < wg_tiles) load_part(OutSteps{}, L->wo, ap->out_steps, Kd, L->bo, rank);
      });
      // ---- output projection
      phase();
      anew(R), anew(group);
      if (splits_of() > 1) merge_splits(splits_of(), R * H);
      project(OutSteps{}, L->wo, ap->out_steps, ap->out_parts, Kd, L->bo, wk_o(), splits_of() > 1);
      team_bar([&]() __attribute__((always_inline)) {
        load_ln(L->ln2_g, L->ln2_b);
        forget_w();
        if (tile0 < Kf * 2) load_tile(L->w1, ap->rot_ffn1, L->b1, tile0);
      });
      // ---- FFN1
      phase();
      anew(R), anew(group);
      anew(tile0);
      make_act(true);
      bar();
      {
        for (int tile = tile0; tile < Kf * 2; tile += TEAM_WAVES * T) {
          if (tile != tile0) load_tile(L->w1, ap->rot_ffn1, L->b1, tile);
          floatx4 v = mul_tile();
          for (int k = 0; k < 4; ++k) v[k] = fmaxf(v[k], 0.f);
          if (col < R) *(uint2 *)&wk_u()[d_act_index(col, tile * 16 + 4 * grp, f)] = make_uint2(pack2(v[0], v[1]), pack2(v[2], v[3]));
        }
      }
      team_bar([&]() __attribute__((always_inline)) {
        forget_w();
        if (rank < wg_tiles) load_part(Parts<TEAM_FFN2_STEPS>{}, L->w2, ap->ffn2_steps, Kf, L->b2, rank);
      });
      // ---- FFN2
      phase();
      anew(R), anew(group);
      project(Parts<TEAM_FFN2_STEPS>{}, L->w2, ap->ffn2_steps, ap->ffn2_parts, Kf, L->b2, wk_u(), false);
      if (i + 1 == ap->n && rank == 0 && threadIdx.x == 64 * (TEAM_WAVES - 1))  // another group that no team has taken
        ctl_store(&slot->next, ctl_add(&ap->ctl->next_group, 1u));
      team_bar([&]() __attribute__((always_inline)) {
        if (i + 1 < ap->n) {
          LayerPtr N = layer_of(i + 1);
          load_ln(N->ln1_g, N->ln1_b);
          forget_w();
          if (tile0 < 3 * wg_tiles) load_tile(N->wqkv, ap->rot_qkv, N->bqkv, tile0);
        } else {
          load_ln(ap->lnf_g, ap->lnf_b);
        }
      });
      if (i + 1 < ap->n) make_act(true);
    }
    // ---- final LayerNorm: a row per wave of the team
    if (threadIdx.x == 64 * (TEAM_WAVES - 1)) s.group = patience > 0 ? (int)ctl_load(&slot->next) : ap->groups;
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
// 1 row at 16 keys 90 -> 48, 16 rows at 200 keys 117 -> 57, at 2000 keys 147 -> 82, 128 rows at 200 keys 148 -> 82;
// (384, 1024) 90 -> 56, 125 -> 67, 161 -> 97, 165 -> 99; (512, 2048) 95 -> 74, 127 -> 89, 161 -> 125, 172 -> 124.
bool bf16_team_ok(int d, int f, int B) {
  return d <= TEAM_MAX_D && f <= TEAM_MAX_F && d % 64 == 0 && f % 32 == 0 && B >= 1 && B <= 128;
}
// d / 2 workgroups share out the keys, the separate kernels spread them over 256 CUs: the time they take grows with rows x
// keys here and with rows x keys x d there.  us per step of 4 layers, separate -> this, by total of cached keys:
//   (64, ffn 256)  32 rows  96 000: 150 -> 139, 128 000: 154 -> 159;  (64, 2048) 64 rows 96 000: 154 -> 155
//   (128, 512)     64 rows  96 000: 132 -> 123, 128 000: 141 -> 141, 192 000: 160 -> 200
//   (192, 768)    128 rows 128 000: 177 -> 180, 64 rows: 175 -> 172
//   (256, 1024)    96 rows 144 000: 212 -> 202, 288 000: 299 -> 310
//   (320, 1024)    96 rows 192 000: 259 -> 256;  (384, 1024) 128 rows 256 000: 353 -> 336
//   (512, 2048)    32 rows 192 000: 326 -> 320, 256 000: 401 -> 400
// Fewer rows than XCDs leave some idle: (512, 2048) one row of 4000 keys 112 -> 106, of 6000 114 -> 118, four of 8000 148 ->
// 141; (384, 1024) one of 8000 119 -> 103, (256, 1024) 96 -> 90, (64, 256) 98 -> 81; more than 8192 keys were not measured.
bool bf16_team_keys(int d, int B, long longest, long total) {
  return total <= (d >= 384 ? 256000 : 320L * (d + 176)) && (B >= 8 || longest <= (d > 384 && B <= 2 ? 4096 : 8192));
}
// As many as the output projection and FFN2 have tiles: a larger team only makes the barriers longer
// (256 wide, 16 rows at 16 keys: 53, 59, 65 us per step of 4 layers with 16, 24, 32), a smaller one has two rounds.
int bf16_team_members(int cus, int d) { return cus < d / 16 ? (cus > 1 ? cus : 1) : d / 16; }
int bf16_team_groups(int B) { return B < 8 ? B : 8; }
size_t bf16_team_rows() { return 8 * TEAM_ROWS; }
size_t bf16_team_part() { return 8 * TEAM_PARTS * (128 + 4); }
// The k-steps of every tile and wave of a projection whose separate kernel has p.waves waves, p.unit k-steps a buffer, p.split
// K parts and maybe a rotated start (table: null, or [N / 16][TEAM_WAVES]); false if they are not among what the column can
// take, at most `most` steps of a wave.
static bool team_steps(TeamStep *table, int N, int K, const TeamSums &p, int most) {
  const int Kf = K / 32;
  if ((p.waves != 8 && p.waves != 4) || p.unit < 1 || p.split < 1 || Kf % p.split || p.split * p.waves > TEAM_SUMS) return false;
  const int n = Kf / p.split;
  int unit = p.unit;
  while (unit > 1 && n % unit) unit >>= 1;  // whole buffers, as the launch takes them
  if (p.rotate && (n % 4 || p.waves != 4 || unit != 1)) return false;
  for (int tile = 0; tile < N / 16; ++tile)
    for (int wave = 0; wave < TEAM_WAVES; ++wave) {
      TeamStep list{};
      int at = 0;
      for (int part = wave / p.waves; part < p.split; part += TEAM_WAVES / p.waves) {  // (wave % p.waves) of the separate kernel
        const int turns = std::max(1, (n / unit - wave % p.waves + p.waves - 1) / p.waves), rot = p.rotate ? ((tile >> 3) * 5 + part * 3) % (n / 4) : 0;
        for (int i = 0; i < turns * unit; ++i) {
          if (at >= most) return false;
          int k = (wave % p.waves + p.waves * (i / unit)) * unit + i % unit;
          uint32_t e = TEAM_STEP_USED;
          if (k < n) e |= TEAM_STEP_K | (part * n + (k + 4 * rot) % n);
          if (i + 1 == turns * unit) e |= TEAM_STEP_LAST;
          list.e[at++] = (uint16_t)(e | (part * p.waves + wave % p.waves) << TEAM_STEP_SUM);
        }
      }
      if (table) table[tile * TEAM_WAVES + wave] = list;
    }
  return true;
}
size_t bf16_team_steps(int d) { return (size_t)(d / 16) * TEAM_WAVES; }
bool bf16_team_sums(TeamArgs &a, int B_pad, const TeamSums &qkv, const TeamSums &out, const TeamSums &ffn1, const TeamSums &ffn2,
                    TeamStep *out_steps, TeamStep *ffn2_steps) {
  a.wide = B_pad >= 96;
  for (const TeamSums *p : {&qkv, &out, &ffn1, &ffn2})
    if (p->tiles != 1 || p->waves != (a.wide ? 4 : 8)) return false;
  for (const TeamSums *p : {&qkv, &ffn1})
    if (p->unit != 1 || p->split != 1 || (p->rotate && (!a.wide || a.d % 128))) return false;
  a.rot_qkv = qkv.rotate;
  a.rot_ffn1 = ffn1.rotate;
  a.out_parts = out.split;
  a.ffn2_parts = ffn2.split;
  return team_steps(out_steps, a.d, a.d, out, a.wide ? TEAM_OUT_STEPS_WIDE : TEAM_OUT_STEPS) &&
         team_steps(ffn2_steps, a.d, a.f, ffn2, TEAM_FFN2_STEPS);
}
// Keys shared out over `states` softmax states in each of `splits` parts.
bool bf16_team_states(const TeamArgs &a, int states, int splits) {
  const int rows = (a.B + a.groups - 1) / a.groups, pairs = rows * (a.d / a.kv.dh);
  return states >= 1 && states <= 16 && !(states & (states - 1)) && splits >= 1 && splits <= TEAM_SPLITS && (splits == 1 || pairs * splits <= TEAM_PARTS);
}

bool bf16_team_column(hipStream_t s, const TeamArgs &a) {
  static_assert(sizeof(TeamLds) <= 96 * 1024, "LDS of a workgroup");
  if (!bf16_team_ok(a.d, a.f, a.B) || a.n < 1 || a.workgroups < 1 || a.members < 1 || !bf16_team_states(a, a.attn_waves, a.attn_splits)) return false;
  const dim3 grid(a.workgroups), blk(TEAM_THREADS);
#define SKD_TEAM_NV(DH, KD, NV)                                                                         \
  {                                                                                                     \
    static std::atomic<uint64_t> done{0};                                                               \
    if (!allow_lds(done, {(const void *)k_team_column<DH, KD, NV>}, sizeof(TeamLds))) return false;     \
    SKD_LAUNCH((k_team_column<DH, KD, NV>), grid, blk, sizeof(TeamLds), s, a);                          \
    break;                                                                                              \
  }
#define SKD_TEAM(DH, KD) if (a.wide) SKD_TEAM_NV(DH, KD, 4) else SKD_TEAM_NV(DH, KD, 8)
  if (a.kv.dh == 64) switch (a.d / 64) {
    case 1: SKD_TEAM(64, 2) case 2: SKD_TEAM(64, 4) case 3: SKD_TEAM(64, 6) case 4: SKD_TEAM(64, 8)
    case 5: SKD_TEAM(64, 10) case 6: SKD_TEAM(64, 12) case 7: SKD_TEAM(64, 14) case 8: SKD_TEAM(64, 16)
  } else switch (a.d / 128) {
    case 1: SKD_TEAM(128, 4) case 2: SKD_TEAM(128, 8) case 3: SKD_TEAM(128, 12) case 4: SKD_TEAM(128, 16)
  }
#undef SKD_TEAM
#undef SKD_TEAM_NV
  return true;
}

}  // namespace skd
