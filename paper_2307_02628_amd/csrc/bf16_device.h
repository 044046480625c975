// Device helpers shared by the bf16 kernels: fragment types, conversions, activation and page addressing.
#pragma once
#include <initializer_list>

#include "once_per_device.h"
#include "skd_kernels.h"

namespace skd {

// Lets the kernels use `bytes` of dynamic LDS on the current device; `done` belongs to these kernels.
inline bool allow_lds(std::atomic<uint64_t> &done, std::initializer_list<const void *> kernels, size_t bytes) {
  int device = 0;
  if (hipGetDevice(&device) != hipSuccess) return false;
  return once_per_device(done, device, [&]() {
    for (const void *k : kernels)
      if (hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) != hipSuccess) return false;
    return true;
  });
}

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float floatx4;
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t uint32x4;

// fp32 -> bf16, round to nearest even: the conversion instruction of gfx950 (v_cvt_pk_bf16_f32), which the compiler
// emits for these casts; the same rounding in integer arithmetic takes five instructions per value.
typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
typedef __attribute__((__vector_size__(2 * sizeof(float)))) float floatx2;
__device__ inline uint32_t f2bf(float f) { return (uint32_t)__builtin_bit_cast(uint16_t, (__bf16)f); }
__device__ inline float bf2f(uint32_t h) { return __uint_as_float(h << 16); }
__device__ inline uint32_t pack2(float lo, float hi) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(floatx2{lo, hi}, bf16x2));
}

template <int N>
__device__ inline void wait_vmcnt() {  // at most N vector-memory operations of this wave outstanding (vmcnt: bits 15:14, 3:0)
  __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}

// Activations [rows][K]: 16-row x 32-column tiles in the order [row / 16][col / 32], each tile 16 rows of 64
// contiguous bytes.  A producer that owns one row writes 64-byte runs (whole 32-byte sectors); a consumer reads a
// tile as one MFMA B-operand fragment, lane l taking the 16 bytes at row l % 16, columns 8 * (l / 16) .. + 7,
// i.e. 16-byte slot act_lane(l) of the 1 KiB tile.
__device__ inline long d_act_index(long row, long col, long K) {
  return ((row >> 4) * (K >> 5) + (col >> 5)) * 512 + (row & 15) * 32 + (col & 31);
}
__device__ inline int act_lane(int lane) { return (lane & 15) * 4 + (lane >> 4); }

// The same tile through LDS: loaded in rows (lane l fetches 16-byte piece staged_piece(l), so four lanes take the 64 bytes of
// a row, not 64 lanes 64 pieces of 16 rows), and read by the lane that needs row l % 16, piece l / 16 at place staged_lane(l).
// The pieces of a row are turned by its row / 4, so that 16 lanes that read one piece of 16 rows meet all 64 banks.
// Loaded in the order of act_lane a fragment costs the CU's vector memory path more, and tiles that are bound by what a CU
// takes in are slower: 912 rows of the 1.3B shape, us per launch, QKV 34.6 -> 31.3, FFN1 34.4 -> 33.1, FFN2 37.3 -> 34.8
// (128 x 256), output 16.7 -> 16.2 (128 x 128); 256 x 256 tiles with every CU busy, which the power limit bounds, alike.
__device__ inline int staged_turn(int row) { return -(row >> 2) & 3; }
__device__ inline int staged_piece(int lane) { return lane ^ staged_turn(lane >> 2); }
__device__ inline int staged_lane(int lane) { return (lane & 15) * 4 + ((lane >> 4) ^ staged_turn(lane & 15)); }

}  // namespace skd
