// The paged KV cache: its geometry and where values lie in a page.  Plain C++: what the kernels compute, the host can check.
#pragma once

namespace skd {

// Geometry of the paged KV cache.  A page holds `page_tokens` consecutive
// positions of ONE batch row in ONE layer, all heads.  On the bf16 path a row's
// keys are stored by real position (column j of a row that starts at column
// start[b] sits in slot j - start[b]; padding columns store nothing), so that a
// left-padded row reads no padding; the fp32 path stores by column.
struct KvGeom {
  int page_tokens;
  int max_pages;      // block-table entries per (layer, row)
  int H, dh;
  long page_elems;    // elements (fp32 or bf16) per page = 2 * page_tokens * H * dh
};

// bf16 page (one batch row, one layer): [head][32-key block][K block | V block],
// K block = [tile 0..1][chunk 0..dh/32-1][lane][8], V block = [dh/16][lane][8].
// A page may be larger than 4 GiB: heads and blocks are in 64 bits.
constexpr long kv_block_base(int h, int tt, const KvGeom &g) {
  return (long)h * g.page_tokens * (g.dh * 2) + (long)(tt >> 5) * (64 * g.dh);
}
constexpr long kv_k_off(int h, int tt, int e, const KvGeom &g) {
  const int kk = tt & 31;
  return kv_block_base(h, tt, g) +
         ((long)((kk >> 4) * (g.dh >> 5) + (e >> 5)) * 64 + (kk & 15) + 16 * ((e & 31) >> 3)) * 8 + (e & 7);
}
constexpr long kv_v_off(int h, int tt, int e, const KvGeom &g) {
  const int kk = tt & 31;
  return kv_block_base(h, tt, g) + 32 * g.dh +
         ((long)(e >> 4) * 64 + 16 * ((kk & 15) >> 2) + (e & 15)) * 8 + 4 * (kk >> 4) + (kk & 3);
}

// The same in parts, for 16 positions (half `half` of a block) at a time: kv_block_base + kv_k_half + kv_k_at is where the
// eight elements from e on (a multiple of 8) of the key at position `key` of the 16 begin, kv_block_base + kv_v_half + kv_v_at
// where the values of element e at four positions from `key` on (a multiple of 4) do.  Parts inside a block fit 32 bits.
constexpr int kv_k_half(int half, int dh) { return half * (dh >> 5) * 512; }
constexpr int kv_k_at(int key, int e) { return (e >> 5) * 512 + ((e & 31) >> 3) * 128 + 8 * key; }
constexpr int kv_v_half(int half, int dh) { return 32 * dh + 4 * half; }
constexpr int kv_v_at(int key, int e) { return (e >> 4) * 512 + (key >> 2) * 128 + (e & 15) * 8; }

// Where the keys and values of a 16-row tile of a prompt pass go.
struct CacheTile {
  int page;  // place of the page's number in a layer's block table
  int at;    // the tile's first position in the page (a multiple of 16) + its real positions - 1: fewer than 16 in the last
             // tile of a sequence; negative past the last sequence
  static constexpr CacheTile none() { return {0, -1}; }
  static constexpr CacheTile of(int page, int slot, int valid) { return {page, slot | (valid - 1)}; }
  static constexpr bool any(int at) { return at >= 0; }
  static constexpr int slot(int at) { return at & ~15; }
  static constexpr int valid(int at) { return (at & 15) + 1; }
};

}  // namespace skd
