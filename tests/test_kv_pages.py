"""Places in a page of the KV cache, on the CPU with the kernels' own arithmetic: pages of more than 4 GiB, whose heads lie beyond
32 bits, and the parts that the prompt tiles add up, against the layout."""
import subprocess

from paper_2307_02628_amd import _build

DRIVER = r"""
#include <cstdint>
#include <cstdio>
#include <initializer_list>
#include "kv_pages.h"
using namespace skd;
#define EXPECT(c) do { if (!(c)) { printf("FAILED %s:%d: %s (head %d, slot %d, element %d, dh %d, page_tokens %d)\n", \
                                          __FILE__, __LINE__, #c, h, slot, e, dh, pt); return 1; } } while (0)
int main() {
  // up to half the positions that an int can count, in whole blocks; 2^19 x 128: head 16 begins at 2^31
  for (int dh : {64, 128})
    for (int pt : {32, 96, 1 << 19, (1 << 23) + 32, 1 << 26, 1 << 30})
      for (int h : {0, 1, 15, 16, 31, 255})
        for (int slot : {0, 16, pt / 64 * 32, pt - 32, pt - 16}) {
          const KvGeom g{pt, 1, 256, dh, 2L * pt * 256 * dh};
          const int64_t block = (int64_t)h * pt * dh * 2 + (int64_t)(slot / 32) * 64 * dh;  // [head][block][K | V][32][dh]
          const int half = slot % 32 / 16;
          for (int e = 0; e < dh; ++e) {
            EXPECT(kv_block_base(h, slot, g) == block);
            for (int key = 0; key < 16; ++key) {
              // K: [half][32 elements][lane][8], lane = key + 16 (8 elements); V: [16 elements][lane][8], lane = element + 16 (4 keys)
              const int64_t k = block + ((half * (dh / 32) + e / 32) * 64 + key + 16 * (e % 32 / 8)) * 8 + e % 8;
              const int64_t v = block + 32 * dh + (e / 16 * 64 + 16 * (key / 4) + e % 16) * 8 + 4 * half + key % 4;
              EXPECT(k < g.page_elems && v < g.page_elems);
              EXPECT(kv_k_off(h, slot + key, e, g) == k && kv_v_off(h, slot + key, e, g) == v);
              EXPECT(kv_block_base(h, slot, g) + kv_k_half(half, dh) + kv_k_at(key, e / 8 * 8) + e % 8 == k);
              EXPECT(kv_block_base(h, slot, g) + kv_v_half(half, dh) + kv_v_at(key, e) + key % 4 == v);
            }
          }
        }
  const int h = 0, e = 0, dh = 0, pt = 0;
  for (int slot : {0, 16, 32, 1 << 26, (1 << 30) + 16, 0x7ffffff0})
    for (int valid = 1; valid <= 16; ++valid) {
      const CacheTile t = CacheTile::of(7, slot, valid);
      EXPECT(t.page == 7 && CacheTile::any(t.at) && CacheTile::slot(t.at) == slot && CacheTile::valid(t.at) == valid);
    }
  const int slot = 0;
  EXPECT(!CacheTile::any(CacheTile::none().at) && CacheTile::none().page == 0);
  printf("all checks passed\n");
  return 0;
}
"""


def test_places(tmp_path):
    src = tmp_path / "driver.cpp"
    src.write_text(DRIVER)
    exe = str(tmp_path / "driver")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-O2", "-fsanitize=undefined", "-I", _build.CSRC, str(src), "-o", exe], check=True)
    res = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0 and "all checks passed" in res.stdout and not res.stderr, res.stdout + res.stderr
