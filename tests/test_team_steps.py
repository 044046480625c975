"""The order in which the one-launch column adds up a projection along K (its tables of k-steps) is the separate kernels', for
every width, ffn, padded batch and K split that they plan (CPU only; the library's function, called by a compiled driver)."""
import os
import subprocess

from paper_2307_02628_amd import _build, skd

DRIVER = r"""
#include <cstdio>
#include <vector>
#include "skd_kernels.h"
using namespace skd;
// k-steps of one wave of the separate kernel, in the order in which it adds them: buffers of `unit` k-steps dealt to the waves in
// turn, or (rotated) stages of four from a stage that depends on the tile and the part
static std::vector<int> reference(int Kf, int split, int unit, int waves, bool rotate, int tile, int part, int wave) {
  std::vector<int> k;
  const int n = Kf / split;
  while (unit > 1 && n % unit) unit >>= 1;
  if (rotate) {
    const int stages = n / 4, first = ((tile >> 3) * 5 + part * 3) % stages;
    for (int i = 0; i < stages; ++i) k.push_back(part * n + (first + i) % stages * 4 + wave);
  } else {
    for (int j = wave; j < n / unit; j += waves)
      for (int u = 0; u < unit; ++u) k.push_back(part * n + j * unit + u);
  }
  return k;
}
static int check(const std::vector<TeamStep> &table, int d, int Kf, const TeamSums &p) {
  for (int tile = 0; tile < d / 16; ++tile) {
    std::vector<int> sums;
    for (int w = 0; w < 8; ++w) {
      std::vector<int> at;
      for (uint32_t e : table[tile * 8 + w].e) {
        if (!e) break;
        if (e & 64) at.push_back(e & 63);
        if (!(e & 128)) continue;
        const int sum = e >> 9;
        if (at != reference(Kf, p.split, p.unit, p.waves, p.rotate, tile, sum / p.waves, sum % p.waves)) return 1;
        sums.push_back(sum);
        at.clear();
      }
      if (!at.empty()) return 2;  // a sum that does not end
    }
    std::vector<int> seen(p.split * p.waves, 0);
    for (int s : sums)
      if (s < 0 || s >= (int)seen.size() || seen[s]++) return 3;
    if ((int)sums.size() != p.split * p.waves) return 4;  // every wave's sum once, those without k-steps as zero
  }
  return 0;
}
int main() {
  long taken = 0, refused = 0;
  for (int d = 64; d <= 512; d += 64)
    for (int f = 32; f <= 2048; f += 32)
      for (int pad : {16, 32, 48, 64, 96, 128}) {
        const int waves = pad >= 96 ? 4 : 8;
        auto plan = [&](int K) {  // K split as long as a wave keeps two k-steps
          const int Kf = K / 32;
          int S = 1;
          while (S < 16 && d / 16 * S < 256 && Kf % (2 * S) == 0 && Kf / (2 * S) >= 2 * waves) S *= 2;
          const bool ws = pad >= 96 && Kf / S % 4 == 0;
          return TeamSums{1, waves, ws ? 1 : pad <= 16 ? 2 : 1, S, ws};
        };
        const bool ws = pad >= 96 && d / 32 % 4 == 0;
        const TeamSums direct{1, waves, 1, 1, ws}, out = plan(d), ffn2 = plan(f);
        std::vector<TeamStep> a(bf16_team_steps(d)), b(bf16_team_steps(d));
        TeamArgs t{};
        t.d = d;
        t.f = f;
        const bool ok = bf16_team_sums(t, pad, direct, out, direct, ffn2, a.data(), b.data());
        if (ok != bf16_team_sums(t, pad, direct, out, direct, ffn2, nullptr, nullptr)) { printf("FAILED %d %d %d: the check alone\n", d, f, pad); return 1; }
        if (!ok) {
          if (pad < 96 || f / 32 % 2 == 0 || f <= 1024) { printf("FAILED %d %d %d: refused\n", d, f, pad); return 1; }
          ++refused;
          continue;
        }
        const int r = check(a, d, d / 32, out), s = check(b, d, f / 32, ffn2);
        if (r || s || t.wide != (pad >= 96) || t.out_parts != out.split || t.ffn2_parts != ffn2.split) { printf("FAILED %d %d %d: %d %d\n", d, f, pad, r, s); return 1; }
        ++taken;
      }
  // what the column cannot take
  TeamArgs t{};
  t.d = 256;
  t.f = 1024;
  const TeamSums good{1, 8, 1, 1, false};
  for (TeamSums bad : {TeamSums{2, 8, 1, 1, false}, TeamSums{1, 4, 1, 1, false}, TeamSums{1, 8, 1, 3, false},
                       TeamSums{1, 8, 1, 8, false}, TeamSums{1, 8, 1, 1, true}, TeamSums{1, 8, 1, 0, false}, TeamSums{1, 8, 0, 1, false}})
    if (bf16_team_sums(t, 16, good, good, good, bad, nullptr, nullptr)) { printf("FAILED: taken %d %d %d %d\n", bad.tiles, bad.waves, bad.unit, bad.split); return 1; }
  if (!bf16_team_sums(t, 16, good, good, good, good, nullptr, nullptr)) { printf("FAILED: refused\n"); return 1; }
  printf("all checks passed: %ld taken, %ld refused\n", taken, refused);
  return 0;
}
"""


def test_tables(tmp_path):
    if not os.path.exists(skd.LIB_PATH):
        _build.build(force=True)
    src, exe = tmp_path / "driver.hip", str(tmp_path / "driver")
    src.write_text(DRIVER)
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "--offload-arch=gfx950", "-std=c++17", "-O1", "-Xclang", "-target-feature", "-Xclang",
                    "-packed-fp32-ops", "-x", "hip", "-I", _build.CSRC, str(src), "-x", "none", skd.LIB_PATH, "-o", exe,
                    "-Wl,-rpath," + os.path.dirname(skd.LIB_PATH)], check=True, capture_output=True)
    res = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert res.returncode == 0 and "all checks passed" in res.stdout, res.stdout + res.stderr
