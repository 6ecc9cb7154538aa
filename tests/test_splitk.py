"""Split-K plans of the adjoint's products over grid rows (csrc/splitk.h, host
arithmetic): no block of a sweep may use more partial slices than the workspace
was sized for, whatever its length."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2208_07731_amd", "csrc")

SCAN = r"""
#include <initializer_list>
#include <cstdio>
#include "splitk.h"
using namespace isdf;
// slices of 128-wide tiles, two workgroups per CU: whole waves against the partials' traffic
static int earlier(long M, long N, bool lower, long K, int slots) {
  const long tm = (M + 127) / 128, tiles = lower ? tm * (tm + 1) / 2 : tm * ((N + 127) / 128);
  int best = 1;
  double best_t = 0;
  for (int s = 1; s <= 32 && (s == 1 || (K + s - 1) / s >= 512); s = s < 8 ? 8 : s + 8) {
    const double t = (double)((tiles * s + slots - 1) / slots) * ((double)K / s) * (32768.0 / (60e12 / slots)) +
                     (s > 1 ? s * 16.0 * M * N / 4e12 : 0.0);
    if (s == 1 || t < best_t * (1 - 1e-9)) best = s, best_t = t;
  }
  return best;
}
int main() {
  const SplitCaps any{MAX_SPLITS, MAX_SPLITS};
  long over = 0, changed = 0, longer = 0;
  for (int slots : {512, 256})
    for (int mu : {64, 168, 352, 355, 371, 519, 527, 1024, 2048})
      for (int n : {16, 64, 200})
        for (bool aliased : {false, true})
          for (int64_t rblock : {4096, 16384, 24576, 35705, 38751, 65536}) {
            const int64_t nr = 3 * rblock + rblock / 4, rest = nr % rblock, n1 = aliased ? mu : 2 * mu;
            const SplitCaps c = bwd_split_caps(nr, rblock, aliased, mu, n, n + n / 2, slots);
            for (int m : {n, n + n / 2})
              for (bool fused : {false, true}) {
                for (int64_t rows = 1; rows <= rblock; rows += 211) {
                  const BwdSplits b = bwd_splits(rows, n1, mu, m, fused, slots, c);
                  over += b.h.splits > c.h || b.q.splits > c.q;
                  longer += b.q.splits < earlier(2 * mu, 2 * m, 0, rows, slots) ||
                            b.h.splits < earlier(n1, n1, fused, rows, slots);
                }
                for (int64_t rows : {rblock, rest}) {  // the sized lengths keep their plans
                  const BwdSplits b = bwd_splits(rows, n1, mu, m, fused, slots, c);
                  const BwdSplits f = bwd_splits(rows, n1, mu, m, fused, slots, any);
                  changed += b.h.splits != f.h.splits || b.h.tile != f.h.tile || b.q.splits != f.q.splits ||
                             b.q.tile != f.q.tile;
                }
              }
            for (bool bf : {false, true})
              for (int64_t cap : {1, 2, 3, 8})
                for (int64_t rows = 32; rows <= rblock; rows += 3200)
                  over += split_k_for(out_tiles(n1, n1, 128, 1), rows, n1 * n1, slots, bf, cap) > cap;
          }
  std::printf("%ld %ld %ld\n", over, changed, longer);
}
"""


def test_no_block_exceeds_the_sized_partials(tmp_path):
    src, exe = tmp_path / "scan.cpp", tmp_path / "scan"
    src.write_text(SCAN)
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", f"-I{CSRC}", str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout
    over, changed, longer = map(int, out.split())
    assert over == 0 and changed == 0, out
    assert longer == 0, out  # no chain of additions longer than 128-wide tiles at two workgroups a CU give
