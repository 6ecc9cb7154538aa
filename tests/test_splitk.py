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
int main() {
  const SplitCaps any{MAX_SPLITS, MAX_SPLITS};
  long over = 0, changed = 0, shorter = 0;
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
                  const BwdSplits f = bwd_splits(rows, n1, mu, m, fused, slots, any);
                  shorter += f.h.splits > c.h || f.q.splits > c.q;
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
  std::printf("%ld %ld %ld\n", over, changed, shorter);
}
"""


def test_no_block_exceeds_the_sized_partials(tmp_path):
    src, exe = tmp_path / "scan.cpp", tmp_path / "scan"
    src.write_text(SCAN)
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", f"-I{CSRC}", str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout
    over, changed, shorter = map(int, out.split())
    assert over == 0 and changed == 0, out
    assert shorter > 0, out  # the scan does hold blocks whose own best plan would not fit
