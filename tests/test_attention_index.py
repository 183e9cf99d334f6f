"""Key-tile indices of the single-load attention form (csrc/attn_span.h), checked
on the CPU: every tile a wavefront loads lies inside its block's key range, and the
wavefronts of a workgroup together compute each tile once. The kernel instance
follows the longest span of a launch, so the blocks of a chained run (prompt
encoding) are taken with the run's own instance."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

HARNESS = r"""
#include <cstdio>
#include <vector>
#include "attn_span.h"

// the kernel's loads and computed tiles for block br of a launch whose instance
// holds NT tiles per wavefront; 0 if every one is in range and each tile is
// computed once
static int check(const AttnSpan& s, int NT, long* idle) {
  const int T = key_tiles(s), buf = sl_buffers(NT);
  if (T < 1) return 1;
  std::vector<int> seen(T, 0);
  for (int wv = 0; wv < SL_WAVES; ++wv) {
    const SlRange r = sl_range(T, wv);
    if (r.nt > NT) return 2;
    if (r.nt == 0) ++*idle;
    for (int i = 0; i < NT; ++i) {
      if (i < r.nt) ++seen[r.t_lo + i];
      if (NT == buf && i >= r.nt) continue;  // this instance loads under i < nt
      const int t = NT == buf ? r.t_lo + i : sl_tile(r, i);
      if (t < 0 || t >= T) return 3;
    }
  }
  for (int n : seen)
    if (n != 1) return 4;
  return 0;
}

int main() {
  long launches = 0, idle = 0;
  const int prefixes[] = {0, 1, 3, 31, 32, 33, 100, 224, 225, 500, 768, 1000, 2016, 3000, 4095};
  const int blocks[] = {1, 7, 16, 25, 32, 33, 50, 64, 100, 255, 256};
  for (int P : prefixes)
    for (int L : blocks)
      for (int chain = 0; chain < 2; ++chain)
        for (int rows = L; rows <= 2048; rows += chain ? (rows < 64 ? 1 : 37) : 2048) {
          const int nb = chain ? (rows + L - 1) / L : 1;
          const AttnSpan last = attn_span(P, L, chain ? rows : 0, nb - 1);
          int NT = (key_tiles(last) + SL_WAVES - 1) / SL_WAVES;
          if (NT > 16) continue;
          if (NT > 8) NT = (NT + 1) / 2 * 2;
          ++launches;
          for (int br = 0; br < nb; ++br) {
            const int e = check(attn_span(P, L, chain ? rows : 0, br), NT, &idle);
            if (e) {
              printf("error %d: prefix %d, blocks of %d, %d rows, block %d, %d tiles\n", e, P, L, rows, br, NT);
              return 1;
            }
          }
        }
  printf("%ld launches, %ld wavefronts without a tile\n", launches, idle);
  return launches > 1000 && idle > 1000 ? 0 : 2;  // the sweep reaches what it is for
}
"""


def test_single_load_tiles_stay_in_range(tmp_path):
    cxx = shutil.which("g++") or shutil.which("amdclang++")
    if not cxx:
        pytest.skip("no host C++ compiler")
    src, exe = tmp_path / "tiles.cpp", tmp_path / "tiles"
    src.write_text(HARNESS)
    subprocess.run([cxx, "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2512_16229_amd", "csrc"),
                    str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
