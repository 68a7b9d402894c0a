"""CPU: the rule that picks how the compression branch runs (csrc/cmp_form.h), compiled with g++: every form it names fits the LDS of a
compute unit and has wavefronts on all four SIMDs, over all score rows the matrix path accepts; and the cases of the GPU test run
the form they name."""
import os
import subprocess

from tests.test_gpu_tile_edges import MANY_BLOCKS

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r"""
#include "cmp_form.h"
#include <cstdio>
#include <cstdlib>
int main(int argc, char **argv) {
  const char *const names[] = {"one_kernel", "tiles_in_lds", "own_tiles_4", "own_tiles_8"};
  for (int i = 1; i + 2 < argc; i += 3) printf("%s\n", names[(int)cmp_form(atoi(argv[i]), atoi(argv[i + 1]), atoi(argv[i + 2]))]);
  if (argc > 1) return 0;
  for (int D = 32; D <= 128; D *= 2)
    for (int hs = 1; hs <= 16; hs *= 2)
      for (int s = 1; s == 1 || cmp_rows_fit(D, hs, s); ++s) {
        const CmpForm f = cmp_form(D, hs, s);
        const size_t lds = f == CmpForm::one_kernel ? cmp_lds_bytes(D, 4, hs, s)
                           : f == CmpForm::tiles_in_lds ? scores_lds_bytes(D, hs, 2, 4, 2, s)
                                                        : scores_lds_bytes(D, hs, 1, f == CmpForm::own_tiles_4 ? 4 : 8, 0, s);
        const int waves = (int)(LDS_CU / ((lds + LDS_GRANULE - 1) / LDS_GRANULE * LDS_GRANULE)) * (f == CmpForm::own_tiles_8 ? 8 : 4);
        if (lds > LDS_CU || waves < 8 || (f == CmpForm::one_kernel && (hs < 4 || s > CMP_ONE_BLOCKS)) || (f == CmpForm::tiles_in_lds && hs < 2)) {
          printf("head_dim %d, %d heads per KV head, %d blocks: %s, %zu bytes, %d wavefronts\n", D, hs, s, names[(int)f], lds, waves);
          return 1;
        }
      }
  return 0;
}
"""


def test_rule(tmp_path):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-Wall", "-Werror", "-I" + os.path.join(ROOT, "paper_2505_17412_amd", "csrc"), "-o", str(exe), str(src)])
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
    args = [str(x) for _, lens, hq, hkv, d, _ in MANY_BLOCKS for x in (d, hq // hkv, max(-(-n // 8) for n in lens))]
    r = subprocess.run([str(exe), *args], capture_output=True, text=True, timeout=60, check=True)
    assert r.stdout.split() == [case[-1] for case in MANY_BLOCKS]
