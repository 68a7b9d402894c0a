"""CPU: the rules that pick how the gate predictor's forward pass runs (csrc/gate_form.h), compiled with g++: the form that was the
faster, or within 3 % of it, where they were measured."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r"""
#include "gate_form.h"
#include <cstdio>
int main() {
  const struct { int n, d_model, columns; bool as_is; } measured[] = {
      {5510, 1024, 48, true}, {62229, 1024, 48, true}, {150000, 1024, 24, true}, {400000, 1024, 48, true}, {5510, 1024, 36, false}, {700, 128, 48, true},
      {57000, 128, 48, false}, {98304, 128, 48, false}, {80000, 128, 48, false}, {250000, 128, 48, false}, {45904, 128, 48, true}, {98304, 128, 24, true},
      {131072, 128, 24, false}, {250000, 128, 24, false}, {65536, 256, 48, true}, {98304, 256, 48, false}, {115000, 256, 48, false}, {250000, 256, 24, true},
      {400000, 256, 24, false}, {115000, 384, 48, true}, {180000, 384, 48, true}, {250000, 384, 48, false}, {400000, 384, 24, true}, {250000, 512, 48, true}, {400000, 512, 48, false},
      {180000, 640, 48, true}, {250000, 640, 48, false}, {250000, 768, 48, false}, {196608, 896, 48, true}, {250000, 896, 48, false}, {131072, 1152, 48, false},
      {115000, 1152, 48, true}, {250000, 1536, 48, true}, {250000, 2048, 48, true}};
  for (const auto &m : measured)
    if (gate_as_is(m.n, m.d_model, m.columns) != m.as_is) {
      printf("%d tokens, %d features, %d columns\n", m.n, m.d_model, m.columns);
      return 1;
    }
  // what has no form of its own: whole contractions of 17 to 32 columns
  for (long long n = 1; n < 2000000000; n = n * 3 / 2 + 1)
    for (int d = 128; d <= 16384; d *= 2)
      if (!gate_split((int)n, d, 2)) return 2;
  return 0;
}
"""


def test_rules(tmp_path):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-Wall", "-Werror", "-fsanitize=undefined", "-fno-sanitize-recover",
                           "-I" + os.path.join(ROOT, "paper_2505_17412_amd", "csrc"), "-o", str(exe), str(src)])
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
