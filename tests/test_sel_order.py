"""CPU: the rule that orders the work chunks of the selection kernels (csrc/sel_order.h), compiled with g++: over token counts and
numbers of KV heads it ends, its buckets fit their table and cover every position."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r"""
#include "sel_order.h"
#include <cstdio>
int main() {
  const int heads[] = {1, 2, 3, 16, 1023, 1024, 1025, 2048, 2049, 4097, 8191, 8192, 8193, 20000, 2000000000};
  const int tokens[] = {1, 63, 24576, 24577, 62229, 1 << 20, 100000007, 666666666};
  for (int h : heads)
    for (int n : tokens) {
      const SelOrder o = sel_order(n, h);
      const bool ok = o.by_length ? n <= BY_LENGTH_TOKENS || h > ORDER_BINS
                                  : o.bucket >= 64 && o.per_head >= 1 && o.classes >= 1 && (long long)o.bucket * o.per_head >= n &&
                                        (long long)o.classes * h * o.per_head <= ORDER_BINS;
      // stretches and classes are no coarser than they have to be
      const bool fine = o.by_length || ((o.bucket == 64 || (long long)o.classes * h * ((n + (o.bucket / 2) - 1ll) / (o.bucket / 2)) > ORDER_BINS) &&
                                        (o.classes == ORDER_CLASSES || 2ll * o.classes * h > ORDER_BINS));
      if (!ok || !fine) {
        printf("%d heads, %d tokens: by_length %d bucket %d per_head %d classes %d\n", h, n, o.by_length, o.bucket, o.per_head, o.classes);
        return 1;
      }
    }
  return 0;
}
"""


def test_rule(tmp_path):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-Wall", "-Werror", "-fsanitize=undefined", "-fno-sanitize-recover",
                           "-I" + os.path.join(ROOT, "paper_2505_17412_amd", "csrc"), "-o", str(exe), str(src)])
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
