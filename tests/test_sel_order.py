"""CPU: the rules on the work chunks of the selection kernels (csrc/sel_order.h), compiled with g++.  Their order: over token counts and
numbers of KV heads it ends, its buckets fit their table and cover every position.  Their length in the one-pass backward: one that was
within 3 % of the fastest where it was measured."""
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
  const struct { int longest, entries, heads, fast, also; } measured[] = {
      {64, 64000, 8, 128, 128}, {64, 256000, 8, 128, 128}, {112, 544000, 8, 256, 128}, {32, 640000, 8, 256, 128}, {64, 1280000, 8, 256, 512}, {64, 2240000, 8, 512, 256},
      {32, 640000, 16, 128, 256}, {64, 16000, 2, 128, 128}, {64, 160000, 2, 256, 512}, {64, 384000, 2, 512, 512}, {64, 640000, 1, 512, 512}, {64, 160000, 1, 256, 512},
      {156, 96000, 8, 256, 128}, {213, 128000, 8, 128, 128}, {192, 256000, 8, 128, 256}, {241, 340960, 8, 512, 256}, {192, 96000, 4, 512, 256}, {192, 480000, 4, 512, 256},
      {192, 480000, 1, 512, 512}, {192, 80000, 1, 512, 256}, {316, 40000, 8, 128, 128}, {1618, 53400, 8, 256, 256}, {2765, 50000, 16, 256, 256}, {365, 64000, 8, 256, 256},
      {335, 136592, 8, 256, 256}, {290, 170480, 8, 256, 256}, {314, 224000, 8, 512, 256}, {290, 384000, 8, 512, 512}, {285, 640000, 8, 256, 512}, {1618, 53400, 1, 512, 512},
      {1004, 32000, 1, 256, 512}, {520, 16000, 1, 256, 256}, {1618, 26700, 8, 128, 256}, {1004, 32000, 16, 128, 128}};
  for (const auto &m : measured) {
    const int len = one_pass_chunk_len(m.longest, m.entries, m.heads);
    if (len != m.fast && len != m.also) {
      printf("blocks of up to %d keys, %d entries, %d heads: chunks of %d\n", m.longest, m.entries, m.heads, len);
      return 1;
    }
  }
  return one_pass_chunk_len(1, 0, 1) == DKV_CHUNK_MIN && one_pass_chunk_len(1 << 30, 1ll << 31, 16) == 512 ? 0 : 1;
}
"""


def test_rule(tmp_path):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-Wall", "-Werror", "-fsanitize=undefined", "-fno-sanitize-recover",
                           "-I" + os.path.join(ROOT, "paper_2505_17412_amd", "csrc"), "-o", str(exe), str(src)])
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
