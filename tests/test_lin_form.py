"""CPU: the rules that pick the projections' tiles (csrc/lin_form.h), compiled with g++: the form that was the faster where both were
measured, and the cases of the GPU tests run the form they name."""
import os
import subprocess

from tests.test_gpu_linear import WEIGHT_GRADIENT_CASES, WIDE_CASES

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r"""
#include "lin_form.h"
#include <cstdio>
#include <cstdlib>
int main(int argc, char **argv) {
  if (argc > 1 && argv[1][0] == 't') {
    for (int i = 2; i + 3 < argc; i += 4) printf("%d\n", lin_tn_splits(atoi(argv[i]), atoi(argv[i + 1]), atoi(argv[i + 2]), atoi(argv[i + 3])));
    return 0;
  }
  const int gradient = argc > 1 && argv[1][0] == 'g';
  for (int i = 1 + gradient; i + 2 < argc; i += 3) printf("%d\n", (int)lin_wide(atoi(argv[i]), atoi(argv[i + 1]), atoi(argv[i + 2]), gradient));
  return 0;
}
"""
#: tokens, features, contraction, time in tiles of 128 over time in tiles of 256
MEASURED = [
    (12800, 1280, 1024, 0.85), (10655, 1408, 1024, 0.73), (10655, 1408, 2048, 0.78), (12800, 1280, 128, 0.81), (20000, 1024, 1024, 0.88),
    (32768, 640, 1024, 0.91), (12800, 1024, 1024, 1.13), (10655, 1280, 1024, 1.15), (32768, 1280, 1024, 1.15), (45904, 1280, 1024, 1.22),
    (45904, 1024, 1024, 1.10), (20000, 1408, 512, 0.97), (24576, 1024, 512, 0.97), (45904, 1280, 512, 1.12), (16384, 1024, 256, 1.15),
    (24576, 1024, 256, 0.94), (12800, 1024, 256, 1.11), (10655, 1280, 512, 1.15), (20000, 640, 256, 1.08), (32768, 384, 512, 0.96), (32768, 384, 256, 0.98),
    (100000, 1408, 128, 1.14), (150000, 1280, 128, 1.17), (150000, 1024, 128, 1.10), (62229, 2048, 128, 0.96), (62229, 1280, 256, 1.11), (24576, 1024, 128, 0.86), (24576, 2048, 128, 0.95), (20000, 2048, 128, 0.90),
]

#: the same of a data gradient with the weight gradient behind it (features are the inputs, the contraction the outputs)
MEASURED_GRADIENT = [
    (160000, 1024, 128, 0.92), (260000, 640, 128, 0.97), (100000, 2048, 128, 0.97), (200000, 2048, 128, 1.04), (260000, 1280, 128, 1.045), (16384, 1024, 256, 1.04),
    (40960, 768, 256, 1.02), (16384, 2048, 256, 1.04), (80000, 1024, 256, 0.95), (160000, 1024, 256, 0.93), (330000, 1024, 256, 0.97), (49152, 1280, 256, 0.96),
    (200000, 2048, 256, 0.98), (260000, 768, 384, 1.05), (131072, 1280, 384, 1.04), (160000, 1024, 512, 1.05),
]

#: tokens, inputs, outputs, workgroups in tiles of 128, time in them over time in tiles of 256 (weight gradient)
MEASURED_TN = [
    (6151, 1024, 1024, 768, 0.97), (12295, 1024, 1024, 768, 1.05), (12295, 256, 2048, 768, 0.92), (32775, 2048, 256, 768, 1.004), (1543, 2048, 2048, 768, 0.90),
    (4103, 2048, 2048, 768, 1.06), (4615, 1024, 1280, 800, 1.08), (3079, 1408, 1280, 880, 1.20), (32775, 1024, 384, 768, 0.93), (32775, 384, 1024, 768, 1.28), (14407, 384, 1024, 744, 1.13),
    (8199, 384, 4096, 768, 1.01), (2055, 384, 4096, 768, 0.91), (3607, 1024, 1280, 800, 0.90), (10927, 640, 1024, 760, 1.22), (26887, 1408, 256, 748, 1.13),
    (40967, 1024, 256, 768, 1.08), (19207, 256, 1024, 736, 0.91), (8327, 384, 2048, 768, 0.99),
]


def forms(tmp_path, sizes, kind=()):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-Wall", "-Werror", "-fsanitize=undefined", "-fno-sanitize-recover",
                           "-I" + os.path.join(ROOT, "paper_2505_17412_amd", "csrc"), "-o", str(exe), str(src)])
    args = [*kind, *(str(x) for s in sizes for x in s)]
    out = subprocess.run([str(exe), *args], capture_output=True, text=True, timeout=60, check=True).stdout
    return [int(line) for line in out.split()]


def test_wide_tiles_where_they_are_faster(tmp_path):
    for (m, f, k, ratio), wide in zip(MEASURED, forms(tmp_path, [s[:3] for s in MEASURED])):
        assert wide == (ratio > 1), (m, f, k, ratio)
    for (m, f, k, ratio), wide in zip(MEASURED_GRADIENT, forms(tmp_path, [s[:3] for s in MEASURED_GRADIENT], "g")):
        assert wide == (ratio > 1), ("gradient", m, f, k, ratio)


def test_weight_gradient_in_wide_tiles_where_they_are_faster(tmp_path):
    for (m, d_in, f, wgs, ratio), splits in zip(MEASURED_TN, forms(tmp_path, [s[:4] for s in MEASURED_TN], "t")):
        assert (splits > 0) == (ratio > 1) and splits <= 64, (m, d_in, f, ratio, splits)


def test_cases_of_the_gpu_test(tmp_path):
    sizes = [(n, d_out, d_in) for _, n, d_in, d_out, _, _ in WIDE_CASES]
    assert forms(tmp_path, sizes) == [wide for *_, wide in WIDE_CASES]
    # a layer's query, key and value projections, and their data gradient, in test_projections_in_wide_tiles
    assert forms(tmp_path, [(12400, 1280, 1024), (12288, 1280, 1024), (12225, 1280, 1024), (32768, 384, 768)]) == [False] + 3 * [True]
    assert forms(tmp_path, [(12400, 1024, 1280)], "g") == [True]
    sizes = [(n, d_in, d_out, wgs) for n, d_in, d_out, wgs, _ in WEIGHT_GRADIENT_CASES]
    assert [s > 0 for s in forms(tmp_path, sizes, "t")] == [wide for *_, wide in WEIGHT_GRADIENT_CASES]
    largest = 2 ** 31 - 1  # tokens x the larger dimension stay below 2^31
    assert all(w in (0, 1) for w in forms(tmp_path, [(0, 128, 128), (1, 128, 128), (largest // 128, 128, 128), (largest // 16384, 16384, 16384)]))
