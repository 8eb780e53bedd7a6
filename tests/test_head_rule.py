"""Which last layers share a kernel with the loss and their input gradient (csrc/tile_rules.hpp, compiled for the host)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r"""
#include <stdio.h>
#include "tile_rules.hpp"
int main() {
  int in, classes;
  while (scanf("%d %d", &in, &classes) == 2) printf("%d\n", (int)sasgd::head_kernel_wins(in, classes));
}
"""
# Measured, us, calls of 64 images (of 1 024 in the last row): inputs, classes; separate kernels, one kernel
MEASURED = [(8, 31, 29.5, 25.3), (8, 301, 39.8, 49.7), (8, 1001, 67.1, 114.5), (8, 3001, 144.2, 308.9), (16, 101, 33.2, 30.4), (16, 1001, 65.0, 119.4), (32, 101, 35.5, 32.5),
            (32, 301, 44.1, 48.7), (32, 1001, 68.8, 121.8), (64, 101, 40.5, 31.2), (64, 301, 54.6, 49.7), (128, 101, 50.7, 31.4), (256, 101, 35.2, 31.7),
            (512, 31, 34.1, 22.8), (1024, 31, 90.7, 45.9)]


def test_the_rule_takes_the_faster_way(tmp_path):
    (tmp_path / "rule.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "paper_1511_05950_amd", "csrc"), str(tmp_path / "rule.cpp"), "-o", str(tmp_path / "rule")], check=True)
    out = subprocess.run([str(tmp_path / "rule")], input="\n".join("%d %d" % m[:2] for m in MEASURED), capture_output=True, text=True, check=True).stdout
    assert [line == "1" for line in out.split()] == [m[3] < m[2] for m in MEASURED]
