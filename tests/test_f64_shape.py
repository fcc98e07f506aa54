"""LDS of the FP64 neural kernels over every tile shape: what a launch asks
for (laid out in f64_shape.hpp) and what the kernels declare statically stay
within a compute unit's 163,840 bytes, and the log-density's scratch, the
input rows, holds the state.  Host arithmetic, built with the host compiler."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2210_12375_amd", "csrc")

# 80 bytes: the most a kernel of f64_mfma.hip or the fused solve declares (the
# adjoint's row flags int[16] and two words)
WALK = r"""
#include <cstdio>
#include "f64_shape.hpp"
using namespace bode::f64t;
int main() {
  const size_t kUnit = 163840, kStatic = 80;
  long bad = 0, most = 0, fits = 0;
  const int Bs[] = {1, 1024, 1025, 2048, 2049, 100000}, slots[] = {0, 7, 8};
  for (int cnf = 0; cnf < 2; ++cnf)
    for (int d = 1; d <= 1100; ++d)
      for (int H = 1; H <= 2600; ++H) {
        if (!tile_fits(d, H, cnf)) continue;
        ++fits;
        if (dims(d, H).SX < d + 1) ++bad;
        for (int B : Bs)
          for (int s : slots) {
            const LdsPlan p =
                lds_plan(row_groups(B, d, H, cnf), d + cnf, d, H, cnf, s);
            if ((long)p.bytes > most) most = p.bytes;
            if (p.bytes + kStatic > kUnit && ++bad <= 20)
              std::printf("d=%d H=%d B=%d cnf=%d slots=%d: %zu\n", d, H, B,
                          cnf, s, p.bytes);
          }
      }
  std::printf("%ld shapes, largest %ld bytes, %ld over\n", fits, most, bad);
  return bad != 0;
}
"""


def test_lds_of_every_shape(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host compiler")
    src, exe = tmp_path / "walk.cpp", tmp_path / "walk"
    src.write_text(WALK)
    subprocess.run([gxx, "-std=c++17", "-O2", "-I", CSRC, str(src), "-o",
                    str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
    assert int(r.stdout.split()[0]) > 1_000_000
