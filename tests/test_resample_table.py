"""The resampling descriptors of the t passes without a GPU: for every supported
time axis, what a row reads of its column exists (samples of the column, prefix
sums among the lane-rows that the pass writes, inside the column's part of the
LDS), and rows and columns give R_z and its transpose.  The table and the index
rule are the library's own: a host program includes the internal header and
links the library."""
import os
import subprocess

import numpy as np
import pytest

from oracle import cnlos_oracle as O
from paper_2301_00406_amd import build_lib
from paper_2301_00406_amd import cnlos as C

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include "cnlos_internal.h"
using namespace cnlos;
int main(int argc, char** argv) {
  const int m = atoi(argv[1]);
  std::vector<float4> rows, cols;
  if (const char* why = resample_descriptors(m, rows, cols)) {
    printf("refused: %s\n", why);
    return 1;
  }
  const int lanes = m / 2 < 64 ? m / 2 : 64;
  printf("%d %d %d\n", lanes, resample_scan_rows(m, lanes) * lanes, resample_long_rows(m));
  for (const auto* t : {&rows, &cols})
    for (const float4& d : *t) {
      int bits;
      memcpy(&bits, &d.w, sizeof(bits));
      const RzIndex x = rz_index(bits);
      printf("%.9g %.9g %.9g %d %d %d %d %d %d\n", d.x, d.y, d.z, bits, x.k0, x.k2, x.p0, x.p2,
             (int)x.lg);
    }
  return 0;
}
"""


@pytest.fixture(scope="module")
def table(tmp_path_factory):
    C.load()                                   # fails loudly when the library is not built
    d = tmp_path_factory.mktemp("resample")
    src, exe = d / "t.hip", d / "t"
    src.write_text(PROGRAM)
    lib = os.path.dirname(C.LIB_PATH)
    subprocess.run([build_lib.hipcc(), "-x", "hip", "--cuda-host-only", "-O1", "-std=c++17",
                    "-I", build_lib.INCLUDE, "-I", build_lib.CSRC, str(src), "-o", str(exe),
                    "-L", lib, "-lcnlos", f"-Wl,-rpath,{lib}"], check=True, capture_output=True)

    def run(m):
        out = subprocess.run([str(exe), str(m)], capture_output=True, text=True)
        assert out.returncode == 0, out.stdout + out.stderr
        lines = out.stdout.splitlines()
        lanes, scanned, long_end = (int(x) for x in lines[0].split())
        v = [[float(x) for x in ln.split()] for ln in lines[1:]]
        return lanes, scanned, long_end, np.array(v[:m]), np.array(v[m:])
    return run


@pytest.mark.parametrize("m", [16, 32, 64, 128, 256, 512, 1024, 2048])
def test_rows_read_only_what_the_pass_writes(table, m):
    lanes, scanned, long_end, rows, cols = table(m)
    k0, k2, p0, p2, lg = (rows[:, i].astype(int) for i in (4, 5, 6, 7, 8))
    assert k0.min() >= 0 and (k0 + 2).max() < m and k2.max() < m
    # prefix sums: entries 0 .. scanned - 1, FP64 where a column has a whole wave,
    # after the m samples in the column's m + m/8 + 4 pairs of floats
    assert min(p0.min(), p2.min()) >= 0 and max(p0.max(), p2.max()) < scanned
    size = 8 if lanes == 64 else 4
    assert 4 * m + size * (max(p0.max(), p2.max()) + 1) <= 8 * (m + m // 8 + 4)
    assert not lg[long_end:].any()             # the other rows are compiled without prefix sums
    assert ((cols[:, 3].astype(int) + 2) < m).all()


@pytest.mark.parametrize("m", [16, 32, 64, 128, 256, 512, 1024, 2048])
def test_descriptors_are_the_resampling_table(table, m):
    _, _, _, rows, cols = table(m)
    R = np.zeros((m, m))
    for q, (w0, w1, w2, _, k0, k2, p0, p2, lg) in enumerate(rows):
        k0, k2 = int(k0), int(k2)
        for k, w in ((k0, w0), (k0 + 1, w1), (k2, w2)):
            R[q, k] += w
        if lg:
            R[q, int(p0):int(p2)] += 1.0       # difference of two exclusive prefix sums
    S = O.resample_matrix(m)
    assert np.abs(R - S).max() <= 2.0 ** -24   # weights are at most 1, rounded to FP32
    T = np.zeros((m, m))
    for k, (w0, w1, w2, q0) in enumerate(cols[:, :4]):
        for j, w in enumerate((w0, w1, w2)):
            T[int(q0) + j, k] += w
    assert np.abs(T - S).max() <= 2.0 ** -24
