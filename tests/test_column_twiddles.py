"""The lane twiddle tables of the column transforms without a GPU: the values that
the register passes assume, [k - 1][lane] for both transforms of a time axis, and
that making them is a small part of a problem's host tables."""
import os
import subprocess

import numpy as np
import pytest

from paper_2301_00406_amd import build_lib
from paper_2301_00406_amd import cnlos as C

PROGRAM = r"""
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include "cnlos_internal.h"
using namespace cnlos;
template <typename F> static double best_us(F f) {
  double best = 1e30;
  for (int i = 0; i < 100; ++i) {
    const auto a = std::chrono::steady_clock::now();
    f();
    const double us = std::chrono::duration<double>(std::chrono::steady_clock::now() - a).count() * 1e6;
    if (us < best) best = us;
  }
  return best;
}
int main(int argc, char** argv) {
  const int logm = atoi(argv[1]), m = 1 << logm;
  std::vector<float2> tw(m), fa, fb;
  for (int j = 0; j < m; ++j) {
    const double a = -M_PI * j / m;
    tw[j] = make_float2((float)cos(a), (float)sin(a));
  }
  std::vector<float4> rows, cols;
  const double t = best_us([&] { column_twiddles(logm, tw, fa, fb); });
  const double r = best_us([&] { resample_descriptors(m, rows, cols); });
  printf("%zu %zu %.3f %.3f\n", fa.size(), fb.size(), t, r);
  for (const auto* v : {&fa, &fb})
    for (const float2& z : *v) printf("%.9g %.9g\n", z.x, z.y);
  return 0;
}
"""


@pytest.fixture(scope="module")
def tables(tmp_path_factory):
    C.load()
    d = tmp_path_factory.mktemp("twiddles")
    src, exe = d / "t.hip", d / "t"
    src.write_text(PROGRAM)
    lib = os.path.dirname(C.LIB_PATH)
    subprocess.run([build_lib.hipcc(), "-x", "hip", "--cuda-host-only", "-O1", "-std=c++17",
                    "-I", build_lib.INCLUDE, "-I", build_lib.CSRC, str(src), "-o", str(exe),
                    "-L", lib, "-lcnlos", f"-Wl,-rpath,{lib}"], check=True, capture_output=True)

    def run(logm):
        out = subprocess.run([str(exe), str(logm)], capture_output=True, text=True, check=True)
        lines = out.stdout.splitlines()
        na, nb, us, us_rows = (float(x) for x in lines[0].split())
        z = np.array([[float(x) for x in ln.split()] for ln in lines[1:]]).reshape(-1, 2)
        z = z[:, 0] + 1j * z[:, 1]
        return z[:int(na)], z[int(na):], us, us_rows
    return run


@pytest.mark.parametrize("logm", [7, 8, 9, 10, 11])
def test_tables_hold_the_roots_of_unity(tables, logm):
    fa, fb, _, _ = tables(logm)
    ea, eb = [], []
    lane = np.arange(64)
    for logf in (logm, logm - 1):
        if not 8 <= logf <= 10:                    # lengths without register passes
            continue
        E = 2 ** logf // 64
        low = {4: 15, 8: 7, 16: 3}[E]              # lane bits that the later pass turns by
        for k in range(1, E):
            ea.append(np.exp(-2j * np.pi * lane * k / 2 ** logf))
            eb.append(np.exp(-2j * np.pi * (lane & low) * k / 64))
        if E == 4:
            eb.append(np.exp(-2j * np.pi * np.arange(16) / 16))
    for got, ref in ((fa, ea), (fb, eb)):
        ref = np.concatenate(ref) if ref else np.zeros(0)
        assert got.shape == ref.shape
        # parts of at most 1 rounded to FP32
        assert max(np.abs(got.real - ref.real).max(initial=0.0),
                   np.abs(got.imag - ref.imag).max(initial=0.0)) <= 2.0 ** -24


def test_tables_cost_little_beside_the_resampling_rows(tables):
    """The entries are looked up: a sine and a cosine for each took a third of the
    time of the resampling rows, the largest of the other tables."""
    _, _, us, us_rows = tables(10)
    assert us <= 0.15 * us_rows, (us, us_rows)
