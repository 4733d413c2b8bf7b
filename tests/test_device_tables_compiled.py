"""The adjoint's table-driven exp2, sine and cosine as they stand in the sources,
compiled for the host (their functions, coefficients and tables taken out of the
files, not written again), against numpy in extended precision.  Bounds: five
roundings of terms of at most 1 for the joined sine (6e-16 with the table's), six
relative ones for exp2 (7e-16)."""
import os
import re
import shutil
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2104_12922_amd", "csrc")
MAIN = """
#include <cmath>
#include <cstdio>
#define __device__
#define __forceinline__ inline
struct double2 { double x, y; };
inline double2 make_double2(double x, double y) { return {x, y}; }
#include "series_tables.h"
#include "sine_table.h"
using namespace synth::voice;
constexpr double kTwoPi = 6.283185307179586476925286766559;
constexpr double kLn2 = 0.693147180559945309417232121458;
%s
int main() {
  double2 sct[256];
  double e2t[64], v;
  for (int j = 0; j < 256; ++j) sct[j] = sincos_entry(j);
  for (int j = 0; j < 64; ++j) e2t[j] = kExp2T[4 * j];
  while (fread(&v, sizeof v, 1, stdin) == 1) {
    double out[3];
    out[0] = exp2_table(e2t, -v);
    sincos_table(sct, v, out[1], out[2]);
    fwrite(out, sizeof out, 1, stdout);
  }
}
"""


def _part(name, first, last):
    txt = open(os.path.join(CSRC, name)).read()
    a = txt.index(first)
    return txt[a:txt.index(last, a) + len(last)]


@pytest.fixture(scope="module")
def evaluate(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("clang++")
    if not cxx:
        pytest.skip("needs a C++ compiler")
    parts = [_part("voice_device.h", "enum {\n  kExpC3", "};"),
             _part("voice_device.h", "static __device__ double kSeriesC", "};")]
    for f in ("double2 sincos_entry", "void sincos_table", "double exp2_table"):
        parts.append(_part("adjoint.hip", "__device__ __forceinline__ " + f, "\n}\n"))
    d = tmp_path_factory.mktemp("tables")
    (d / "main.cpp").write_text(MAIN % "\n".join(parts))
    subprocess.run([cxx, "-std=c++17", "-O1", "-ffp-contract=off", "-I", CSRC, str(d / "main.cpp"), "-o",
                    str(d / "eval")], check=True)

    def run(v):
        out = subprocess.run([str(d / "eval")], input=np.asarray(v, np.float64).tobytes(),
                             capture_output=True, check=True).stdout
        return np.frombuffer(out, np.float64).reshape(-1, 3).T
    return run


def test_the_tables_of_the_kernel_are_these():
    txt = open(os.path.join(CSRC, "adjoint.hip")).read()
    assert re.search(r"sct\[j\] = sincos_entry\(j\);", txt)
    assert re.search(r"e2t\[j\] = kExp2T\[4 \* j\];", txt)


def test_exp2(evaluate):
    rng = np.random.default_rng(1)
    y = np.concatenate([rng.uniform(0.0, 60.0, 100000), rng.uniform(0.0, 1000.0, 20000),
                        np.arange(0.0, 20.0, 1.0 / 128), [0.0]])
    e = evaluate(y)[0]
    assert np.abs(e / np.exp2(-np.longdouble(1) * y) - 1).max() <= 7e-16
    assert evaluate([5000.0])[0][0] == 0.0


def test_sine_and_cosine(evaluate):
    rng = np.random.default_rng(0)
    th = np.concatenate([rng.uniform(0.0, 4.0, 200000), np.arange(1025) / 256, np.arange(2049) / 512])
    _, s, c = evaluate(th)
    ref = np.longdouble(2) * np.longdouble("3.14159265358979323846264338327950288") * th
    assert np.abs(s - np.sin(ref)).max() <= 6e-16 and np.abs(c - np.cos(ref)).max() <= 6e-16
