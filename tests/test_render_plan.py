"""The render's default launch plan (host arithmetic, compiled from its header):
a chunk's passes are split only while the chip has fewer than two workgroups per
CU (512), never into more parts than there are passes, and never where the split
parts would walk carries; with carries, a voice is split into its chunks or not at
all."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2104_12922_amd", "csrc")
BATCHES = (1, 2, 8, 127, 128, 129, 255, 256, 300, 511, 512, 513, 1000, 2047, 2048, 4096, 16384,
           100000, 536870912, 0x7FFFFFFF)
SAMPLES = (1, 100, 1600, 1601, 3200, 4410, 6200, 6201, 12400, 24800, 24801, 44100, 176400, 26460000)
MAIN = """
#include <stdio.h>
#include "render_plan.h"
int main() {
  long long b, n;
  int carried;
  while (scanf("%lld %lld %d", &b, &n, &carried) == 3) {
    const synth::RenderPlan p = synth::default_render_plan(44100.0, 441.0, b, n, carried != 0);
    printf("%d %d %d\\n", p.rps, p.slices, p.pass_split);
  }
}
"""


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("clang++")
    if not cxx:
        pytest.skip("needs a C++ compiler")
    d = tmp_path_factory.mktemp("plan")
    (d / "main.cpp").write_text(MAIN)
    subprocess.run([cxx, "-std=c++17", "-I", CSRC, str(d / "main.cpp"), "-o", str(d / "plan")], check=True)
    keys = [(b, n, c) for b in BATCHES for n in SAMPLES for c in (0, 1)]
    out = subprocess.run([str(d / "plan")], input="\n".join("%d %d %d" % k for k in keys), text=True,
                         capture_output=True, check=True).stdout.splitlines()
    return {k: tuple(map(int, line.split())) for k, line in zip(keys, out)}


def test_plans(plans):
    for (batch, n, carried), (rps, slices, split) in plans.items():
        J = -(-n // 100)
        chunks, passes = -(-J // 62), -(-J // 16)
        what = (batch, n, carried, slices, split)
        assert rps == 4 and 1 <= slices <= chunks and split in (1, 2, 4), what
        if carried:
            assert slices == (chunks if batch < 2048 else 1), what
        else:
            assert slices <= max(1, chunks // 4), what
        if split > 1:
            assert (split // 2) * batch * slices < 512 and split // 2 < passes, what
            assert carried and slices > 1 or chunks == 1, what
        assert batch * slices * split <= 0x7FFFFFFF, what


def test_batches_of_short_sounds_are_not_split(plans):
    for batch in BATCHES:
        for n in (100, 1600, 4410, 6200):
            if batch >= 512:
                assert plans[batch, n, 0] == (4, 1, 1), (batch, n)
    assert plans[8, 1600, 0][2] == 1 and plans[8, 1601, 0][2] == 2 and plans[8, 4410, 0][2] == 4
