"""How projections of pseudo queries are cut into waves (csrc/qproj_plan.h, compiled here for the host): every plan there is has a kernel
that adds up its planes, and its waves cover the hidden axis."""
import os
import subprocess

import pytest

from paper_2603_11564_amd import build
from qproj_shapes import SPLIT_SHAPES

PROGRAM = r"""
#include <cstdio>
#include <initializer_list>
#include "qproj_plan.h"
using namespace dapq;

static dapq_qproj describe(int layers, int heads, int d, int rows, int hidden) {
  dapq_qproj s = {};
  s.n_layers = layers, s.n_q_heads = heads, s.head_dim = d, s.rows = rows, s.hidden = hidden;
  return s;
}

int main(int argc, char**) {
  if (argc > 1) {  // the plans of the shapes on standard input
    int l, h, d, r, k;
    while (scanf("%d %d %d %d %d", &l, &h, &d, &r, &k) == 5) {
      const QprojPlan p = make_qproj_plan(describe(l, h, d, r, k));
      printf("%d %d\n", p.waves, p.k_splits);
    }
    return 0;
  }
  long split = 0, wrong = 0;
  for (int rows : {0, 1, 16, 32, 33, 64, 65, 128, 129, 148, 200, 256, 300})
    for (int blocks = 1; blocks <= 300; ++blocks)
      for (int tiles = 1; tiles <= 800; ++tiles) {
        const QprojPlan p = make_qproj_plan(describe(1, tiles, 64, rows, blocks * kBlockK));
        if (rows == 0) continue;  // (nothing is launched)
        const long covered = (long)p.k_splits * p.waves * p.kb_per_split;
        const size_t plane = (size_t)p.sweeps * 32 * p.mb * p.tiles_f * 32 * p.ft * sizeof(float);
        bool ok = covered >= blocks;
        if (p.workspace_bytes > 0) ok = ok && qproj_planes_have_a_kernel(p.k_splits) && p.ft == 2 && p.k_splits * plane <= p.workspace_bytes;
        else ok = ok && p.k_splits == 1 && p.waves == 1;
        split += p.workspace_bytes > 0;
        if (!ok && wrong++ < 5) printf("rows %d, %d blocks, %d tiles: waves %d, planes %d\n", rows, blocks, tiles, p.waves, p.k_splits);
      }
  printf("%ld split, %ld wrong\n", split, wrong);
  return 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    folder = tmp_path_factory.mktemp("qproj_plan")
    (folder / "plan.cc").write_text(PROGRAM)
    out = str(folder / "plan")
    r = subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC,
                        str(folder / "plan.cc"), "-o", out], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    return out


def test_every_plan_has_its_kernels(program):
    """All numbers of 64-feature tiles that are split, over hidden axes of up to 19200 channels."""
    report = subprocess.run([program], capture_output=True, text=True, check=True, timeout=120).stdout
    split, wrong = (int(part.split()[0]) for part in report.splitlines()[-1].split(","))
    assert split > 1000000 and wrong == 0, report


def test_the_shapes_of_the_gpu_tests_get_the_plans_they_stand_for(program):
    lines = "".join("%d %d %d %d %d\n" % shape for shape in SPLIT_SHAPES)
    out = subprocess.run([program, "-"], input=lines, capture_output=True, text=True, check=True, timeout=60).stdout
    got = dict(zip(SPLIT_SHAPES, (tuple(map(int, line.split())) for line in out.splitlines())))
    assert got == SPLIT_SHAPES
    assert {planes for waves, planes in got.values() if waves == 4} == set(range(1, 9))
