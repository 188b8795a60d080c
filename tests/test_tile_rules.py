"""Which tile size a launch takes (fwd_small_tiles, bwd_small_tiles): the cases that the GPU tests run on both sides of the rules'
lines lie on the sides that these tests name.  CPU only."""
import os
import shutil
import subprocess

import pytest

from tests.test_gpu_forward_tiles import CASES as FORWARD
from tests.test_gpu_row_blocks import TILE_CASES as BACKWARD, tiles_and_columns

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2408_08490_amd", "csrc")
PROGRAM = """
#include "layer_host.h"
#include <cstdio>
int main() {
  int bwd, dtype, flag, width, tiles;   // flag: a ReLU; both products
  hgnn::BwdCols c;
  while (scanf("%d %d %d %d %d %d %d %d", &bwd, &dtype, &flag, &width, &tiles, &c.c128, &c.c64, &c.types) == 8)
    printf("%d\\n", (bwd ? hgnn::bwd_small_tiles(dtype, tiles, width, c, flag) : hgnn::fwd_small_tiles(dtype, width, flag, tiles)) ? 64 : 128);
}
"""


def test_cases_lie_on_the_sides_they_name(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    (tmp_path / "rules.cpp").write_text(PROGRAM)
    cmd = [gxx, "-std=c++20", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + CSRC, "-w", "-o", str(tmp_path / "rules"), str(tmp_path / "rules.cpp")]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    kind = {"f32": 0, "bf16": 1}
    asked, edges = [], []
    for dtype, relu, H, tiles, edge in FORWARD:
        asked.append((0, kind[dtype], int(relu), H, tiles, 0, 0, 0))
        edges.append(edge)
    for case in BACKWARD:
        tiles, (c128, c64, types) = tiles_and_columns(case)[1:]
        asked.append((1, kind[case[0]], int(len(case) == 6), case[2], tiles, c128, c64, types))
        edges.append(case[5])
    run = subprocess.run([str(tmp_path / "rules")], input="\n".join(" ".join(map(str, a)) for a in asked), capture_output=True, text=True)
    got = [int(v) for v in run.stdout.split()]
    assert len(got) == len(asked)
    assert [(a, e) for a, e, g in zip(asked, edges, got) if e != g] == []
