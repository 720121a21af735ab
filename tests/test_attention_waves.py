"""The waves per attention workgroup by the rows that the streams have (CPU: the
rule is host code).  The launch is as deep for every stream as for the longest
one; with uneven row caps most of its workgroups have no rows, and the rule must
not take them for work."""
import os
import subprocess

import pytest

HIPCC = "/opt/rocm/bin/hipcc"
MAIN = r"""
#include <cstdio>
#include <cstdlib>
#include "common.hpp"
// waves TUNED H N QTILES KNOWN ROWS...
int main(int argc, char** argv) {
  incvit::Shape sh = {};
  sh.H = atoi(argv[2]);
  sh.N = atoi(argv[3]);
  sh.Npad = incvit::round_up(sh.N, 32);
  int rows[incvit::kMaxViews], B = argc - 6, most = 0;
  for (int v = 0; v < B; ++v) most = std::max(most, rows[v] = atoi(argv[6 + v]));
  printf("%d\n", incvit::attn_waves_of(atoi(argv[1]), sh, B, atoi(argv[4]), most, atoi(argv[5]) ? rows : nullptr));
}
"""

CASES = [
    # tuned, H, N, query tiles, known, rows, waves
    # even: the workgroups are all at work
    (0, 16, 1024, 2, 1, [1024], 4),            # 512 workgroups: 4 waves still give 2048
    (0, 16, 256, 2, 1, [256] * 8, 2),          # 1024
    (0, 16, 256, 2, 1, [256] * 32, 1),         # 4096
    (0, 16, 256, 2, 1, [1], 4),
    (0, 4, 256, 1, 1, [256] * 31, 2),          # 1984: one workgroup-row short of one wave
    (0, 4, 256, 1, 1, [256] * 32, 1),          # 2048
    # uneven: few of the launched workgroups have rows
    (0, 16, 1024, 2, 1, [700, 300, 4, 4, 4, 4, 4, 4], 4),  # 608 of 2816
    (0, 16, 256, 2, 1, [256] + [1] * 7, 4),                # 240 of 1024
    (0, 16, 1024, 2, 1, [1024] + [1] * 7, 4),              # 624 of 4096
    (0, 16, 256, 2, 1, [256] + [0] * 7, 4),                # streams without a row
    # so many empty ones that starting them is the work
    (0, 16, 1024, 2, 1, [1024] + [1] * 31, 1),             # 1008 of 16384
    # the rows are not known, or the caller chose
    (0, 16, 1024, 2, 0, [1024] * 16, 8),
    (0, 16, 256, 2, 0, [256] * 32, 4),
    (8, 16, 256, 2, 1, [256] * 32, 8),
]


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
def test_attention_waves_by_the_workgroups_that_have_rows(tmp_path):
    from paper_2607_12287_amd import build as hip_build

    src, exe = str(tmp_path / "waves.hip"), str(tmp_path / "waves")
    with open(src, "w") as f:
        f.write(MAIN)
    subprocess.check_call([HIPCC, *hip_build.COMMON, "--cuda-host-only", src, "-o", exe])
    for tuned, H, N, qtiles, known, rows, waves in CASES:
        args = [str(x) for x in (tuned, H, N, qtiles, known, *rows)]
        got = int(subprocess.check_output([exe, *args], text=True))
        assert got == waves, (tuned, H, N, qtiles, known, rows)
