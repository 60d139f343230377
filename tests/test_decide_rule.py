"""The rule for the decide kernel's workgroups (CPU only): what is added to the
one counter is bounded also where few sessions are taken but bins are many."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = """
#include <stdio.h>
#include "rc_plan.h"
int main() {
    unsigned units, thr;
    while (scanf("%u %u", &units, &thr) == 2) printf("%d\\n", (int)rc_plan::decide_few(units, thr));
}
"""


def test_decide_few(tmp_path):
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("g++ is not available")
    src, exe = str(tmp_path / "rule.cpp"), str(tmp_path / "rule")
    with open(src, "w") as f:
        f.write(SOURCE)
    subprocess.run([gxx, "-std=c++17", "-Wall", "-Werror", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_2608_12123_amd", "csrc"), "-o", exe, src], check=True)
    cases = [(u, t) for u in (1, 3, 4, 256, 391, 1041, 1045, 3907, 65_537, 1 << 23) for t in (0, 1, 16, 62, 63, 64, 65536)]
    out = subprocess.run([exe], input="".join("%d %d\n" % c for c in cases), capture_output=True, text=True,
                         check=True).stdout.split()
    for (units, thr), few in zip(cases, out):
        # a bin adds if one of its 256 sessions is taken
        adds = units * (1.0 - (1.0 - thr / 65536.0) ** 256)
        if few == "0":
            assert adds <= 256 and thr < 64, (units, thr)
        else:
            assert thr >= 64 or adds > 0.85 * 256, (units, thr)
    assert len(out) == len(cases)
