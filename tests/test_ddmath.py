"""The double-double exponential of the factor generation (csrc/ddmath.h), compiled for the host: an entry is the
exact value rounded once, also where that lies close to the middle between two doubles."""
import os
import shutil
import subprocess

import mpmath
import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include")

SRC = r"""
#include "ddmath.h"
#include <cstdio>
int main() {
    double hi, lo;
    while (std::scanf("%la %la", &hi, &lo) == 2) {
        const double2 e = fio::dd_expi2pi(fio::dd{hi, lo});
        std::printf("%a %a\n", e.x, e.y);
    }
}
"""


@pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir(os.path.join(ROCM, "hip")),
                    reason="no host compiler or HIP headers")
def test_entries_near_a_tie_are_rounded_correctly(tmp_path):
    # Arguments whose cosine (or sine) lies 2^-95 of its value beside the middle between two doubles.  The
    # double-double operations err by at most 2^-104 each, a dozen of them reach the result undamped:
    # under 2^-100.  What a term of the series loses in double precision (2^-53 of the sixth: 2^-86) rounds
    # about half of these wrongly.
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(SRC)
    subprocess.run(["g++", "-std=c++17", "-O1", "-ffp-contract=off", "-w", "-D__HIP_PLATFORM_AMD__", "-I", ROCM,
                    "-I", os.path.join(ROOT, "paper_2609_11520_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    rng = np.random.default_rng(5)
    args, want = [], []
    with mpmath.workdps(60):
        turn = 2 * mpmath.pi
        for i in range(400):
            lo = float(rng.uniform(0.72, 0.99)) if i % 4 < 2 else float(rng.uniform(0.05, 0.7))
            up = float(np.nextafter(lo, 1.0))
            tie = (mpmath.mpf(lo) + mpmath.mpf(up)) / 2
            y = tie * (1 + mpmath.ldexp(1 if i & 1 else -1, -95))
            f = (mpmath.acos(y) if i % 4 < 2 else mpmath.asin(y)) / turn
            hi = float(f)
            a = (hi, float(f - hi))
            x = turn * (mpmath.mpf(a[0]) + mpmath.mpf(a[1]))      # the argument as passed
            v = mpmath.cos(x) if i % 4 < 2 else mpmath.sin(x)
            assert abs(v / tie - 1) > mpmath.ldexp(1, -98)
            args.append(a)
            want.append((i % 4 >= 2, up if v > tie else lo))
    text = "".join("%s %s\n" % (a.hex(), b.hex()) for a, b in args)
    out = subprocess.run([str(exe)], input=text, capture_output=True, text=True, check=True).stdout.split("\n")
    got = [[float.fromhex(t) for t in line.split()] for line in out[:len(args)]]
    bad = [i for i, (s, w) in enumerate(want) if got[i][int(s)] != w]
    assert not bad, "%d of %d" % (len(bad), len(args))
