"""CPU check of the multishift CG's scalar stages: what a stage carried by a
stencil launch writes, the launch's site blocks do not read (a wave that sees a
flag change leaves before the others reach the barriers).  ``scalars.h`` is
compiled by g++ as one lane of a block (``host_scalar_stages.cpp``)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

# what scalars.h needs of device.h, for one lane: the others hold zeros
DEVICE = r"""
#pragma once
#include <cmath>
#define __device__
#define __global__
#define __forceinline__ inline
#define __shared__ static
struct Idx { unsigned x; };
static const Idx threadIdx{0};
inline double __shfl_xor(double, int, int) { return 0.0; }
inline void __syncthreads() {}
inline int __syncthreads_count(int v) { return v != 0; }
using std::fmax;
using std::isfinite;
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not on PATH")
def test_carried_stages_leave_their_launch_flags_alone(tmp_path):
    csrc = tmp_path / "a" / "csrc"
    csrc.mkdir(parents=True)
    shutil.copytree(os.path.join(ROOT, "include"), tmp_path / "include")
    shutil.copy(os.path.join(ROOT, "paper_1410_7170_amd", "csrc", "scalars.h"), csrc)
    (csrc / "device.h").write_text(DEVICE)
    exe = str(tmp_path / "stages")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wno-unknown-pragmas", "-I", str(tmp_path / "a"),
                           os.path.join(HERE, "host_scalar_stages.cpp"), "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stdout + r.stderr
