"""Even-odd Wilson solve on lattices of a few sites, where the vector kernels'
blocks outnumber those of a flat launch.  On the CPU: the partial sums reserved
for a kernel (``eo_plan.h``, compiled by g++) hold a sum of each of its blocks,
for every lattice size.  On the GPU: the residual recomputed by the oracle
meets the tolerance."""
import os
import shutil
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

MAIN = r"""
#include <cstdio>
#include "csrc/eo_plan.h"
int main()
{
    const int bs = 256;
    for (long Vh = 8; Vh <= 1 << 22; Vh += Vh < 70000 ? 1 : 977) {
        const ovl::EoPlan p = ovl::eo_plan((int)Vh, bs);
        const bool covers = (long)p.nh * bs >= Vh && 6 % p.parts == 0;
        // hops: nh sums; vector kernels: nh * parts; flat launches: 6 and 12 arrays
        if (!covers || p.slots < p.nh || p.slots < p.nh * p.parts || p.slots < ovl::eo_flat_blocks((int)Vh, 6, bs) ||
            p.slots < ovl::eo_flat_blocks((int)Vh, 12, bs)) {
            std::printf("FAIL Vh = %ld: %d slots\n", Vh, p.slots);
            return 1;
        }
    }
    std::printf("ok\n");
    return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not on PATH")
def test_partial_sums_fit_their_slots(tmp_path):
    (tmp_path / "main.cpp").write_text(MAIN)
    exe = str(tmp_path / "plan")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_1410_7170_amd"),
                           str(tmp_path / "main.cpp"), "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr


# 8, 16 and 40 even sites: below the 43 from which a flat launch has as many
# blocks; 48 above
@pytest.mark.gpu
@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (4, 2, 2, 2), (10, 2, 2, 2), (4, 6, 2, 2)])
def test_even_odd_solve_on_few_sites(dims):
    import torch

    import oracle
    import paper_1410_7170_amd as ovl
    import synth
    m0, tol = -0.2, 1e-11
    print(f"even-odd solve dims={dims}", flush=True)
    lat, olat = ovl.Lattice(dims), oracle.Lattice(dims)
    U = synth.gauge(dims, 0.5, 73)
    G = ovl.Gauge(lat, torch.from_numpy(U).cuda())
    b = synth.gaussian_spinor(lat.V, 74, 2)
    B = ovl.Spinor.from_canonical(lat, torch.from_numpy(np.ascontiguousarray(b)).cuda(), ovl.F64)
    X = ovl.Spinor(lat, ovl.F64, 2)
    ovl.wilson_solve(lat, G, m0, B, X, ovl.default_params(tol=tol, maxiter=500, even_odd=1))
    x = X.to_canonical().cpu().numpy()
    for r in range(2):
        res = np.linalg.norm(b[r] - oracle.dw(olat, U, m0, x[r])) / np.linalg.norm(b[r])
        # recomputed from the rounded x it may differ by FP64 rounding of D_W x
        assert res <= 1.01 * tol, (r, res)
