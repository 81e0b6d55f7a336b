"""GPU parity of the plain FP64 overlap apply, which params.verify asks for
with block = 0 (every shifted vector updated in every iteration, their weighted
sum formed at the end), against the oracle at the FP64 path's 1e-12, with the
true residual of every shift; and the form that the benchmark calls plain."""
import numpy as np
import pytest
import torch

import oracle
import synth
from parity import field_check

RHO = 1.6


def test_benchmark_forms_take_their_routes():
    import bench
    import paper_1410_7170_amd as ovl
    plain = bench.params_for(ovl, "fp64_plain", 1e-10)
    # a weighted sum leaves the plain form only without verify (or with a block length)
    assert plain.mode == ovl.SOLVE_F64 and plain.block == 0 and plain.verify == 1
    assert bench.params_for(ovl, "fp64", 1e-10).verify == 0
    assert bench.params_for(ovl, "fp64_blocked", 1e-10).block > 0


@pytest.mark.gpu
@pytest.mark.parametrize("dims,nrhs", [((4, 4, 4, 4), 1), ((8, 4, 4, 6), 3)])
def test_plain_overlap_matches_oracle(dims, nrhs):
    import bench
    import paper_1410_7170_amd as ovl
    print(f"plain overlap dims={dims} nrhs={nrhs}", flush=True)
    lat, olat = ovl.Lattice(dims), oracle.Lattice(dims)
    U = synth.gauge(dims, 0.3, 31, n_stout=2)
    G = ovl.Gauge(lat, torch.from_numpy(U).cuda())
    b = synth.gaussian_spinor(lat.V, 32, nrhs)
    if nrhs > 2:
        b[2] = 0
    s, w, _ = oracle.zolotarev(*oracle.spectral_interval(olat, U, -RHO, synth.gaussian_spinor(lat.V, 99)[0], 300), 20)
    B = ovl.Spinor.from_canonical(lat, torch.from_numpy(np.ascontiguousarray(b)).cuda(), ovl.F64)
    O = ovl.Spinor(lat, ovl.F64, nrhs)
    st = ovl.overlap_apply(lat, G, RHO, s, w, B, O, bench.params_for(ovl, "fp64_plain", 1e-13))
    got = O.to_canonical().cpu().numpy()
    for r in range(nrhs):
        if not np.any(b[r]):
            assert not np.any(got[r])
            continue
        ref, _, _ = oracle.overlap(olat, U, RHO, s, w, b[r], 1e-13, 5000)
        ratio, r2 = field_check(got[r], ref, dims, 1e-12)
        worst = max(st["true_residual"][r][:20])
        print(f"  rhs {r}: worst/bound {ratio:.3g}, L2 {r2:.2e}, residual {worst:.2e}", flush=True)
        # recursive residuals reach 1e-13; the true ones stop at the rounding
        # of x, about 64 eps |Q|^2 / s ~ 1e-11 at worst
        assert ratio <= 1.0 and 0.0 < worst <= 1e-11
