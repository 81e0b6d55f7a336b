"""GPU parity of the Lanczos sign mode on every form of its stencil (one site
per thread, tiles, time streams) against the oracle's Lanczos approximation
after the same, odd number of steps: an unconverged sequence compares the
recurrence itself, and pass 2 ends on a single step.  The tolerance is the
same-steps one of tests/test_gpu_lanczos.py."""
import numpy as np
import pytest
import torch

import oracle
import synth
from oracle import krylov
from parity import field_check

pytestmark = pytest.mark.gpu

M0 = -1.6

# one-site form, its blocks partly without sites; tile form, extents not of
# the tile; streaming form
LATTICES = [((6, 6, 6, 10), 3), ((18, 18, 18, 24), 2), ((32, 16, 16, 32), 2)]


@pytest.mark.parametrize("dims,nrhs", LATTICES)
def test_lanczos_forms_match_oracle(dims, nrhs):
    import paper_1410_7170_amd as ovl
    print(f"lanczos forms dims={dims} nrhs={nrhs}", flush=True)
    steps = 35   # past one convergence check
    lat, olat = ovl.Lattice(dims), oracle.Lattice(dims)
    assert (lat.stream_t64 > 0) == (dims == (32, 16, 16, 32))
    U = synth.gauge(dims, 0.3, 51)
    G = ovl.Gauge(lat, torch.from_numpy(U).cuda(), (ovl.F64,))
    b = synth.gaussian_spinor(lat.V, 52, nrhs)
    b[nrhs - 1] = 0
    b[0] *= 1e5   # every RHS has its own scale
    B = ovl.Spinor.from_canonical(lat, torch.from_numpy(np.ascontiguousarray(b)).cuda(), 0)
    O = ovl.Spinor(lat, 0, nrhs)
    s, w, _ = ovl.zolotarev(0.4, 6.0, 12)   # ignored by the Lanczos mode
    prm = ovl.default_params(tol=1e-13, maxiter=steps, mode=ovl.SOLVE_LANCZOS)
    st = ovl.sign_q_apply(lat, G, M0, s, w, B, O, prm, allow_not_converged=True)
    got = O.to_canonical().cpu().numpy()
    assert list(st["iterations"]) == [steps] * (nrhs - 1) + [0]
    assert not np.any(got[nrhs - 1])
    for r in range(nrhs - 1):
        ref, n = krylov.lanczos_sign(lambda v: oracle.q(olat, U, M0, v), b[r], steps)
        ratio, r2 = field_check(got[r], ref, dims, 1e-9)
        print(f"  rhs {r}: worst/bound {ratio:.3g}, L2 {r2:.2e}", flush=True)
        assert n == steps and ratio <= 1.0
