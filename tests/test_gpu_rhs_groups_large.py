"""GPU check of the streaming stencil's RHS groups where a launch forms them (from
2^19 sites on, a die's blocks spanning little more than an x1 plane): every RHS of
groups of three, of two and two and of three, three and one, against the oracle
with the stencil's tolerance of each type (tests/test_gpu_stencil.py); and the
weighted sum of a multishift solve, whose partial sums come from grouped launches,
by its RHS alone."""
import numpy as np
import pytest
import torch

import oracle
import synth
from parity import field_check, stencil_check

pytestmark = pytest.mark.gpu

M0 = -1.6
DIMS, DIMS32 = (16, 16, 64, 32), (32, 16, 64, 32)


@pytest.mark.parametrize("dims,prec,tol,nrhs", [(DIMS, 0, 1e-12, 7), (DIMS32, 1, 1e-6, 6), (DIMS32, 0, 1e-12, 4)])
def test_groups_match_oracle(dims, prec, tol, nrhs):
    import paper_1410_7170_amd as ovl
    print(f"rhs groups large dims={dims} nrhs={nrhs} prec={prec}", flush=True)
    lat, olat = ovl.Lattice(dims), oracle.Lattice(dims)
    assert lat.stream_t > 0 and lat.stream_t64 > 0 and lat.V >= 1 << 19
    U = synth.gauge(dims, 0.5, 171)
    G = ovl.Gauge(lat, torch.from_numpy(U).cuda(), (prec,))
    psi = synth.gaussian_spinor(lat.V, 172, nrhs)
    if prec == 1:
        psi = psi.astype(np.complex64).astype(np.complex128)
        U = U.astype(np.complex64).astype(np.complex128)
    inp = ovl.Spinor.from_canonical(lat, torch.from_numpy(np.ascontiguousarray(psi)).cuda(), prec)
    out = ovl.Spinor(lat, prec, nrhs)
    ovl.wilson_apply(lat, G, M0, inp, out)
    got = out.to_canonical().cpu().numpy()
    for r in range(nrhs):
        ratio, r2 = stencil_check(got[r], oracle.dw(olat, U, M0, psi[r]), psi[r], dims, M0, tol)
        assert ratio <= 1.0, (r, ratio, r2)


def test_grouped_solve_matches_single_rhs():
    import paper_1410_7170_amd as ovl
    nrhs = 5
    print(f"rhs groups large solve nrhs={nrhs}", flush=True)
    lat = ovl.Lattice(DIMS)
    G = ovl.Gauge(lat, torch.from_numpy(synth.gauge(DIMS, 0.3, 173, n_stout=1)).cuda(), (ovl.F64, ovl.F32))
    b = torch.from_numpy(synth.gaussian_spinor(lat.V, 174, nrhs)).cuda()
    s, w = np.array([0.3, 1.0, 4.0, 12.0]), np.array([0.4, 0.3, 0.2, 0.5])
    prm = ovl.default_params(tol=1e-10)
    Y = ovl.Spinor(lat, ovl.F64, nrhs)
    ovl.multishift_cg(lat, G, M0, s, w, ovl.Spinor.from_canonical(lat, b, ovl.F64), Y, prm)
    got = Y.to_canonical().cpu().numpy()
    one = ovl.Spinor(lat, ovl.F64, 1)
    for r in (0, nrhs - 1):
        ovl.multishift_cg(lat, G, M0, s, w, ovl.Spinor.from_canonical(lat, b[r:r + 1].contiguous(), ovl.F64), one, prm)
        # the same iterates: rounding of up to about 100 steps
        ratio, r2 = field_check(got[r], one.to_canonical().cpu().numpy()[0], DIMS, 1e-11)
        assert ratio <= 1.0, (r, ratio, r2)
