"""GPU parity of the launches that take the stencil's tile form by the rule that
tests/test_tile_plan.py pins, on tiles with threads that hold no site: D_W, Q and
Q^2 + s against the oracle element by element with the tile form's tolerances
(tests/test_gpu_tile.py), and the Lanczos passes against the oracle's after the
same, odd number of steps (tests/test_gpu_lanczos_forms.py)."""
import numpy as np
import pytest
import torch

import oracle
import synth
from oracle import krylov
from parity import field_check, r48, stencil_check

pytestmark = pytest.mark.gpu

M0 = -1.6
TOL = {0: 1e-12, 3: 1e-11}

# share of threads with a site 0.56; 0.77, several fields; 0.94; 0.875 of 256
LATTICES = [((18, 18, 18, 24), 2, 0), ((64, 14, 14, 14), 3, 0), ((20, 22, 26, 30), 1, 3), ((10, 30, 26, 28), 1, 3)]


@pytest.mark.parametrize("dims,nrhs,prec", LATTICES)
def test_operators_on_partial_tiles(dims, nrhs, prec):
    import paper_1410_7170_amd as ovl
    print(f"tile rule dims={dims} nrhs={nrhs} prec={prec}", flush=True)
    bc = (-1, 1, -1, 1)
    lat, olat = ovl.Lattice(dims, bc), oracle.Lattice(dims, bc)
    assert lat.stream_t == 0 and lat.stream_t64 == 0 and lat.V >= 131072
    U = synth.gauge(dims, 0.5, 161)
    G = ovl.Gauge(lat, torch.from_numpy(U).cuda(), (ovl.F64,))
    psi = synth.gaussian_spinor(lat.V, 162, nrhs)
    if prec == 3:
        psi = r48(psi)
    inp = ovl.Spinor.from_canonical(lat, torch.from_numpy(np.ascontiguousarray(psi)).cuda(), prec)
    out = ovl.Spinor(lat, prec, nrhs)
    for apply, ref in ((ovl.wilson_apply, oracle.dw), (ovl.q_apply, oracle.q)):
        apply(lat, G, M0, inp, out)
        got = out.to_canonical().cpu().numpy()
        for r in range(nrhs):
            ratio, r2 = stencil_check(got[r], ref(olat, U, M0, psi[r]), psi[r], dims, M0, TOL[prec])
            assert ratio <= 1.0, (r, ratio, r2)
    ovl.q2_apply(lat, G, M0, 0.31, inp, out)
    got = out.to_canonical().cpu().numpy()
    for r in range(nrhs):
        ratio, r2 = stencil_check(got[r], oracle.q2(olat, U, M0, psi[r], 0.31), psi[r], dims, M0, TOL[prec], 0.31)
        assert ratio <= 1.0, (r, ratio, r2)


@pytest.mark.parametrize("dims,nrhs", [((18, 18, 18, 24), 1), ((8, 8, 32, 64), 2)])
def test_lanczos_on_tiles(dims, nrhs):
    import paper_1410_7170_amd as ovl
    print(f"tile rule lanczos dims={dims} nrhs={nrhs}", flush=True)
    steps = 35
    lat, olat = ovl.Lattice(dims), oracle.Lattice(dims)
    U = synth.gauge(dims, 0.3, 163)
    G = ovl.Gauge(lat, torch.from_numpy(U).cuda(), (ovl.F64,))
    b = synth.gaussian_spinor(lat.V, 164, nrhs)
    B = ovl.Spinor.from_canonical(lat, torch.from_numpy(np.ascontiguousarray(b)).cuda(), ovl.F64)
    O = ovl.Spinor(lat, ovl.F64, nrhs)
    s, w, _ = ovl.zolotarev(0.4, 6.0, 12)   # ignored by the Lanczos mode
    prm = ovl.default_params(tol=1e-13, maxiter=steps, mode=ovl.SOLVE_LANCZOS)
    st = ovl.sign_q_apply(lat, G, M0, s, w, B, O, prm, allow_not_converged=True)
    got = O.to_canonical().cpu().numpy()
    assert list(st["iterations"])[:nrhs] == [steps] * nrhs
    for r in range(nrhs):
        ref, n = krylov.lanczos_sign(lambda v: oracle.q(olat, U, M0, v), b[r], steps)
        ratio, r2 = field_check(got[r], ref, dims, 1e-9)
        assert n == steps and ratio <= 1.0, (r, ratio, r2)
