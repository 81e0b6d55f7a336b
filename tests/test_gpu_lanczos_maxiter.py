"""GPU check that the Lanczos sign mode looks at its last step: a sequence cut
off by maxiter uses all of its maxiter steps, whatever maxiter's distance from
the regular checks (every 32 steps) and however many right-hand sides are open,
and one that converges between the last regular check and maxiter is reported
as converged.  The same number of steps by the oracle gives the same vector,
with the tolerance of tests/test_gpu_lanczos.py."""
import numpy as np
import pytest
import torch

import oracle
import synth
from oracle import krylov
from parity import field_check

pytestmark = pytest.mark.gpu

M0 = -1.6


def setup(dims, seed, nrhs, stout):
    import paper_1410_7170_amd as ovl
    lat, olat = ovl.Lattice(dims), oracle.Lattice(dims)
    U = synth.gauge(dims, 0.3, seed, n_stout=stout)
    b = synth.gaussian_spinor(lat.V, seed + 1, nrhs)
    G = ovl.Gauge(lat, torch.from_numpy(U).cuda(), (ovl.F64,))
    B = ovl.Spinor.from_canonical(lat, torch.from_numpy(np.ascontiguousarray(b)).cuda(), ovl.F64)
    s, w, _ = ovl.zolotarev(0.4, 6.0, 12)   # ignored by the Lanczos mode

    def sign(tol, maxiter):
        O = ovl.Spinor(lat, ovl.F64, nrhs)
        prm = ovl.default_params(tol=tol, maxiter=maxiter, mode=ovl.SOLVE_LANCZOS)
        st = ovl.sign_q_apply(lat, G, M0, s, w, B, O, prm, allow_not_converged=True)
        got = O.to_canonical().cpu().numpy()
        try:
            ovl.sign_q_apply(lat, G, M0, s, w, B, O, prm)
            converged = True
        except ovl.OvlError as e:
            assert e.status == ovl.NOT_CONVERGED
            converged = False
        return converged, list(st["iterations"])[:nrhs], got

    def check(got, steps):
        for r in range(nrhs):
            ref, n = krylov.lanczos_sign(lambda v: oracle.q(olat, U, M0, v), b[r], steps)
            ratio, r2 = field_check(got[r], ref, dims, 1e-9)
            assert n == steps and ratio <= 1.0, (r, steps, ratio, r2)

    return sign, check


@pytest.mark.parametrize("nrhs,steps", [(1, 31), (1, 33), (2, 34), (3, 35), (3, 64), (1, 66)])
def test_cut_off_sequence_uses_every_step(nrhs, steps):
    print(f"lanczos maxiter nrhs={nrhs} steps={steps}", flush=True)
    sign, check = setup((6, 6, 6, 10), 111, nrhs, 0)
    converged, iters, got = sign(1e-13, steps)
    assert not converged and iters == [steps] * nrhs
    check(got, steps)


def test_convergence_between_checks_is_seen():
    # the coefficients of steps 286 and 256 differ by 4.5e-11 |b|, those of 256
    # and 224 by 5.3e-10 |b|
    print("lanczos convergence at maxiter", flush=True)
    sign, check = setup((8, 4, 4, 8), 103, 1, 2)
    converged, iters, got = sign(1e-10, 286)
    assert converged and iters == [286]
    check(got, 286)
