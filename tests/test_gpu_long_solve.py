"""GPU check of multishift solves of about 2000 iterations (64x4^3 close to the
critical mass, smallest shift 1e-6), where the blocked form carries t = Q p by
recurrence from the first iteration to the last: its true residuals, recomputed
by the oracle, meet the tolerance as the plain form's do, which forms t anew in
every iteration.  Allowed above the tolerance is what the recursive residual
cannot see, the rounding of N updates: eps sqrt(N) |Q|^2 |x|, |Q| <= 8."""
import numpy as np
import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("block", [0, 1, 16])
def test_two_thousand_iterations(block):
    import paper_1410_7170_amd as ovl
    dims, m0, tol, shifts = (64, 4, 4, 4), -0.02, 1e-10, [1e-6, 0.1]
    print(f"long solve block={block}", flush=True)
    lat, olat = ovl.Lattice(dims), oracle.Lattice(dims)
    U = synth.gauge(dims, 0.3, 151, n_stout=2)
    b = synth.gaussian_spinor(lat.V, 152, 1)
    G = ovl.Gauge(lat, torch.from_numpy(U).cuda(), (ovl.F64,))
    B = ovl.Spinor.from_canonical(lat, torch.from_numpy(b).cuda(), ovl.F64)
    X = ovl.Spinor(lat, ovl.F64, 2)
    st = ovl.multishift_cg(lat, G, m0, shifts, None, B, X, ovl.default_params(tol=tol, maxiter=5000, block=block))
    x = X.to_canonical().cpu().numpy()
    n = st["iterations"][0]
    assert n > 1500
    for j, s in enumerate(shifts):
        res = np.linalg.norm(b[0] - oracle.q2(olat, U, m0, x[j], s)) / np.linalg.norm(b[0])
        unseen = 2.2e-16 * n ** 0.5 * 64 * np.linalg.norm(x[j]) / np.linalg.norm(b[0])
        print(f"  shift {s}: {n} iterations, residual {res:.4e}, unseen {unseen:.1e}", flush=True)
        assert res <= tol + unseen, (j, res, unseen)
