"""GPU check of the FP64 multishift CG where Q has an exact kernel: unit links,
periodic in every direction, m0 = 0, so that Q maps constant spinors to zero
exactly.  (Q^2 + s) x = b is as well posed as ever for s > 0, and for a
constant b its solution is b / s; every form has to solve it, alone and beside
a source that is not in the kernel.  Residuals are recomputed by the oracle."""
import numpy as np
import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu

DIMS, BC, TOL = (4, 4, 4, 4), (1, 1, 1, 1), 1e-10
SHIFTS = np.array([0.05, 0.3, 1.0, 2.0, 6.0])
WEIGHTS = np.array([0.4, 0.3, 0.2, 0.5, 1.0])


@pytest.mark.parametrize("block", [0, 1, 8])
@pytest.mark.parametrize("form", ["solutions", "sum", "verified sum"])
@pytest.mark.parametrize("sources", [1, 2])
def test_source_in_the_kernel(block, form, sources):
    import paper_1410_7170_amd as ovl
    print(f"singular Q block={block} form={form} sources={sources}", flush=True)
    lat, olat = ovl.Lattice(DIMS, BC), oracle.Lattice(DIMS, BC)
    U = np.zeros((lat.V, 4, 3, 3), complex)
    U[...] = np.eye(3)
    G = ovl.Gauge(lat, torch.from_numpy(U).cuda())
    b = np.ones((sources, lat.V, 4, 3), complex)
    b[1:] = synth.gaussian_spinor(lat.V, 131, 1)
    assert not np.any(oracle.q(olat, U, 0.0, b[0]))
    B = ovl.Spinor.from_canonical(lat, torch.from_numpy(b).cuda(), ovl.F64)
    n = len(SHIFTS)
    X = ovl.Spinor(lat, ovl.F64, sources * (n if form == "solutions" else 1))
    prm = ovl.default_params(tol=TOL, block=block, verify=int(form == "verified sum"))
    st = ovl.multishift_cg(lat, G, 0.0, SHIFTS, None if form == "solutions" else WEIGHTS, B, X, prm)
    x = X.to_canonical().cpu().numpy()
    if form == "solutions":
        for j, s in enumerate(SHIFTS):
            # the base shift's own CG step is exact; a few roundings of b / s
            assert np.abs(x[j * sources] - b[0] / s).max() <= 1e-14 / s, (j, s)
            for r in range(sources):
                d = b[r] - oracle.q2(olat, U, 0.0, x[j * sources + r], s)
                assert np.linalg.norm(d) <= 1.01 * TOL * np.linalg.norm(b[r]), (j, r)
    else:
        want = (WEIGHTS / SHIFTS).sum()
        assert np.abs(x[0] - want).max() <= 1e-14 * want
    if form == "verified sum":
        assert max(st["true_residual"][0][:n]) <= 1.01 * TOL
    assert st["iterations"][0] <= 2
