"""The routes of the FP64 multishift CG against each other: shifted solutions
from the blocked form (on an extra unshifted base while one more system fits)
against the plain form's, and the weighted sum of params.block = 0 (blocked
from 4 shifts on) against the plain form that params.verify asks for.  The
iterates are the same, so the results differ by rounding: up to about 200
steps of 1e-16, times the 1e2 by which (Q^2 + s)^-1 spreads it."""
import numpy as np
import pytest
import torch

import synth
from parity import field_check

pytestmark = pytest.mark.gpu

M0 = -1.6
TOL = 1e-11


def inputs(ovl, dims, nrhs):
    lat = ovl.Lattice(dims)
    G = ovl.Gauge(lat, torch.from_numpy(synth.gauge(dims, 0.3, 91, n_stout=2)).cuda())
    b = synth.gaussian_spinor(lat.V, 92, nrhs)
    return lat, G, ovl.Spinor.from_canonical(lat, torch.from_numpy(b).cuda(), ovl.F64)


@pytest.mark.parametrize("nshift,block", [(1, 8), (5, 1), (12, 5), (31, 16), (32, 32)])
def test_blocked_solutions_match_plain(nshift, block):
    import paper_1410_7170_amd as ovl
    dims, nrhs = (6, 4, 8, 6), 2
    print(f"blocked solutions nshift={nshift} block={block}", flush=True)
    lat, G, B = inputs(ovl, dims, nrhs)
    s = np.geomspace(0.02, 30.0, nshift)
    got = {}
    for m in (0, block):
        X = ovl.Spinor(lat, ovl.F64, nshift * nrhs)
        st = ovl.multishift_cg(lat, G, M0, s, None, B, X, ovl.default_params(tol=1e-11, block=m))
        got[m] = X.to_canonical().cpu().numpy(), st
    (x0, st0), (x1, st1) = got[0], got[block]
    for f in range(nshift * nrhs):
        ratio, r2 = field_check(x1[f], x0[f], dims, TOL)
        assert ratio <= 1.0, (f, ratio, r2)
    assert st1["iterations"] == st0["iterations"] and st1["shift_iters"] == st0["shift_iters"]


@pytest.mark.parametrize("npoles", [3, 4, 20, 32])
def test_default_sum_matches_plain(npoles):
    import paper_1410_7170_amd as ovl
    dims, nrhs = (6, 4, 8, 6), 3
    print(f"default sum npoles={npoles}", flush=True)
    lat, G, B = inputs(ovl, dims, nrhs)
    s, w, _ = ovl.zolotarev(0.36, 6.75, npoles)
    got = []
    for verify in (0, 1):
        O = ovl.Spinor(lat, ovl.F64, nrhs)
        ovl.sign_q_apply(lat, G, M0, s, w, B, O, ovl.default_params(tol=1e-12, verify=verify))
        got.append(O.to_canonical().cpu().numpy())
    for r in range(nrhs):
        ratio, r2 = field_check(got[0][r], got[1][r], dims, TOL)
        assert ratio <= 1.0, (r, ratio, r2)
