"""GPU parity of the multishift CG on the stencil forms that its modes take on
lattices between the small ones and the streaming ones (tests/test_tile_plan.py
pins the rule): tiles whose threads all hold a site and that carry the scalar
stages (8x8x32x64), with threads without one (18x18x18x24, one field), tiles that
do not carry (20x22x26x30, one field), the one-site form on several fields of such
a lattice, and the one-site form in blocks of 256 with carried stages
(14x14x14x18: 194 blocks).  Where there are three right-hand sides they differ in
convergence and one is zero; the residual of every x_j is recomputed by the
oracle, and the weighted sums, FP64 and mixed, are compared with the sum of those
x_j."""
import numpy as np
import pytest
import torch

import oracle
import synth
from parity import field_check

pytestmark = pytest.mark.gpu

M0, TOL = -1.6, 1e-9
LATTICES = [((8, 8, 32, 64), 3), ((18, 18, 18, 24), 1), ((20, 22, 26, 30), 1), ((18, 18, 18, 24), 3),
            ((14, 14, 14, 18), 3)]


@pytest.fixture(scope="module", params=LATTICES, ids=lambda c: "x".join(map(str, c[0])) + f"_{c[1]}")
def case(request):
    import paper_1410_7170_amd as ovl
    dims, nrhs = request.param
    print(f"solve forms dims={dims} nrhs={nrhs}", flush=True)
    lat, olat = ovl.Lattice(dims), oracle.Lattice(dims)
    assert lat.stream_t == 0 and lat.stream_t64 == 0   # neither streams
    assert (lat.V >= 131072) == (dims != (14, 14, 14, 18))   # tiles from 131072 sites on
    U = synth.gauge(dims, 0.3, 141, n_stout=2)
    G = ovl.Gauge(lat, torch.from_numpy(U).cuda())
    b = synth.gaussian_spinor(lat.V, 142, 3)
    for _ in range(3):   # less of the low modes: converges sooner
        b[1] = oracle.q2(olat, U, M0, b[1], 0.0)
    b[2] = 0
    b = b[:nrhs]
    B = ovl.Spinor.from_canonical(lat, torch.from_numpy(np.ascontiguousarray(b)).cuda(), ovl.F64)
    return ovl, lat, olat, U, G, b, B


# a positive smallest shift (extra unshifted base), one that is zero (the base
# itself), and as many as there can be (a shifted base: p0 is kept)
@pytest.mark.parametrize("first,nshift,block", [(0.05, 5, 0), (0.05, 5, 8), (0.0, 5, 8), (0.05, 32, 16)])
def test_solutions_and_sums(case, first, nshift, block):
    ovl, lat, olat, U, G, b, B = case
    print(f"  smallest shift {first}, {nshift} shifts, block {block}", flush=True)
    s = np.geomspace(0.05, 30.0, nshift)
    s[0] = first
    w = np.linspace(1.0, 0.3, nshift)
    nrhs = len(b)
    live = min(nrhs, 2)
    X = ovl.Spinor(lat, ovl.F64, nrhs * nshift)
    st = ovl.multishift_cg(lat, G, M0, s, None, B, X, ovl.default_params(tol=TOL, block=block))
    if nrhs == 3:
        assert st["iterations"][0] > st["iterations"][1] > 0 and st["iterations"][2] == 0
    x = X.to_canonical().cpu().numpy().reshape(nshift, nrhs, lat.V, 4, 3)
    del X
    assert not np.any(x[:, live:])
    for r in range(live):
        for j in range(nshift):
            d = b[r] - oracle.q2(olat, U, M0, x[j, r], s[j])
            assert np.linalg.norm(d) <= 1.01 * TOL * np.linalg.norm(b[r]), (r, j)
    want = np.tensordot(w, x, 1)
    del x
    Y = ovl.Spinor(lat, ovl.F64, nrhs)
    ovl.multishift_cg(lat, G, M0, s, w, B, Y, ovl.default_params(tol=TOL, block=block))
    y = Y.to_canonical().cpu().numpy()
    assert not np.any(y[live:])
    for r in range(live):
        # the same iterates: up to about 200 steps of 1e-16, times the 1e2 by
        # which (Q^2 + s)^-1 spreads it
        ratio, r2 = field_check(y[r], want[r], lat.dims, 1e-11)
        assert ratio <= 1.0, (r, ratio, r2)
    if first > 0.0:
        ovl.multishift_cg(lat, G, M0, s, w, B, Y, ovl.default_params(tol=TOL, mode=ovl.SOLVE_MIXED))
        y = Y.to_canonical().cpu().numpy()
        assert not np.any(y[live:])
        for r in range(live):
            # both within residuals of tol |b|: 2 tol |b| sum_j w_j / s_j
            assert np.linalg.norm(y[r] - want[r]) <= 2 * TOL * np.linalg.norm(b[r]) * (w / s).sum(), r
