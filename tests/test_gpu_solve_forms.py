"""GPU parity of the multishift CG on the stencil forms that its modes take on
lattices between the small ones and the streaming ones: tiles whose launches
carry the scalar stages (18x18x18x24: 486 tiles of 288 sites in 512 threads),
tiles that do not (26x22x22x20: 1573 tiles of 160 sites in 256 threads) and the
one-site form in blocks of 256 with carried stages (14x14x14x18: 194 blocks).
Three right-hand sides of different convergence, one of them zero; the residual
of every x_j is recomputed by the oracle, and the weighted sums, FP64 and
mixed, are compared with the sum of those x_j."""
import numpy as np
import pytest
import torch

import oracle
import synth
from parity import field_check

pytestmark = pytest.mark.gpu

M0, TOL = -1.6, 1e-9
LATTICES = [(18, 18, 18, 24), (26, 22, 22, 20), (14, 14, 14, 18)]


@pytest.fixture(scope="module", params=LATTICES, ids=lambda d: "x".join(map(str, d)))
def case(request):
    import paper_1410_7170_amd as ovl
    dims = request.param
    print(f"solve forms dims={dims}", flush=True)
    lat, olat = ovl.Lattice(dims), oracle.Lattice(dims)
    assert lat.stream_t == 0 and lat.stream_t64 == 0   # neither streams
    assert (lat.V >= 131072) == (dims != (14, 14, 14, 18))   # tiles from 131072 sites on
    U = synth.gauge(dims, 0.3, 141, n_stout=2)
    G = ovl.Gauge(lat, torch.from_numpy(U).cuda())
    b = synth.gaussian_spinor(lat.V, 142, 3)
    for _ in range(3):   # less of the low modes: converges sooner
        b[1] = oracle.q2(olat, U, M0, b[1], 0.0)
    b[2] = 0
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
    X = ovl.Spinor(lat, ovl.F64, 3 * nshift)
    st = ovl.multishift_cg(lat, G, M0, s, None, B, X, ovl.default_params(tol=TOL, block=block))
    assert st["iterations"][0] > st["iterations"][1] > 0 and st["iterations"][2] == 0
    x = X.to_canonical().cpu().numpy().reshape(nshift, 3, lat.V, 4, 3)
    del X
    assert not np.any(x[:, 2])
    for r in range(2):
        for j in range(nshift):
            d = b[r] - oracle.q2(olat, U, M0, x[j, r], s[j])
            assert np.linalg.norm(d) <= 1.01 * TOL * np.linalg.norm(b[r]), (r, j)
    want = np.tensordot(w, x, 1)
    del x
    Y = ovl.Spinor(lat, ovl.F64, 3)
    ovl.multishift_cg(lat, G, M0, s, w, B, Y, ovl.default_params(tol=TOL, block=block))
    y = Y.to_canonical().cpu().numpy()
    assert not np.any(y[2])
    for r in range(2):
        # the same iterates: up to about 200 steps of 1e-16, times the 1e2 by
        # which (Q^2 + s)^-1 spreads it
        ratio, r2 = field_check(y[r], want[r], lat.dims, 1e-11)
        assert ratio <= 1.0, (r, ratio, r2)
    if first > 0.0:
        ovl.multishift_cg(lat, G, M0, s, w, B, Y, ovl.default_params(tol=TOL, mode=ovl.SOLVE_MIXED))
        y = Y.to_canonical().cpu().numpy()
        assert not np.any(y[2])
        for r in range(2):
            # both within residuals of tol |b|: 2 tol |b| sum_j w_j / s_j
            assert np.linalg.norm(y[r] - want[r]) <= 2 * TOL * np.linalg.norm(b[r]) * (w / s).sum(), r
