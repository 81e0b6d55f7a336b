"""GPU parity of the Wilson stencil's tile form (FP64 and 48-bit fields on
lattices of 131072 sites and more whose default is not the streaming form)
against the FP64 oracle, element by element, with the tolerances of the other
forms: 1e-12 M_x in FP64, 1e-11 M_x on 48-bit fields (tests/parity.py)."""
import numpy as np
import pytest
import torch

import oracle
import synth
from parity import r48, stencil_check

pytestmark = pytest.mark.gpu

M0 = -1.6
TOL = {0: 1e-12, 3: 1e-11}

# 512-site tiles of whole x3 rows; rows cut in two; a direction of extent 2
# inside every tile with odd rows of 23; threads without a site
LATTICES = [((32, 16, 16, 16), 1), ((8, 8, 32, 64), 2), ((34, 2, 44, 46), 2), ((18, 18, 18, 24), 3)]


@pytest.mark.parametrize("prec", [0, 3])
@pytest.mark.parametrize("dims,nrhs", LATTICES)
def test_tile_form_matches_oracle(dims, nrhs, prec):
    import paper_1410_7170_amd as ovl
    print(f"tile form dims={dims} nrhs={nrhs} prec={prec}", flush=True)
    bc = (-1, 1, -1, 1)
    lat, olat = ovl.Lattice(dims, bc), oracle.Lattice(dims, bc)
    assert lat.stream_t64 == 0 and lat.V >= 131072
    U = synth.gauge(dims, 0.5, 41)
    G = ovl.Gauge(lat, torch.from_numpy(U).cuda(), (ovl.F64,))
    psi = synth.gaussian_spinor(lat.V, 42, nrhs)
    if prec == 3:
        psi = r48(psi)
    inp = ovl.Spinor.from_canonical(lat, torch.from_numpy(np.ascontiguousarray(psi)).cuda(), prec)
    out = ovl.Spinor(lat, prec, nrhs)
    ovl.wilson_apply(lat, G, M0, inp, out)
    got = out.to_canonical().cpu().numpy()
    for r in range(nrhs):
        ratio, r2 = stencil_check(got[r], oracle.dw(olat, U, M0, psi[r]), psi[r], dims, M0, TOL[prec])
        assert ratio <= 1.0, (dims, prec, r, ratio, r2)
    ovl.q2_apply(lat, G, M0, 0.31, inp, out)
    got = out.to_canonical().cpu().numpy()
    for r in range(nrhs):
        ratio, r2 = stencil_check(got[r], oracle.q2(olat, U, M0, psi[r], 0.31), psi[r], dims, M0, TOL[prec], 0.31)
        assert ratio <= 1.0, (dims, prec, r, ratio, r2)
