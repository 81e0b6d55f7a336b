"""GPU check of the streaming stencil's RHS groups (blocks of at most three
RHS side by side): every RHS of a launch of 4 to 12, with and without RHS
tiles and ragged last groups, against the oracle with the stencil's tolerance
of each type (tests/test_gpu_stencil.py)."""
import numpy as np
import pytest
import torch

import oracle
import synth
from parity import stencil_check

pytestmark = pytest.mark.gpu

M0 = -1.6


@pytest.mark.parametrize("prec,tol", [(0, 1e-12), (1, 1e-6)])
@pytest.mark.parametrize("nrhs,tile", [(4, 1), (5, 1), (7, 1), (12, 1), (11, 2)])
def test_rhs_groups_match_oracle(nrhs, tile, prec, tol):
    import paper_1410_7170_amd as ovl
    dims = (8, 8, 8, 8)
    print(f"rhs groups nrhs={nrhs} tile={tile} prec={prec}", flush=True)
    lat, olat = ovl.Lattice(dims), oracle.Lattice(dims)
    lat.stream_t = lat.stream_t64 = 4
    lat.rhs_tile = tile
    U = synth.gauge(dims, 0.5, 61)
    G = ovl.Gauge(lat, torch.from_numpy(U).cuda(), (prec,))
    psi = synth.gaussian_spinor(lat.V, 62, nrhs)
    if prec == 1:
        psi = psi.astype(np.complex64).astype(np.complex128)
        U = U.astype(np.complex64).astype(np.complex128)
    inp = ovl.Spinor.from_canonical(lat, torch.from_numpy(np.ascontiguousarray(psi)).cuda(), prec)
    out = ovl.Spinor(lat, prec, nrhs)
    ovl.wilson_apply(lat, G, M0, inp, out)
    got = out.to_canonical().cpu().numpy()
    for r in range(nrhs):
        ratio, r2 = stencil_check(got[r], oracle.dw(olat, U, M0, psi[r]), psi[r], dims, M0, tol)
        assert ratio <= 1.0, (nrhs, tile, prec, r, ratio, r2)
