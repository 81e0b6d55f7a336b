"""GPU check of the one-site stencil's launches in blocks of one wave: D_W and
Gamma_5 D_W of every type against the oracle, and a multishift solve, whose
stages add up the partial sums, with its residuals recomputed by the oracle;
on lattices that leave threads without a site and on both sides of the 16384
sites up to which launches with partial sums take one wave a block."""
import numpy as np
import pytest
import torch

import oracle
import synth
from parity import stencil_check

pytestmark = pytest.mark.gpu

M0 = -1.6


@pytest.mark.parametrize("dims,nrhs", [((2, 2, 2, 2), 1), ((6, 4, 6, 10), 3), ((16, 16, 8, 8), 2), ((14, 14, 14, 6), 1)])
def test_wave_blocks_match_oracle(dims, nrhs):
    import paper_1410_7170_amd as ovl
    print(f"wave blocks dims={dims} nrhs={nrhs}", flush=True)
    lat, olat = ovl.Lattice(dims), oracle.Lattice(dims)
    assert lat.stream_t == 0 and lat.stream_t64 == 0
    U = synth.gauge(dims, 0.5, 91)
    G = ovl.Gauge(lat, torch.from_numpy(U).cuda())
    psi = synth.gaussian_spinor(lat.V, 92, nrhs)
    canon = torch.from_numpy(np.ascontiguousarray(psi)).cuda()
    for prec, tol in ((ovl.F64, 1e-12), (ovl.F32, 1e-6)):
        inp = ovl.Spinor.from_canonical(lat, canon, prec)
        out = ovl.Spinor(lat, prec, nrhs)
        for apply, ref in ((ovl.wilson_apply, oracle.dw), (ovl.q_apply, oracle.q)):
            apply(lat, G, M0, inp, out)
            got = out.to_canonical().cpu().numpy()
            for r in range(nrhs):
                ratio, r2 = stencil_check(got[r], ref(olat, U, M0, psi[r]), psi[r], dims, M0, tol)
                assert ratio <= 1.0, (prec, r, ratio, r2)
    shifts, tol = [0.02, 0.3, 2.0], 1e-9
    B = ovl.Spinor.from_canonical(lat, canon, ovl.F64)
    X = ovl.Spinor(lat, ovl.F64, nrhs * len(shifts))
    for block in (0, 1):
        ovl.multishift_cg(lat, G, M0, shifts, None, B, X, ovl.default_params(tol=tol, maxiter=2000, block=block))
        x = X.to_canonical().cpu().numpy().reshape(-1, lat.V, 4, 3)
        for r in range(nrhs):
            for j, s in enumerate(shifts):
                d = psi[r] - oracle.q2(olat, U, M0, x[j * nrhs + r], s)
                res = np.linalg.norm(d) / np.linalg.norm(psi[r])
                assert res <= 1.01 * tol, (block, r, j, res)
