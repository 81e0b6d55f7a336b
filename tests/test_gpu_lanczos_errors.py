"""GPU check that the Lanczos sign mode leaves nothing in flight when it ends
with an error: a link that is not a number makes the first check's coefficients
so, and the call returns OVL_ERR_NONFINITE with its stream idle (the caller may
reuse the links and the workspace at once).  With twelve open right-hand sides
on a small lattice the steps run furthest ahead of that check."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nrhs,maxiter", [(1, 20), (12, 64)])
def test_nonfinite_links_end_with_an_idle_stream(nrhs, maxiter):
    import paper_1410_7170_amd as ovl
    dims = (6, 6, 6, 10)
    print(f"lanczos nonfinite links nrhs={nrhs}", flush=True)
    lat = ovl.Lattice(dims)
    U = synth.gauge(dims, 0.3, 121)
    U[7, 2, 0, 1] = np.nan
    G = ovl.Gauge(lat, torch.from_numpy(U).cuda(), (ovl.F64,))
    B = ovl.Spinor.from_canonical(lat, torch.from_numpy(synth.gaussian_spinor(lat.V, 122, nrhs)).cuda(), ovl.F64)
    O = ovl.Spinor(lat, ovl.F64, nrhs)
    s, w, _ = ovl.zolotarev(0.4, 6.0, 12)
    prm = ovl.default_params(tol=1e-10, maxiter=maxiter, mode=ovl.SOLVE_LANCZOS)
    ws = ovl.workspace(lat, ovl.OP_MSCG, ovl.F64, nrhs, 12, prm)
    torch.cuda.synchronize()
    with pytest.raises(ovl.OvlError) as e:
        ovl.sign_q_apply(lat, G, -1.6, s, w, B, O, prm, ws)
    idle = torch.cuda.current_stream().query()
    assert e.value.status == ovl.ERR_NONFINITE and idle
