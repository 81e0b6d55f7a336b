"""GPU check of the one-pass link packing and of the unpacked spinor against
the layout itself, bit for bit: [parity][direction][component][site pair] with
rows 0 and 1 of each link, on lattices whose last block is not full."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


def even_odd(a, dims):
    """(V, ...) in lexicographic order -> (2, V/2, ...) by parity."""
    par = np.indices(dims).sum(0).reshape(-1) % 2
    return np.stack([a[par == 0], a[par == 1]])


@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (4, 2, 6, 10), (4, 4, 4, 4), (6, 6, 10, 14)])
def test_pack_copies_layout(dims):
    import paper_1410_7170_amd as ovl
    print(f"pack copies dims={dims}", flush=True)
    lat = ovl.Lattice(dims)
    U = synth.gauge(dims, 0.7, 81)
    canon = torch.from_numpy(U).cuda()
    rows = even_odd(U.reshape(lat.V, 4, 9)[:, :, :6], dims).transpose(0, 2, 3, 1)   # (2, 4, 6, V/2)
    per = {ovl.F64: (np.float64, 1), ovl.F32: (np.float32, 2), ovl.F16S: (np.float16, 2)}
    every = ovl.Gauge(lat, canon)
    for prec, (real, comps) in per.items():
        raw = every.bufs[prec].cpu().numpy().view(real)
        got = raw[: raw.size // (2 * 4 * 12) * (2 * 4 * 12)].reshape(2, 4, 6 // comps, -1, 2 * comps)[:, :, :, : lat.V // 2]
        ref = np.stack([rows.real, rows.imag], -1)                                   # (2, 4, 6, V/2, 2)
        ref = ref.astype(real)   # rounded once, to the nearest
        ref = ref.reshape(2, 4, 6 // comps, comps, lat.V // 2, 2).transpose(0, 1, 2, 4, 3, 5)
        assert np.array_equal(got, ref.reshape(2, 4, 6 // comps, lat.V // 2, 2 * comps)), prec
        alone = ovl.Gauge(lat, canon, (prec,)).bufs[prec].cpu().numpy().view(real)
        alone = alone[: raw.size // (2 * 4 * 12) * (2 * 4 * 12)].reshape(2, 4, 6 // comps, -1, 2 * comps)
        assert np.array_equal(alone[:, :, :, : lat.V // 2], got), prec
    psi = synth.gaussian_spinor(lat.V, 82, 3)
    back = ovl.Spinor.from_canonical(lat, torch.from_numpy(psi).cuda(), 0).to_canonical().cpu().numpy()
    assert np.array_equal(back, psi)
