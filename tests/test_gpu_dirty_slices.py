"""Vector-unit dirty map at the edges of its work split (64 columns and one strip
a workgroup, the segments in eight slices): days shorter than the slices, slices
that end inside a stage, ragged columns and strips; X within 1e-5 of S (float64
path 1e-12), Xbb within one rounding of the band sum of the call's own X, rows of
a sub-band bitwise those of the whole band, the batched plan bitwise the call."""
import numpy as np
import pytest

import synth
from tests._cases import freqs, make_csd, x_error

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

F0, DF = 20.0, 0.25


@pytest.mark.parametrize("f64", [False, True], ids=["f32", "f64"])
@pytest.mark.parametrize("nside,nt,k0,nf,anti", [
    (1, 1, 0, 1, True),        # one segment, one bin, six pairs
    (2, 7, 63, 66, True),      # fewer segments than slices; a strip's last bin, one whole, one bin
    (4, 67, 5, 200, True),     # slices of nine; 96 columns
    (4, 130, 31, 97, False),   # no pairing, 192 columns
    (8, 65, 32, 64, True),     # slices of nine, the last of two
])
def test_slices_vs_oracle(oracle_mod, nside, nt, k0, nf, anti, f64):
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    import paper_1803_08285_amd as sg

    dt = torch.float64 if f64 else torch.float32
    g, t = sg.build_geometry(synth.baseline_sites("AC"), nside, sg.TGrid(nt, 0.0, 86164.0905 / nt, 86164.0905 / nt),
                             dtype=dt)
    f = freqs(F0, DF, k0, nf)
    C, w = make_csd(50 + nt, nt, f, dtype=np.complex128 if f64 else np.complex64)
    Cd, wd, fg = torch.from_numpy(C).cuda(), torch.from_numpy(w).cuda(), sg.FGrid(F0, DF)
    X, _ = sg.make_maps(Cd, wd, fg, k0, g, t, antipodal=anti, want_gamma=False)
    Xo, _, S = oracle_mod.maps(C, w, F0, DF, k0, g.cpu().numpy(), t.cpu().numpy(), with_scale=True)
    torch.cuda.synchronize()
    assert x_error(X.cpu().numpy(), Xo, S) <= (1e-12 if f64 else 1e-5)
    lo = nf // 3
    Xs, _ = sg.make_maps(Cd[:, lo:], wd[:, lo:], fg, k0 + lo, g, t, antipodal=anti, want_gamma=False)
    assert torch.equal(Xs, X[lo:])
    if f64:
        return
    Xb, _, Xbb, _ = sg.make_maps_band(Cd, wd, fg, k0, g, t, None, lo, nf, antipodal=anti, want_gamma=False)
    assert torch.equal(Xb, X)
    Xh = X.double().cpu().numpy()[lo:]
    assert np.all(np.abs(Xbb.cpu().numpy() - Xh.sum(axis=0)) <=
                  2.0 ** -24 * np.abs(Xh.sum(axis=0)) + 1e-12 * np.abs(Xh).sum(axis=0) + 1e-300)
    out = [torch.empty_like(X), torch.empty_like(Xbb)]
    plan = sg.Plan([sg.Job(Cd, wd, fg, k0, g, t, X=out[0], band=(lo, nf), Xbb=out[1], antipodal=anti)],
                   autotune=False)
    for _ in range(2):
        plan.launch()
        torch.cuda.synchronize()
        assert torch.equal(out[0], X) and torch.equal(out[1], Xbb)
    plan.close()
