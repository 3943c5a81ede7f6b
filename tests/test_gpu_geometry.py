"""Seed matrices at the edges of the geometry kernel's work split (two pixels a
lane, runs of segments): the smallest spheres, single segments, runs that do not
divide the day, outputs aligned to their element alone.  gamma meets the FP64
oracle within float32 rounding of gamma <= 2 (float64: 1e-14), tau within 1e-15 s,
and the seeds are exactly antipodally symmetric."""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("f64", [False, True], ids=["f32", "f64"])
@pytest.mark.parametrize("nside,nt", [(1, 1), (1, 130), (2, 65), (4, 700), (16, 67), (64, 33)])
def test_seeds_vs_oracle(oracle_mod, nside, nt, f64):
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    import paper_1803_08285_amd as sg

    npix, dt = 12 * nside * nside, torch.float64 if f64 else torch.float32
    sites = synth.baseline_sites("AC")
    # one element into a larger buffer: aligned to the element, not to a pair of them
    g = torch.empty(nt * npix + 1, dtype=dt, device="cuda")[1:].view(nt, npix)
    t = torch.empty(nt * npix + 1, dtype=torch.float64, device="cuda")[1:].view(nt, npix)
    stride = 86164.0905 / nt
    sg.build_geometry(sites, nside, sg.TGrid(nt, 11.0, stride, stride), dtype=dt, out=(g, t))
    torch.cuda.synchronize()
    go, to = oracle_mod.geometry(sites, nside, nt, 11.0, stride, stride)[:2]
    gh, th = g.cpu().numpy(), t.cpu().numpy()
    assert np.abs(gh - go).max() <= (1e-14 if f64 else 2.0 * 2.0 ** -24 + 1e-14)
    assert np.abs(th - to).max() <= 1e-15
    _, anti = sg.healpix_centres(nside)
    a = anti.long()
    assert torch.equal(g[:, a], g) and torch.equal(t[:, a], -t)
