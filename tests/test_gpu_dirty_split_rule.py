"""Vector-unit dirty map around its split rule: days are walked whole, or their
segments are split in four or eight slices, by the segments and the columns.  On
both sides of every line X is within 1e-5 of S (float64 path 1e-12), Xbb within
one rounding of the band sum of the call's own X, rows of a sub-band bitwise those
of the whole band, the batched plan bitwise the call; and a short day costs little
more than its write."""
import numpy as np
import pytest

import synth
from tests._cases import freqs, make_csd, x_error

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

F0, DF = 20.0, 0.25


@pytest.mark.parametrize("f64", [False, True], ids=["f32", "f64"])
@pytest.mark.parametrize("nside,nt,anti", [
    (8, 15, True), (8, 16, True),      # whole, eight
    (16, 31, True), (16, 33, True), (16, 59, True), (16, 60, True),  # whole, four, four, eight
    (16, 31, False), (16, 32, False), (16, 61, False),
    (32, 47, True), (32, 49, True), (32, 99, True), (32, 100, True),
    (32, 79, False), (32, 80, False), (32, 101, False),  # whole, four, four
    (64, 79, True), (64, 81, True), (64, 159, False), (64, 160, False),
])
def test_split_rule_edges(oracle_mod, nside, nt, anti, f64):
    """Both sides of every line of the split rule: sampled outputs against the
    oracle, rows of a sub-band and a plan's job bitwise the call's."""
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    import paper_1803_08285_amd as sg

    k0, nf, npix = 61, 70, 12 * nside * nside
    dt = torch.float64 if f64 else torch.float32
    g, t = sg.build_geometry(synth.baseline_sites("AC"), nside, sg.TGrid(nt, 0.0, 86164.0905 / nt, 86164.0905 / nt),
                             dtype=dt)
    C, w = make_csd(50 + nt, nt, freqs(F0, DF, k0, nf), dtype=np.complex128 if f64 else np.complex64)
    Cd, wd, fg = torch.from_numpy(C).cuda(), torch.from_numpy(w).cuda(), sg.FGrid(F0, DF)
    X, _ = sg.make_maps(Cd, wd, fg, k0, g, t, antipodal=anti, want_gamma=False)
    rng = np.random.default_rng(nt)
    pix = np.concatenate([[0, npix // 2 - 1, npix // 2, npix - 1], rng.integers(0, npix, 12)])
    cols, pp = np.repeat(np.arange(nf), pix.size), np.tile(pix, nf)
    Xo, _, S = oracle_mod.maps_at(C, w, F0, DF, k0, g.cpu().numpy(), t.cpu().numpy(), cols, pp)
    assert x_error(X.cpu().numpy()[cols, pp], Xo, S) <= (1e-12 if f64 else 1e-5)
    Xs, _ = sg.make_maps(Cd[:, 5:], wd[:, 5:], fg, k0 + 5, g, t, antipodal=anti, want_gamma=False)
    assert torch.equal(Xs, X[5:])
    if f64:
        return
    Xb, _, Xbb, _ = sg.make_maps_band(Cd, wd, fg, k0, g, t, None, 3, 67, antipodal=anti, want_gamma=False)
    assert torch.equal(Xb, X)
    Xh = X.double()[3:67]
    assert bool(((Xbb.double() - Xh.sum(0)).abs() <= 2.0 ** -24 * Xh.sum(0).abs() + 1e-12 * Xh.abs().sum(0)).all())
    out = [torch.empty_like(X), torch.empty_like(Xbb)]
    plan = sg.Plan([sg.Job(Cd, wd, fg, k0, g, t, X=out[0], band=(3, 67), Xbb=out[1], antipodal=anti),
                    sg.Job(Cd[:3], wd[:3], fg, k0, g[:3], t[:3], X=torch.empty_like(X), antipodal=anti)],
                   autotune=False)  # jobs of two counts of slices
    for _ in range(2):
        plan.launch()
        torch.cuda.synchronize()
        assert torch.equal(out[0], X) and torch.equal(out[1], Xbb)
    plan.close()


@pytest.mark.parametrize("anti", [True, False], ids=["pairs", "pixels"])
def test_a_short_day_is_bound_by_its_write(anti):
    """A map of one segment costs little more than writing it: less than three times a
    fill of the same bytes (1.4 and 1.3 measured; with the segments of every day in eight
    slices 5 and 7)."""
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    import paper_1803_08285_amd as sg

    nside, nf = 32, 6823
    g, t = sg.build_geometry(synth.baseline_sites("AB"), nside, sg.TGrid(1, 0.0, 86164.0, 86164.0))
    C, w = make_csd(3, 1, freqs(F0, DF, 0, nf))
    Cd, wd = torch.from_numpy(C).cuda(), torch.from_numpy(w).cuda()
    X = torch.empty((nf, 12 * nside * nside), device="cuda")

    def best(f):
        times = []
        for _ in range(12):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            f()
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b))
        return min(times)

    fill = best(lambda: X.fill_(0.0))
    call = best(lambda: sg.make_maps(Cd, wd, sg.FGrid(F0, DF), 0, g, t, antipodal=anti, want_gamma=False,
                                     out=(X, None)))
    print(f"fill {1e3 * fill:.0f} us, map {1e3 * call:.0f} us")
    assert call <= 3.0 * fill
