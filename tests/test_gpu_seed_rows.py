"""The matrix-core dirty map reads no seeds beyond the day: gamma and tau are the
first rows of larger tensors whose later rows are NaN, and the workspace is filled
with NaN patterns before the call.  At days that end inside a chunk of 16 segments
(one to fifteen left over) and days shorter than a chunk, for every form, X is
finite, the bits of a call on seeds and a workspace of their own, and within 1e-5
of S of the oracle.  The row arithmetic itself runs on the CPU for every day of up
to 1200 segments."""
import numpy as np
import pytest

import synth
from tests._cases import freqs, make_csd, x_error
from tests.test_host_policy_cpu import _build_and_run

torch = pytest.importorskip("torch")

F0, K0, NF, NSIDE = 20.0, 37, 150, 8


def test_rows_on_the_cpu(tmp_path):
    assert "all checks passed" in _build_and_run(tmp_path, "seed_rows_test")


def _inside_nan(a, rows=24):
    """a as the first rows of a larger tensor, NaN behind it."""
    big = torch.full((a.shape[0] + rows, a.shape[1]), float("nan"), dtype=a.dtype, device=a.device)
    big[:a.shape[0]] = a
    return big[:a.shape[0]]


def _dirty(nbytes):
    return torch.full((nbytes + (1 << 20),), 255, dtype=torch.uint8, device="cuda")


def _clean(nbytes):
    return torch.zeros(nbytes, dtype=torch.uint8, device="cuda")


@pytest.mark.gpu
@pytest.mark.parametrize("bl,df,f0,form", [("AB", 1 / 32, F0, "mfma4"), ("AC", 1 / 32, F0, "mfma5"),
                                           ("AD", 1 / 32, F0, "mfma5_split"), ("AB", 1 / 32, 6.3e6, "mfma4")],
                         ids=["mfma4", "mfma5", "mfma5_split", "beyond_fixed_point"])
@pytest.mark.parametrize("nt", [1, 2, 7, 8, 9, 15, 16, 17, 18, 25, 31, 33])
def test_no_seed_beyond_the_day(oracle_mod, nt, bl, df, f0, form):
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    import paper_1803_08285_amd as sg

    # a full day's grid, so that the first segments' delays reach the form's bound
    g, t = sg.build_geometry(synth.baseline_sites(bl), NSIDE, sg.TGrid(48, 0.0, 86164.0905 / 48, 86164.0905 / 48))
    g, t = g[:nt].clone(), t[:nt].clone()
    C, w = make_csd(60 + nt, nt, freqs(F0, df, K0, NF))
    Cd, wd, fg = torch.from_numpy(C).cuda(), torch.from_numpy(w).cuda(), sg.FGrid(f0, df)
    need = sg.workspace_bytes(nt, NF, 12 * NSIDE ** 2, True)
    ws = _dirty(need)
    X, _ = sg.make_maps(Cd, wd, fg, K0, _inside_nan(g), _inside_nan(t), want_gamma=False, workspace=ws)
    ran = sg.last_x_form()  # read from the workspace
    assert ran == form if nt >= 15 else ran.startswith("mfma")
    Xr, _ = sg.make_maps(Cd, wd, fg, K0, g, t, want_gamma=False, workspace=_clean(need))
    torch.cuda.synchronize()
    assert bool(torch.isfinite(X).all())
    assert torch.equal(X, Xr)
    Xo, _, S = oracle_mod.maps(C, w, f0, df, K0, g.cpu().numpy(), t.cpu().numpy(), with_scale=True)
    assert x_error(X.cpu().numpy(), Xo, S) <= 1e-5


@pytest.mark.gpu
@pytest.mark.parametrize("nt,stride", [(898, 86164.0905 / 898), (905, 86164.0905 / 905), (5, 96.0), (9, 96.0), (20, 96.0)])
def test_no_seed_beyond_the_day_overlap(oracle_mod, nt, stride):
    """The overlap terms (pairs' seeds in the workspace, 128-bin strips)."""
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    import paper_1803_08285_amd as sg

    g, t = sg.build_geometry(synth.baseline_sites("AB"), NSIDE, sg.TGrid(nt, 0.0, stride, 2 * stride))
    f = freqs(F0, 1 / 32, K0, NF)
    rng = np.random.default_rng(nt)
    v = (rng.uniform(0.5, 1.5, (nt, 1)) * (synth.spectrum_H(f) / synth.noise_psd(f) ** 2)).astype(np.float32)
    u, w = (a.astype(np.float32) for a in synth.overlap_series(v.astype(np.float64)))
    d = [torch.from_numpy(a).cuda() for a in (v, u, w)]
    fg, npix = sg.FGrid(F0, 1 / 32), 12 * NSIDE ** 2
    need = sg.fisher_overlap_workspace_bytes(nt, NF, npix)
    ws = _dirty(need)
    G = sg.fisher_overlap(*d, fg, K0, _inside_nan(g), _inside_nan(t), workspace=ws)
    assert sg.last_x_form() == "mfma4"
    Gr = sg.fisher_overlap(*d, fg, K0, g, t, workspace=_clean(need))
    torch.cuda.synchronize()
    assert bool(torch.isfinite(G).all())
    assert torch.equal(G, Gr)
    cols = np.repeat(np.arange(NF), 16)
    pix = rng.integers(0, npix, cols.size)
    Go, _, S = oracle_mod.fisher_overlap_at(v, u, w, F0, 1 / 32, K0, g.cpu().numpy(), t.cpu().numpy(), cols, pix)
    err = np.abs(G.cpu().numpy()[cols, pix].astype(np.float64) - Go) / S
    assert err.max() <= 1e-4
