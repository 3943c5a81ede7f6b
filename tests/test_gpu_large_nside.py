"""Matrix-core dirty map at nside 2048, where a chunk's seeds span more than 32 bits
of bytes: rows that a 32-bit offset cannot reach are read through 64-bit addresses.
Samples over the whole sky and every segment, against float64 arithmetic on the
host, and the vector-unit kernel, within 1e-5 of S."""
import numpy as np
import pytest

import synth
from tests._cases import freqs, make_csd

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_seed_rows_beyond_32_bit_offsets():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    import paper_1803_08285_amd as sg

    nside, nt, nf, k0, f0, df = 2048, 18, 3, 62, 20.0, 1 / 32
    npix = 12 * nside * nside
    assert (nt - 1) * (npix // 2) * 16 > 2 ** 32  # the last amplitude row's offset
    g, t = sg.build_geometry(synth.baseline_sites("AB"), nside, sg.TGrid(nt, 0.0, 86164.0905 / nt, 86164.0905 / nt))
    C, w = make_csd(nt, nt, freqs(f0, df, k0, nf))
    Cd, wd, fg = torch.from_numpy(C).cuda(), torch.from_numpy(w).cuda(), sg.FGrid(f0, df)
    ws = torch.full((sg.workspace_bytes(nt, nf, npix, True),), 255, dtype=torch.uint8, device="cuda")
    X, _ = sg.make_maps(Cd, wd, fg, k0, g, t, want_gamma=False, workspace=ws)
    assert sg.last_x_form() == "mfma4"
    V, _ = sg.make_maps(Cd, wd, fg, k0, g, t, want_gamma=False, x_kernel="valu")
    rng = np.random.default_rng(1)
    pix = np.concatenate([[0, npix // 2 - 1, npix // 2, npix - 1], rng.integers(0, npix, 2000)])
    at = torch.from_numpy(pix).cuda()
    gh, th = g[:, at].double().cpu().numpy(), t[:, at].cpu().numpy()
    y = w.astype(np.float64) * C.astype(np.complex128)
    f = f0 + (k0 + np.arange(nf)) * df
    ref = np.stack([(gh * (y[:, c, None] * np.exp(2j * np.pi * f[c] * th)).real).sum(0) for c in range(nf)])
    S = np.stack([(np.abs(gh) * np.abs(y[:, c, None])).sum(0) for c in range(nf)])
    assert np.all(np.abs(X[:, at].double().cpu().numpy() - ref) <= 1e-5 * S)
    Sp = torch.from_numpy(np.abs(y)).float().cuda().t() @ g.abs()
    assert bool(((X - V).abs() <= 2e-5 * Sp).all())
