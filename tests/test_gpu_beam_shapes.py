"""Both wave-tile shapes of the beam GEMM give the same bits.

The 2x4 shape (default) shares the pixel-side fragments of a workgroup through
LDS; the 4x4 shape (picked by the plan autotuner, or SGWB_BEAM_SHAPE=4x4 for
single calls) reads both operands per wave.  Every output accumulates the
same products in the same order in both, so Gamma must be bitwise equal.  The
shape of single calls is read once per process, so the 4x4 side runs in a
child process on the same inputs.  Cases cover ragged bin and pixel blocks
(padding blocks of the fragment arrays) and 1, 2, 3 and 4 K-steps (every
tail of the K loop, which is unrolled by three).  The 2x4 results are checked
against the oracle elsewhere.
"""
import os
import subprocess
import sys

import numpy as np
import pytest

import synth
from tests._cases import freqs, make_csd

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CASES = [  # baseline, nside, nf, nt, antipodal
    ("AC", 16, 203, 61, True),   # 7 bin blocks, 4 K-steps
    ("AB", 8, 96, 33, True),     # 3 bin blocks, 3 K-steps
    ("BC", 4, 300, 17, False),   # 10 bin blocks, 2 K-steps, no antipodal pairs
    ("AB", 2, 31, 5, True),      # one partial block, one K-step
]

CHILD = r"""
import sys, numpy as np, torch
sys.path.insert(0, sys.argv[1])
import paper_1803_08285_amd as sg
d = np.load(sys.argv[2])
out = {}
for i in range(int(d["n"])):
    w = torch.from_numpy(d[f"w{i}"]).cuda()
    g = torch.from_numpy(d[f"g{i}"]).cuda()
    t = torch.from_numpy(d[f"t{i}"]).cuda()
    C = torch.zeros(w.shape, dtype=torch.complex64, device="cuda")
    _, G = sg.make_maps(C, w, sg.FGrid(20.0, 0.25), 0, g, t, antipodal=bool(d[f"a{i}"]), want_x=False)
    torch.cuda.synchronize()
    out[f"G{i}"] = G.cpu().numpy()
np.savez(sys.argv[3], **out)
print("child done", flush=True)
"""


@pytest.fixture(scope="module")
def sg():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    import paper_1803_08285_amd as sg

    return sg


def test_beam_4x4_matches_2x4_bitwise(sg, tmp_path):
    inputs, ref = {"n": len(CASES)}, []
    for i, (bl, nside, nf, nt, anti) in enumerate(CASES):
        tg = sg.TGrid(nt, 0.0, 86164.0905 / nt, 86164.0905 / nt)
        g, t = sg.build_geometry(synth.baseline_sites(bl), nside, tg)
        _, w = make_csd(11 + i, nt, freqs(20.0, 0.25, 0, nf))
        wt = torch.from_numpy(w).cuda()
        C = torch.zeros(wt.shape, dtype=torch.complex64, device="cuda")
        _, G = sg.make_maps(C, wt, sg.FGrid(20.0, 0.25), 0, g, t, antipodal=anti, want_x=False)
        torch.cuda.synchronize()
        ref.append(G.cpu().numpy())
        inputs.update({f"w{i}": w, f"g{i}": g.cpu().numpy(), f"t{i}": t.cpu().numpy(), f"a{i}": anti})
    src, dst = tmp_path / "in.npz", tmp_path / "out.npz"
    np.savez(src, **inputs)
    env = dict(os.environ, SGWB_BEAM_SHAPE="4x4")
    r = subprocess.run([sys.executable, "-c", CHILD, ROOT, str(src), str(dst)], env=env, capture_output=True,
                       text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    got = np.load(dst)
    for i, G in enumerate(ref):
        assert np.array_equal(got[f"G{i}"], G), f"case {CASES[i]}"


@pytest.mark.parametrize("nt,nf,npix", [(1, 1, 12), (3, 63, 65), (15, 64, 64), (17, 65, 100), (33, 130, 768)])
def test_float64_beam_at_tile_edges(nt, nf, npix):
    """The float64 Fisher diagonal at the edges of its 64 x 64 tiles and 16-segment
    steps, for any pixels (no pairing): sums of at most 33 positive terms, so
    within 64 units of 2^-53 of the exact value; padding adds nothing."""
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    import paper_1803_08285_amd as sg

    rng = np.random.default_rng(nt * 1000 + nf)
    w, g = rng.uniform(0.1, 2.0, (nt, nf)), rng.normal(size=(nt, npix))
    C = torch.zeros((nt, nf), dtype=torch.complex128, device="cuda")
    G = torch.full((nf, npix), -1.0, dtype=torch.float64, device="cuda")
    sg.make_maps(C, torch.from_numpy(w).cuda(), sg.FGrid(20.0, 0.25), 0, torch.from_numpy(g).cuda(),
                 torch.zeros((nt, npix), dtype=torch.float64, device="cuda"), antipodal=False, want_x=False,
                 out=(None, G))
    torch.cuda.synchronize()
    ref = (w.astype(np.longdouble).T @ (g.astype(np.longdouble) ** 2)).astype(np.float64)
    assert np.all(np.abs(G.cpu().numpy() - ref) <= 64 * 2.0 ** -53 * ref)


@pytest.mark.parametrize("nt", [1, 17, 64, 65, 129])
@pytest.mark.parametrize("nside,nf,antipodal", [(32, 720, True), (16, 1400, False)])
def test_small_calls_are_rows_of_large_ones(sg, nt, nside, nf, antipodal):
    """Calls of up to 4096 blocks of 32 x 32 outputs take one block a wave, larger
    ones 2 x 4: a small call's rows are bitwise those of the large one (1 to 9
    K-steps, the small form holds four in flight), which
    meet a float64 sum."""
    npix = 12 * nside * nside
    assert (nf + 31) // 32 * (npix // (64 if antipodal else 32)) > 4096
    g, t = sg.build_geometry(synth.baseline_sites("AB"), nside, sg.TGrid(nt, 0.0, 300.0, 300.0))
    w = torch.rand((nt, nf), generator=torch.Generator().manual_seed(nt), dtype=torch.float32).cuda()
    C = torch.zeros(w.shape, dtype=torch.complex64, device="cuda")

    def beam(lo, n):
        cut = slice(lo, lo + n)
        return sg.make_maps(C[:, cut].contiguous(), w[:, cut].contiguous(), sg.FGrid(20.0, 0.25), lo, g, t,
                            antipodal=antipodal, want_x=False)[1]

    G = beam(0, nf)
    for lo, n in ((0, 1), (31, 33), (5, 96), (nf - 64, 64)):
        assert torch.equal(beam(lo, n), G[lo:lo + n]), (lo, n)
    ref = w.cpu().double().T @ g.cpu().double() ** 2
    assert float(((G.cpu().double() - ref).abs() / ref.clamp_min(1e-300)).max()) <= 1e-4


@pytest.mark.parametrize("nf,npix", [(1, 700), (32, 96), (33, 97), (64, 32), (2, 33)])
def test_float64_beam_of_few_bins_or_columns(nf, npix):
    """Waves of a 64 x 64 tile that lie past the bins or the columns do nothing: the
    rest meets a float64 sum within 64 units of 2^-53."""
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    import paper_1803_08285_amd as sg

    nt = 19
    rng = np.random.default_rng(nf)
    w, g = rng.uniform(0.1, 2.0, (nt, nf)), rng.normal(size=(nt, npix))
    G = torch.full((nf, npix), -1.0, dtype=torch.float64, device="cuda")
    sg.make_maps(torch.zeros((nt, nf), dtype=torch.complex128, device="cuda"), torch.from_numpy(w).cuda(),
                 sg.FGrid(20.0, 0.25), 0, torch.from_numpy(g).cuda(),
                 torch.zeros((nt, npix), dtype=torch.float64, device="cuda"), antipodal=False, want_x=False,
                 out=(None, G))
    torch.cuda.synchronize()
    ref = (w.astype(np.longdouble).T @ (g.astype(np.longdouble) ** 2)).astype(np.float64)
    assert np.all(np.abs(G.cpu().numpy() - ref) <= 64 * 2.0 ** -53 * ref)


def test_float64_beam_of_few_bins_costs_less_than_a_full_tile(sg):
    """Three bins of a large map against 70 (two tiles of 64): 0.35 of the time (0.49
    where every wave of the tile works)."""
    nside, nt = 128, 240
    g, t = sg.build_geometry(synth.baseline_sites("AB"), nside, sg.TGrid(nt, 0.0, 300.0, 300.0), dtype=torch.float64)
    times = []
    for nf in (3, 70):
        C = torch.zeros((nt, nf), dtype=torch.complex128, device="cuda")
        w = torch.ones((nt, nf), dtype=torch.float64, device="cuda")
        G = torch.empty((nf, 12 * nside * nside), dtype=torch.float64, device="cuda")
        best = 1e9
        for _ in range(12):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            for _ in range(4):
                sg.make_maps(C, w, sg.FGrid(20.0, 0.25), 0, g, t, want_x=False, out=(None, G))
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b))
        times.append(best)
    print(f"3 bins {250 * times[0]:.0f} us, 70 bins {250 * times[1]:.0f} us")
    assert times[0] <= 0.42 * times[1]
