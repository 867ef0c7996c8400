"""Spectra of the D2Q9 model at lengths of every kind of factor (the transforms
take factors 8, 4, 2, 3, 5 as butterflies and other primes directly), odd and
even, smallest and largest of each workgroup size, against numpy's FFT of the
exported fields; alone and in a batch."""
import numpy as np
import pytest

from gpu_util import require_gpu, say

pytestmark = pytest.mark.gpu

PRM = dict(a=0.02, b=0.1, kappa=0.1, rho_c=1.0, kT=1e-4, tau=0.8, init_sigma=0.01)


def _spectra(st, L):
    d, jx, jy = (np.fft.fft2(v.reshape(L, L)) for v in (st["rho"] - 1.0, st["j"][0], st["j"][1]))
    m = np.fft.fftfreq(L) * L
    if L % 2 == 0:
        m[L // 2] = L // 2  # folded into (-L/2, L/2]
    my, mx = np.meshgrid(m, m, indexing="ij")
    kn = np.hypot(mx, my)
    kn[0, 0] = 1.0
    hx, hy = mx / kn, my / kn
    return {k: np.abs(v) ** 2 / L ** 2 for k, v in (("S", d), ("Jx", jx), ("Jy", jy), ("Jpar", hx * jx + hy * jy),
                                                   ("Jperp", hx * jy - hy * jx))}


def _close(got, want, what):
    """FP64 transforms of FP64 sums of the same state: rounding of order 1e-15
    of the largest mode, and 1e-16 in every exported density; the k = 0 modes
    (conserved sums near zero) left out."""
    for k in want:
        w, g = want[k].reshape(-1)[1:], got[k].reshape(-1)[1:]
        assert np.max(np.abs(g - w)) <= 1e-10 * np.max(np.abs(w)), (what, k)


@pytest.mark.parametrize("L", [4, 5, 6, 7, 8, 9, 10, 11, 13, 14, 15, 18, 20, 21, 22, 25, 27, 30, 32, 35, 49, 50, 77,
                               94, 97, 100, 127, 143, 180, 250, 257, 341, 343, 376, 500, 683, 684, 1000, 1365, 1367])
def test_any_length(L):
    lbf = require_gpu()
    say(f"spectra L={L}")
    g = lbf.Sim2D(L, 5, sample_every=2, **PRM)
    want = None
    for _ in range(2):
        g.step(2)
        sp = _spectra(g.fields(), L)
        want = sp if want is None else {k: want[k] + sp[k] for k in sp}
    got = g.spectra()
    assert got["n_samples"] == 2
    _close(got, want, L)
    again = g.spectra()
    assert all(np.array_equal(got[k], again[k]) for k in want)


@pytest.mark.parametrize("L,R", [(4, 3), (7, 40), (36, 9), (100, 16), (128, 20), (200, 12), (600, 3)])
def test_batches(L, R):
    """The columns of a batch are transformed several a workgroup: each
    replica's spectra are those of its lone handle, bit for bit."""
    lbf = require_gpu()
    say(f"spectra L={L} x {R}")
    prms = [dict(PRM, a=0.01 + 0.001 * r, sample_every=2) for r in range(R)]
    bat = lbf.Sim2D.batch(L, list(range(R)), prms)
    bat.step(4)
    for r in sorted({0, R // 2, R - 1}):
        one = lbf.Sim2D(L, r, **prms[r])
        one.step(4)
        a, b = bat.spectra(r), one.spectra()
        assert a["n_samples"] == b["n_samples"] == 2
        assert all(np.array_equal(a[k], b[k]) for k in ("S", "Jx", "Jy", "Jpar", "Jperp")), r
