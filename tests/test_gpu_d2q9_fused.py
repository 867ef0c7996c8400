"""Several D2Q9 steps in one launch (small lattices) against the same steps one
at a time: fields bit for bit, at edges where tiles stick out of the lattice or
are wider than it, with samples, step counts and imports between launches."""
import numpy as np
import pytest

from gpu_util import require_gpu, say

pytestmark = pytest.mark.gpu

PRM = dict(a=0.02, b=0.1, kappa=0.1, rho_c=1.0, kT=1e-4, tau=0.8, init_sigma=0.01)


@pytest.mark.parametrize("L", [4, 5, 15, 16, 17, 23, 32, 40, 63, 100, 255, 256, 257])
def test_steps_in_one_launch(L):
    lbf = require_gpu()
    say(f"fused steps L={L}")
    a, b = lbf.Sim2D(L, 9, **PRM), lbf.Sim2D(L, 9, **PRM)
    for n in (1, 2, 3, 4, 5, 13):
        a.step(n)
        for _ in range(n):
            b.step(1)
        fa, fb = a.fields(f=True), b.fields(f=True)
        for k in ("rho", "j", "f"):
            assert np.array_equal(fa[k], fb[k]), (n, k)


def test_samples_and_imports_between():
    lbf = require_gpu()
    L = 48
    a, b = (lbf.Sim2D(L, 3, sample_every=5, **PRM) for _ in range(2))
    a.step(12)
    for _ in range(12):
        b.step(1)
    assert a.spectra()["n_samples"] == b.spectra()["n_samples"] == 2
    f = a.fields(f=True)["f"]
    a.set_populations(f)
    a.step(9)
    for _ in range(9):
        b.step(1)
    assert np.array_equal(a.fields(f=True)["f"], b.fields(f=True)["f"])
    sa, sb = a.spectra(), b.spectra()
    assert sa["n_samples"] == 4
    assert all(np.array_equal(sa[k], sb[k]) for k in ("S", "Jx", "Jy", "Jpar", "Jperp"))


def test_batch_and_instability():
    """A batch small enough for several steps a launch against lone handles,
    and the sticky flag from a step inside a launch."""
    lbf = require_gpu()
    L, R = 20, 5
    prms = [dict(PRM, a=0.01 * r) for r in range(R)]
    bat = lbf.Sim2D.batch(L, list(range(R)), prms)
    bat.step(7)
    for r in range(R):
        one = lbf.Sim2D(L, r, **prms[r])
        for _ in range(7):
            one.step(1)
        assert np.array_equal(bat.fields(f=True, replica=r)["f"], one.fields(f=True)["f"]), r
    bad = lbf.Sim2D(L, 1, **dict(PRM, a=0.9))  # c_s^2 beyond the covariance's domain
    bad.step(3)
    with pytest.raises(lbf.LBError) as e:
        bad.sync()
    assert e.value.code == lbf.LB_EUNSTABLE
