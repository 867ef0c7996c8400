"""Large copies to and from host memory, which go through pinned pieces on
several threads, against lb_fields_static, whose copies stay with the runtime:
sizes on both sides of the threshold (6 MiB) and with a ragged last piece."""
import ctypes

import numpy as np
import pytest

from gpu_util import require_gpu

pytestmark = pytest.mark.gpu

PRM = dict(a=0.01, b=0.1, kappa=0.1, rho_c=1.0, kT=1e-4, tau=0.8, init_sigma=1e-2)


def _static(lbf, sim, rho, j, f):
    N = sim.Ls[0] ** 3
    out = [np.full(n * N, np.nan) if on else None for n, on in ((1, rho), (3, j), (19, f))]
    dp = ctypes.POINTER(ctypes.c_double)
    rc = lbf.lib().lb_fields_static(sim._h, 0, *[None if a is None else a.ctypes.data_as(dp) for a in out])
    assert rc == 0
    return out


# rho of 92^3 is 6.23e6 bytes, of 93^3 6.43e6 (the threshold is 6.29e6)
@pytest.mark.parametrize("L,rho,j,f", [(92, True, False, False), (93, True, False, False), (64, True, True, False),
                                       (56, False, False, True), (47, True, True, True)])
def test_fields_down(L, rho, j, f):
    lbf = require_gpu()
    sim = lbf.Sim(L, 3, **PRM)
    sim.step(2)
    got, want = sim.fields(rho=rho, j=j, f=f), _static(lbf, sim, rho, j, f)
    for k, w in zip(("rho", "j", "f"), want):
        if w is not None:
            assert np.array_equal(got[k].reshape(-1), w), k


@pytest.mark.parametrize("L", [33, 35, 50])  # 5.5 MB, 6.5 MB, 19 MB of populations
def test_populations_up_and_down(L):
    lbf = require_gpu()
    a = lbf.Sim(L, 3, **PRM)
    a.step(3)
    f = a.fields(f=True)["f"]
    b = lbf.Sim(L, 3, **PRM)
    b.set_populations(f)
    b.set_step(3)
    assert np.array_equal(b.fields(f=True)["f"], f)
    a.step(2)
    b.step(2)
    assert np.array_equal(b.fields(f=True)["f"], a.fields(f=True)["f"])


def test_spectra_and_fields_2d():
    lbf = require_gpu()
    L = 1000  # 8 MB an array
    g = lbf.Sim2D(L, 4, sample_every=1, a=0.02, b=0.1, kappa=0.1, rho_c=1.0, kT=1e-4, tau=0.8)
    g.step(1)
    st = g.fields(f=True)
    assert np.allclose(st["f"].sum(axis=0), st["rho"], rtol=0, atol=1e-12)
    h = lbf.Sim2D(L, 4, sample_every=1, a=0.02, b=0.1, kappa=0.1, rho_c=1.0, kT=1e-4, tau=0.8)
    h.set_populations(st["f"])
    assert np.array_equal(h.fields(f=True)["f"], st["f"])
    # Parseval over all modes
    d = st["rho"] - 1.0
    assert abs(g.spectra()["S"].sum() - (d * d).sum()) <= 1e-9 * (d * d).sum()
