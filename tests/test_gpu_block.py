"""Block and two-pass steps against the marching kernels, bit for bit (the
plans share their arithmetic), at the edges of the blocks: lattices narrower
than a block, partial last blocks, halos that wrap; samples on the way."""
import numpy as np
import pytest

from gpu_util import require_gpu, say

pytestmark = pytest.mark.gpu

PRM = dict(a=0.01, b=0.5, kappa=0.1, rho_c=1.0, kT=1e-4, tau=0.8, init_sigma=1e-3)


def _state(lbf, L, kernel, tile, steps=7, graph=0, **kw):
    sim = lbf.Sim(L, 31 + L, sample_every=3, series_capacity=4, **PRM, **kw)
    sim.set_plan(kernel, tile, graph)
    sim.step(steps)
    m = sim.moments(series=True)
    return sim.fields(f=True)["f"], m["levels"], m["sk"], m["series"]


def _same(a, b):
    assert np.array_equal(a[0], b[0])
    assert a[1] == b[1]
    assert np.array_equal(a[2], b[2]) and np.array_equal(a[3], b[3])


@pytest.mark.parametrize("storage", ["fp32", "fp16"])
@pytest.mark.parametrize("L", [4, 5, 7, 8, 15, 16, 17, 31, 33, 36, 64])
def test_force_blocks(L, storage):
    lbf = require_gpu()
    say(f"blocks L={L} {storage}")
    ref = _state(lbf, L, "fused", (32, 8, 7), storage=storage)
    for kernel, tile in (("fused", (16, 8, 1)), ("fused", (16, 8, 4)), ("fused", (32, 8, 4)), ("split", (0, 0, 0))):
        _same(_state(lbf, L, kernel, tile, storage=storage), ref)


@pytest.mark.parametrize("L", [4, 8, 12, 36, 64])
def test_eq_blocks(L):
    lbf = require_gpu()
    say(f"eq blocks L={L}")
    ref = _state(lbf, L, "split", (0, 0, 0), eq_pressure=True)
    for tz in (1, 2):
        _same(_state(lbf, L, "rows", (32, 8, tz), eq_pressure=True), ref)


def test_force_off_and_graph():
    """No force (the potential is formed but not used), and a captured loop."""
    lbf = require_gpu()
    ref = _state(lbf, 20, "fused", (32, 8, 7), steps=12, force_off=True)
    for kernel, tile in (("rows", (16, 8, 1)), ("rows", (16, 8, 4)), ("split", (0, 0, 0))):
        _same(_state(lbf, 20, kernel, tile, steps=12, graph=6, force_off=True), ref)


@pytest.mark.parametrize("kernel,tile", [("rows", (16, 8, 4)), ("split", (0, 0, 0)), ("rows", (32, 8, 12))])
def test_batch_dealt_to_the_xcds(kernel, tile):
    """Uneven replicas (more and fewer than the eight XCDs, so that the dealt
    lists are padded): each equals the lone handle."""
    lbf = require_gpu()
    for Ls in ([8, 24, 4, 12, 40, 8, 16, 4, 20, 12, 8], [4, 36, 8]):
        prms = [dict(PRM, a=0.01 * k, sample_every=3) for k in range(len(Ls))]
        bat = lbf.Sim.batch(Ls, [50 + k for k in range(len(Ls))], prms)
        bat.set_plan(kernel, tile)
        bat.step(7)
        for r, L in enumerate(Ls):
            one = lbf.Sim(L, 50 + r, **prms[r])
            one.set_plan("fused", (32, 8, 7))
            one.step(7)
            assert np.array_equal(bat.fields(r, f=True)["f"], one.fields(f=True)["f"]), (Ls, r)
            assert bat.moments(r)["levels"] == one.moments()["levels"], (Ls, r)


def test_default_plans_by_size():
    lbf = require_gpu()
    S, F, R = lbf.LB_KERNEL_SPLIT, lbf.LB_KERNEL_FUSED, lbf.LB_KERNEL_ROWS
    for L, kw, want in ((8, {}, (R, 16, 8, 1)), (27, {}, (F, 16, 8, 1)), (40, {}, (S, 0, 0, 0)),
                        (48, {}, (R, 16, 8, 4)), (64, {}, (R, 32, 8, 4)), (66, {}, (S, 0, 0, 0)),
                        (96, {}, (S, 0, 0, 0)), (96, dict(storage="fp16"), (S, 0, 0, 0)),
                        (128, dict(storage="fp16"), (R, 64, 8, 8)), (32, dict(eq_pressure=True), (R, 32, 8, 1)),
                        (64, dict(eq_pressure=True), (R, 32, 8, 2)), (30, dict(eq_pressure=True), (S, 0, 0, 0))):
        p = lbf.Sim(L, 1, **PRM, **kw).plan()
        assert (p["kernel"], p["tile_x"], p["tile_y"], p["tile_z"]) == want, (L, kw, p)
