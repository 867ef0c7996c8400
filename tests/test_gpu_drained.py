"""Staged tiles that wait at every barrier (rows that are no whole sectors)
against the two-pass plan, bit for bit, samples on the way."""
import numpy as np
import pytest

from gpu_util import require_gpu, say

pytestmark = pytest.mark.gpu

PRM = dict(a=0.02, b=0.1, kappa=0.1, kT=1e-4, tau=0.8, sample_every=2)


@pytest.mark.parametrize("L,storage,kernel,tile", [
    (72, "fp16", "rows", (32, 8, 16)), (72, "fp16", "rows", (64, 4, 5)), (40, "fp16", "rows", (16, 16, 40)),
    (24, "fp16", "rows", (16, 8, 7)), (132, "fp32", "rows", (32, 8, 16)), (132, "fp32", "staged", (16, 16, 9)),
    (100, "fp32", "staged", (16, 8, 16)), (196, "fp32", "rows", (64, 4, 16)), (248, "fp16", "rows", (64, 8, 62)),
    (308, "fp32", "rows", (64, 8, 77))])
def test_drained_tiles(L, storage, kernel, tile):
    lbf = require_gpu()
    say(f"drained L={L} {storage} {kernel} {tile}")
    a, b = (lbf.Sim(L, 5, storage=storage, **PRM) for _ in range(2))
    a.set_plan("split", (0, 0, 0), 0)
    b.set_plan(kernel, tile, 0)
    a.step(3)
    b.step(3)
    fa, fb = a.fields(), b.fields()
    for k in ("rho", "j"):
        assert np.array_equal(fa[k], fb[k]), k
    ma, mb = a.moments(), b.moments()
    assert ma["n_samples"] == mb["n_samples"] == 1
    assert np.array_equal(ma["sk"], mb["sk"])
