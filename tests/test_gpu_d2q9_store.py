"""D2Q9 batches on both sides of the cache-size rule for their stores, and a
lone lattice: replicas against handles of their own, bit for bit."""
import numpy as np
import pytest

from gpu_util import require_gpu, say

pytestmark = pytest.mark.gpu

PRM = dict(a=0.02, b=0.1, kappa=0.1, rho_c=1.0, kT=1e-4, tau=0.8, init_sigma=0.01)


# 72 bytes a site against 256 MiB: 3.73e6 sites
@pytest.mark.parametrize("L,R", [(256, 56), (256, 57), (320, 37), (1024, 4), (300, 42), (1536, 2)])
def test_batch_stores(L, R):
    lbf = require_gpu()
    say(f"stores L={L} R={R}")
    bat = lbf.Sim2D.batch(L, list(range(R)), [PRM] * R)
    bat.step(2)
    for r in (0, R // 2, R - 1):
        one = lbf.Sim2D(L, r, **PRM)
        one.step(2)
        assert np.array_equal(bat.fields(f=True, replica=r)["f"], one.fields(f=True)["f"]), r
