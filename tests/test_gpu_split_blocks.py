"""The split plan's collide pass on both of its block shapes (by storage and
number of sites) against the marching kernels, bit for bit: edges that leave
partial blocks in every direction, a lattice thinner than a block, samples."""
import numpy as np
import pytest

from gpu_util import require_gpu, say

pytestmark = pytest.mark.gpu

PRM = dict(a=0.02, b=0.1, kappa=0.1, kT=1e-4, tau=0.8, sample_every=2)


@pytest.mark.parametrize("L,storage", [(4, "fp32"), (17, "fp16"), (33, "fp32"), (35, "fp16"), (62, "fp32"),
                                       (189, "fp32"), (190, "fp32"), (190, "fp16")])
def test_split_blocks(L, storage):
    lbf = require_gpu()
    say(f"split blocks L={L} {storage}")
    a, b = (lbf.Sim(L, 5, storage=storage, **PRM) for _ in range(2))
    a.set_plan("split", (0, 0, 0), 0)
    b.set_plan("fused", (32, 8, max(16, L // 8)), 0)
    a.step(3)
    b.step(3)
    fa, fb = a.fields(), b.fields()
    for k in ("rho", "j"):
        assert np.array_equal(fa[k], fb[k]), k
    ma, mb = a.moments(), b.moments()
    assert ma["n_samples"] == mb["n_samples"] == 1
    assert np.array_equal(ma["sk"], mb["sk"])
