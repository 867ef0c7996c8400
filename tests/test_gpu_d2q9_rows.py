"""The one-step D2Q9 kernel on both sides of the rule that gives it scalar row
bases (work of the launch, another line for batches than for one lattice):
a replica of a batch equals the lone lattice bit for bit."""
import numpy as np
import pytest

from gpu_util import require_gpu, say

pytestmark = pytest.mark.gpu

PRM = dict(a=0.02, b=0.1, kappa=0.1, rho_c=1.0, kT=1e-4, tau=0.8, init_sigma=1e-3)


# alone / in a batch of two: below the rule both, above it in the batch only
# (full rows, ragged rows, a last tile of one column), above it both
@pytest.mark.parametrize("L", [536, 544, 601, 705, 886, 888])
def test_row_bases(L):
    lbf = require_gpu()
    say(f"row bases L={L}")
    one = lbf.Sim2D(L, 8, **PRM)
    two = lbf.Sim2D.batch(L, [7, 8], [dict(PRM, a=0.01), PRM])
    one.step(3)
    two.step(3)
    assert np.array_equal(one.fields(f=True)["f"], two.fields(f=True, replica=1)["f"])
