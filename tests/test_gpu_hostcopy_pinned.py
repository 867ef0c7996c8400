"""Large fields into and out of arrays that are pinned already (the runtime's
own copy) against pageable ones (pinned pieces)."""
import ctypes

import numpy as np
import pytest

from gpu_util import require_gpu

pytestmark = pytest.mark.gpu

PRM = dict(a=0.01, b=0.1, kappa=0.1, rho_c=1.0, kT=1e-4, tau=0.8, init_sigma=1e-2)


def test_pinned_arrays():
    lbf = require_gpu()
    import torch
    L = 60  # 33 MB of populations
    a = lbf.Sim(L, 3, **PRM)
    a.step(2)
    f = torch.empty(19 * L ** 3, dtype=torch.float64, pin_memory=True)
    p = ctypes.cast(f.data_ptr(), ctypes.POINTER(ctypes.c_double))
    assert lbf.lib().lb_fields(a._h, 0, None, None, p) == lbf.LB_OK
    want = a.fields(f=True)["f"].reshape(-1)
    assert np.array_equal(f.numpy(), want)
    b = lbf.Sim(L, 3, **PRM)
    assert lbf.lib().lb_set_populations(b._h, 0, p) == lbf.LB_OK
    b.set_step(2)
    assert np.array_equal(b.fields(f=True)["f"].reshape(-1), want)
