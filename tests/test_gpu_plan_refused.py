"""A plan that cannot be had for want of device memory (an allocator that
refuses) leaves the handle on the plan it had, and able to step."""
import ctypes

import numpy as np
import pytest

from gpu_util import require_gpu

pytestmark = pytest.mark.gpu

PRM = dict(a=0.01, b=0.1, kappa=0.1, rho_c=1.0, kT=1e-4, tau=0.8, init_sigma=1e-3)


@pytest.mark.parametrize("had", [("split", (0, 0, 0)), ("rows", (32, 8, 12)), ("rows", (16, 8, 4))])
def test_refused_plan_changes_nothing(had):
    lbf = require_gpu()
    import torch
    ref = lbf.Sim(24, 9, **PRM)  # torch's allocator is in place from here on
    refuse = []

    def alloc(n, _ctx):
        return None if refuse else torch.cuda.caching_allocator_alloc(int(n))

    hooks = lbf._ALLOC_T(alloc), lbf._FREE_T(lambda p, _ctx: torch.cuda.caching_allocator_delete(p))
    lbf._check(lbf.lib().lb_set_allocator(hooks[0], hooks[1], None), "lb_set_allocator")
    try:
        sim = lbf.Sim(24, 9, **PRM)
    finally:
        lbf._check(lbf.lib().lb_set_allocator(lbf._torch_hooks[0], lbf._torch_hooks[1], None), "lb_set_allocator")
    sim.set_plan(*had)
    sim.step(3)
    before = sim.plan()
    refuse.append(True)
    for want in (("fused", (16, 16, 24)), ("split", (0, 0, 0))):
        if want != had:
            with pytest.raises(lbf.LBError):
                sim.set_plan(*want)
    refuse.clear()
    assert sim.plan() == before
    sim.step(4)
    ref.step(7)
    assert np.array_equal(sim.fields(f=True)["f"], ref.fields(f=True)["f"])
    sim.set_plan("fused", (16, 16, 24))
    sim.step(1)
    ref.step(1)
    assert np.array_equal(sim.fields(f=True)["f"], ref.fields(f=True)["f"])
    del sim  # while its allocator's functions are alive
