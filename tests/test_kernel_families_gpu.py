"""Small layouts run kernels of their own (csrc/ef_small.h) where plan creation chooses; the setting that picks the
worker's kernel sends every call to the kernels of the larger layouts, which is how the other tests reach those
with layouts of a few tiles."""
import zlib

import numpy as np
import pytest
import torch

import oracle
import paper_1905_10936_amd as ef
from tests.parity_util import F, GpuState, to_np
from tests.test_parity_gpu import LAYOUTS, ROUTES, _offs

pytestmark = pytest.mark.gpu

T = 4096
EVERY = {"worker", "server", "update"}


def test_which_calls_are_small_ones():
    plan = ef.ef_plan_create(_offs([30000] * 17), 4)
    assert plan.small_calls(4) == EVERY
    for choice in (True, False):
        plan.set_persistent(choice)
        assert plan.small_calls(4) == set()
    plan.set_persistent(None)
    assert plan.small_calls(4) == EVERY
    # a residual that is finished by a second pass keeps a call from them, and so does the deferred server
    plan.tune(fuse_limit=2)
    assert plan.small_calls(4) == {"update"}
    plan = ef.ef_plan_create(_offs([30000] * 17), 4)
    plan.set_lazy(True)
    assert plan.small_calls(4) == {"worker", "update"}
    plan.set_lazy(False)
    state = ef.ef_state_create(plan, 4)
    assert plan.small_calls(4) == EVERY
    state.close()
    # more workgroups than twice what is resident; a block that is too long
    assert ef.ef_plan_create(_offs([30000] * 60), 16).small_calls(16) == {"server", "update"}
    assert ef.ef_plan_create(_offs([257 * T]), 1).small_calls(1) == set()
    assert ef.ef_plan_create(_offs([200 * T, 200 * T, 112 * T]), 1).small_calls(1) == EVERY
    assert ef.ef_plan_create(_offs([200 * T, 200 * T, 112 * T, 1]), 1).small_calls(1) == {"worker", "server"}


@pytest.mark.parametrize("route", ROUTES)
def test_the_routes_of_the_parity_tests_are_those_of_the_larger_layouts(route):
    assert GpuState(_offs([5000, 20000, 7]), 2, route=route).plan.small_calls(2) == set()


@pytest.mark.parametrize("name", list(LAYOUTS))
def test_update_kernels_of_the_larger_layouts(name):
    """Both updates, bit for bit (elementwise fp32, one rounding per operation on both sides)."""
    offs = _offs(LAYOUTS[name])
    d = int(offs[-1])
    rng = np.random.default_rng(zlib.crc32(name.encode()) + 6)
    plan = ef.ef_plan_create(offs, 1)
    plan.set_persistent(False)
    assert plan.small_calls(1) == set()
    x, mt = rng.standard_normal(d).astype(F), rng.standard_normal(d).astype(F)
    xg, mg = torch.from_numpy(x.copy()).cuda(), torch.from_numpy(mt.copy()).cuda()
    for eta in (0.1, 0.05):
        signs, scales = oracle.compress(rng.standard_normal(d).astype(F), offs)
        sg, cg = torch.from_numpy(signs.view(np.int64)).cuda(), torch.from_numpy(scales).cuda()
        oracle.apply(x, signs, scales, offs, F(eta))
        ef.ef_apply(plan, xg, sg, cg, eta)
        oracle.apply_wd(x, mt, signs, scales, offs, F(eta), F(0.9), F(5e-4))
        ef.ef_apply_wd(plan, xg, mg, sg, cg, eta, 0.9, 5e-4)
        torch.cuda.synchronize()
        assert np.array_equal(to_np(xg).view(np.uint32), x.view(np.uint32))
        assert np.array_equal(to_np(mg).view(np.uint32), mt.view(np.uint32))
