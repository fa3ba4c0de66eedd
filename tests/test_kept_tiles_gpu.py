"""Blocks beyond the one-pass limit: their last whole tiles wait for the block's scale in the main kernel, the tiles before
them are parked and, in the worker kernel with one workgroup per tile, written out in groups.  Numbers of parked tiles
that leave part of a group at the end, one tile over a group, one short of it.  Same bar as the other parity tests, and
no wait, a group's among them, runs out."""
import numpy as np
import pytest
import torch

import paper_1905_10936_amd as ef
from tests.parity_util import F, GpuState, synced_step
from tests.test_parity_gpu import _offs

pytestmark = pytest.mark.gpu

T = 4096
LAYOUTS = {                 # whole tiles of the blocks beyond a limit of 8: 2, 10, 16, 18, 24, 34 and others parked
    "on_the_tiles": [10 * T, 18 * T, 24 * T, 8 * T, 26 * T, 32 * T, 42 * T],
    "off_the_tiles": [9 * T + 100, 20 * T - 300, 3, 25 * T + 1, 27 * T + 500, 41 * T + 7, 5 * T],
}


@pytest.mark.parametrize("group", [2, 3, 16, 256])
@pytest.mark.parametrize("variant", ["momentum", "momentum_free", "diagnosing"])
@pytest.mark.parametrize("name", list(LAYOUTS))
def test_every_group_ends(name, variant, group):
    offs = _offs(LAYOUTS[name])
    d = int(offs[-1])
    M = 2
    rng = np.random.default_rng(group + len(variant))
    st = GpuState(offs, M, route="direct")
    st.plan.tune(fuse_limit=8)
    st.plan.set_sync_group(group)
    g = rng.standard_normal((M, d)).astype(F)
    st.set_grads(g)
    if variant == "momentum":
        synced_step(st, 0.9, 0.0, 0.1, None, "%s group %d" % (name, group))
        ef.ef_worker_step(st.plan, st.g, st.m, st.e, 0.9, 0.1, 0.1, st.ws, st.wc)
    elif variant == "momentum_free":
        ef.ef_worker_step_sgd(st.plan, st.g, st.e, 0.0, 0.1, st.ws, st.wc)
    else:
        q = torch.zeros((M, 2), dtype=torch.float64, device="cuda")
        ef.ef_worker_step_quality(st.plan, st.g, st.m, st.e, 0.9, 0.0, 0.1, st.ws, st.wc, q)
    assert st.plan.last_fallbacks() == (0, 0)
    st.plan.close()


def test_the_gather_of_a_block_of_more_rounds_than_polls():
    """A block's partial sums are read 1024 at a time, and a round that finds all of them costs no poll: with 96 polls the
    scale of 100 * 1024 + 8 tiles is still formed in the main kernel.  (Its kept tiles may give up on so small a budget.)
    The scale is the mean of |g|, rounded once from a sum in 64 bits."""
    d = (100 * 1024 + 8) * T
    plan = ef.ef_plan_create(np.array([0, d]), 1)
    plan.set_persistent(False)
    plan.tune(spin_limit=96)
    g = torch.randn(d, dtype=torch.float32, device="cuda", generator=torch.Generator("cuda").manual_seed(7))
    e = torch.zeros_like(g)
    ws = torch.zeros(plan.W, dtype=torch.int64, device="cuda")
    wc = torch.zeros(1, dtype=torch.float32, device="cuda")
    ef.ef_worker_step_sgd(plan, g, e, 0.0, 0.1, ws, wc)
    assert plan.last_fallbacks()[1] == 0
    scale = sum(float(part.abs().sum(dtype=torch.float64)) for part in g.split(1 << 24)) / d
    assert abs(float(wc) - scale) <= 2.0 ** -23 * scale         # one rounding to 32 bits, and the order of the 64-bit sum
    assert torch.equal(e, torch.where(g >= 0, g - wc, g + wc))
    plan.close()
