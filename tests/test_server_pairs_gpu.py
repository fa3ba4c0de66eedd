"""The server with two whole tiles of a block to a workgroup: runs of an even and an odd number of whole tiles, blocks of
exactly two, ends inside tiles, worker counts on both sides of the two tables, every route by which a block is
finished.  Same bar as the other parity tests; the layouts are short, so the kernels for large launches are asked for."""
import numpy as np
import pytest
import torch

import paper_1905_10936_amd as ef
from tests.parity_util import F, GpuState, synced_step
from tests.test_parity_gpu import _offs

pytestmark = pytest.mark.gpu

T = 4096
LAYOUTS = {
    "even_runs": [2 * T, 4 * T, 2 * T, 6 * T, 8 * T],
    "odd_runs": [9 * T, 11 * T, 13 * T, T, 15 * T],
    "off_the_tiles": [8 * T + 100, 9 * T - 300, 10 * T + 1, 2 * T + 200, 12 * T - 1, 7, 11 * T + 5],
    "long": [T - 5, 301 * T + 9, 3, 40 * T],
    "dense_between": [16 * T] + [33] * 150 + [21 * T, 12 * T + 7],
}


def _steps(name, M, limit=-1, spin=None, fused=False):
    offs = _offs(LAYOUTS[name])
    d = int(offs[-1])
    rng = np.random.default_rng(M + len(name))
    st = GpuState(offs, M, x0=rng.standard_normal(d).astype(F), fused=fused)
    st.plan.set_persistent(False)
    st.plan.tune(fuse_limit=limit) if limit >= 0 else None
    st.plan.tune(spin_limit=spin) if spin is not None else None
    assert st.plan.server_pairs(M) == (M <= 16 and limit != 0)
    eta_prev, stats = 0.0, {}
    for t, eta in enumerate([0.1, 0.05]):
        g = rng.standard_normal((M, d)).astype(F)
        g[rng.random((M, d)) < 0.05] = 0.0
        st.set_grads(g)
        synced_step(st, 0.9, eta_prev, eta, stats, "%s M=%d step %d" % (name, M, t))
        eta_prev = eta
    if spin is None:
        assert st.plan.last_fallbacks() == (0, 0)
    assert stats["scales_not_bit_equal"] == 0


@pytest.mark.parametrize("M", [1, 7, 8, 9, 12, 13, 16, 17])
@pytest.mark.parametrize("name", list(LAYOUTS))
def test_runs_of_whole_tiles(name, M):
    _steps(name, M, fused=M == 7)


@pytest.mark.parametrize("limit", [0, 1, 2, 5, 300])
@pytest.mark.parametrize("name", list(LAYOUTS))
def test_one_pass_limits(name, limit):
    _steps(name, 3 if limit != 5 else 10, limit=limit)


@pytest.mark.parametrize("M", [4, 11])
@pytest.mark.parametrize("name", list(LAYOUTS))
def test_no_wait_succeeds(name, M):
    _steps(name, M, spin=0)


WHICH = {           # layout, and whether calls of up to eight workers, of more, take pairs by plan creation's choice
    "whole_tiles": ([64 * T] * 20, True, False),
    "many_whole_tiles": ([64 * T] * 50, True, False),
    "off_the_tiles": ([100 * T + 77] * 30, True, True),
    "one_ragged_end": ([64 * T] * 40 + [33 * T + 55], True, False),
    "longer_than_one_tile_alone_takes": ([1100 * T] * 3, True, True),
    "dense_and_all_resident": ([33] * 20000 + [330 * T] * 4, False, False),
    "dense": ([33] * 20000 + [700 * T] * 4, True, True),
    "no_two_of_a_block": ([7 * T // 4] * 1400, False, False),
}


@pytest.mark.parametrize("name", list(WHICH))
def test_which_calls_take_pairs(name):
    """The choice, and the same results from every kernel it picks: a plan for sixteen workers and one for as many as there are
    agree on sign words, scales and the residual."""
    sizes, few, many = WHICH[name]
    offs = _offs(sizes)
    d = int(offs[-1])
    plan = ef.ef_plan_create(offs, 16)
    assert (plan.server_pairs(8), plan.server_pairs(9), plan.server_pairs(16)) == (few, many, many)
    assert not plan.server_pairs(17) and not ef.ef_plan_create(offs, 17).server_pairs(16)
    gen = torch.Generator("cuda").manual_seed(3)
    ws = torch.randint(-2 ** 63, 2 ** 63 - 1, (16, plan.W), dtype=torch.int64, device="cuda", generator=gen)
    wc = torch.rand(16, plan.B, device="cuda", generator=gen)
    te = torch.randn(d, device="cuda", generator=gen)
    for M in (3, 8, 9, 16):
        outs = []
        for p in (plan, ef.ef_plan_create(offs, M), ef.ef_plan_create(offs, 17)):
            e = te.clone()
            s, c = torch.zeros(plan.W, dtype=torch.int64, device="cuda"), torch.zeros(plan.B, device="cuda")
            ef.ef_server_step(p, M, ws[:M].contiguous(), wc[:M].contiguous(), e, 0.1, 0.05, s, c)
            assert p.last_fallbacks() == (0, 0)
            outs.append((s, c.view(torch.int32), e.view(torch.int32)))
        for other in outs[1:]:
            assert all(torch.equal(a, b) for a, b in zip(outs[0], other)), "%s M=%d" % (name, M)
