"""Tiles where blocks meet, in the kernels for large launches: a few segments (taken among the whole tiles), many
(a kernel of their own), and blocks without whole tiles that go from one kind into the other.  A block of 257 tiles
keeps these layouts from the kernels for small launches.  Same bar as the other parity tests."""
import numpy as np
import pytest
import torch

import paper_1905_10936_amd as ef  # noqa: F401
from tests.parity_util import F, GpuState, synced_step
from tests.test_parity_gpu import _offs

pytestmark = pytest.mark.gpu

T = 4096
BIG = [257 * T + 5]
LAYOUTS = {
    # 2 to 9 segments a tile: both sides of the limit of 6
    "two_to_nine": BIG + [v for n in range(2, 10) for v in [T // n] * (2 * n)] + [7],
    # dense tiles beside few-segment ones, joined by blocks of two tiles without a whole one
    "joined": BIG + [33] * 130 + [5000] + [1500] * 4 + [6000, 40, 40, 5000] + [9] * 500 + [4200] * 3 + [64] * 70 + [5 * T] + [100],
    # blocks with whole tiles between tiles of each kind; whole vector ends inside a few-segment tile
    "whole_between": [T - 3] + BIG + [20] * 300 + [3 * T + 7, 4 * T - 9, 2 * T, 11] + [2000, 2100] * 5 + [300 * T + 1] + [3, 2, 1],
    # aligned blocks, then a ragged end alone
    "ragged_end": [257 * T, 2 * T, T, 3 * T, 1],
}


@pytest.mark.parametrize("spin", [None, 0])
@pytest.mark.parametrize("persistent", [False, True])
@pytest.mark.parametrize("name", list(LAYOUTS))
def test_tiles_where_blocks_meet(name, persistent, spin):
    offs = _offs(LAYOUTS[name])
    d, M = int(offs[-1]), 2 if persistent else 9
    rng = np.random.default_rng(len(name) + 7 * persistent)
    st = GpuState(offs, M, x0=rng.standard_normal(d).astype(F))
    st.plan.set_persistent(persistent)
    if spin is not None:
        st.plan.tune(spin_limit=spin)
    eta_prev, stats = 0.0, {}
    for t, eta in enumerate([0.1, 0.05]):
        g = rng.standard_normal((M, d)).astype(F)
        g[rng.random((M, d)) < 0.05] = 0.0
        st.set_grads(g)
        synced_step(st, 0.9, eta_prev, eta, stats, "%s step %d" % (name, t))
        eta_prev = eta
    if spin is None:
        assert st.plan.last_fallbacks() == (0, 0)
    assert stats["scales_not_bit_equal"] == 0


@pytest.mark.parametrize("M", [1, 7, 8, 16])
@pytest.mark.parametrize("limit", [-1, 0, 3, 258])
def test_one_pass_limits_and_worker_counts(limit, M):
    offs = _offs(LAYOUTS["whole_between"])
    d = int(offs[-1])
    rng = np.random.default_rng(M)
    st = GpuState(offs, M, fused=M == 7)
    st.plan.set_persistent(False)
    st.plan.tune(fuse_limit=limit)
    for t, eta in enumerate([0.1, 0.2]):
        st.set_grads(rng.standard_normal((M, d)).astype(F))
        synced_step(st, 0.5, 0.1 * t, eta, None, "M=%d limit=%d step %d" % (M, limit, t))


@pytest.mark.parametrize("spin", [None, 0])
@pytest.mark.parametrize("name", list(LAYOUTS))
def test_momentum_free_and_diagnosing_workers(name, spin):
    """The other variants of the worker's kernels give the bits of the plain call (checked against the oracle above),
    also where every wait gives up."""
    offs = _offs(LAYOUTS[name])
    d, M = int(offs[-1]), 3
    rng = np.random.default_rng(len(name))
    g, m, e = (rng.standard_normal((M, d)).astype(F) for _ in range(3))

    def run(kind, mu, spin):
        st = GpuState(offs, M)
        st.plan.set_persistent(False)
        if spin is not None:
            st.plan.tune(spin_limit=spin)
        st.set_grads(g)
        st.m[:, :d].copy_(torch.as_tensor(m))
        st.e[:, :d].copy_(torch.as_tensor(e))
        if kind == "sgd":
            ef.ef_worker_step_sgd(st.plan, st.g, st.e, 0.1, 0.2, st.ws, st.wc)
        elif kind == "quality":
            q = torch.zeros((M, 2), dtype=torch.float64, device="cuda")
            ef.ef_worker_step_quality(st.plan, st.g, st.m, st.e, mu, 0.1, 0.2, st.ws, st.wc, q)
        else:
            ef.ef_worker_step(st.plan, st.g, st.m, st.e, mu, 0.1, 0.2, st.ws, st.wc)
        torch.cuda.synchronize()
        return st

    for kind, mu in (("sgd", 0.0), ("quality", 0.9)):
        want, got = run("plain", mu, None), run(kind, mu, spin)
        for field in ("ws", "wc", "e"):
            assert torch.equal(getattr(want, field), getattr(got, field)), "%s: %s" % (kind, field)
