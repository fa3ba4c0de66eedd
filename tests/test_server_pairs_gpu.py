"""The server with two whole tiles of a block to a workgroup: runs of an even and an odd number of whole tiles, blocks of
exactly two, ends inside tiles, worker counts on both sides of the two tables, every route by which a block is
finished.  Same bar as the other parity tests; the layouts are short, so the kernels for large launches are asked for."""
import numpy as np
import pytest

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
