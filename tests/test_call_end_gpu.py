"""Calls that their main kernel ends (no kernel after it): the last workgroup to begin steps the call state, and a workgroup whose
wait runs out either finishes its segment itself, if all have begun, or leaves it to the last one to begin.  Launches of
more workgroups than are resident at once, so that both happen, for whole tiles, pairs, tiles of few segments and dense ones;
every result has the bits of a plan whose waits succeed, call after call, and calls that k_tail ends stand between."""
import numpy as np
import pytest
import torch

import paper_1905_10936_amd as ef

pytestmark = pytest.mark.gpu

T = 4096
LAYOUTS = {
    "whole_tiles": [16 * T] * 300,
    "one_tile_blocks": [T] * 4500,
    "few_segments": [15 * T + 300, 7, 9 * T - 100] * 170,
    "dense": [33] * 120_000,
    "dense_between": ([40] * 300 + [6 * T + 5]) * 400,
}


def _tensors(offs, M, seed):
    d, B, W = int(offs[-1]), len(offs) - 1, (int(offs[-1]) + 63) // 64
    ds = (d + 3) // 4 * 4
    gen = torch.Generator("cuda").manual_seed(seed)
    t = {k: torch.randn(M, ds, device="cuda", generator=gen) for k in ("g", "m", "e")}
    t["te"] = torch.randn(d, device="cuda", generator=gen)
    t["ws"], t["wc"] = torch.zeros(M, W, dtype=torch.int64, device="cuda"), torch.zeros(M, B, device="cuda")
    t["ss"], t["sc"] = torch.zeros(W, dtype=torch.int64, device="cuda"), torch.zeros(B, device="cuda")
    return t


def _step(plan, t, M, sgd):
    if sgd:
        ef.ef_worker_step_sgd(plan, t["g"], t["e"], 0.1, 0.05, t["ws"], t["wc"])
    else:
        ef.ef_worker_step(plan, t["g"], t["m"], t["e"], 0.9, 0.1, 0.05, t["ws"], t["wc"])
    given_up = [plan.last_fallbacks()[0]]
    ef.ef_server_step(plan, M, t["ws"], t["wc"], t["te"], 0.1, 0.05, t["ss"], t["sc"])
    given_up.append(plan.last_fallbacks()[0])
    return given_up


@pytest.mark.parametrize("M", [1, 2, 9])
@pytest.mark.parametrize("name", list(LAYOUTS))
def test_waits_that_run_out_end_with_the_same_bits(name, M):
    offs = np.concatenate([[0], np.cumsum(LAYOUTS[name])])
    good, bad = ef.ef_plan_create(offs, M), ef.ef_plan_create(offs, M)
    a, b = _tensors(offs, M, 5), _tensors(offs, M, 5)
    for p in (good, bad):
        p.set_persistent(False)
    for k, spin in enumerate((0, 1, 0, 4, 2048)):
        bad.tune(spin_limit=spin)
        if k == 3:                      # a call that k_tail ends, in between: every block in two passes
            for p, t in ((good, a), (bad, b)):
                limit = p.fuse_limit
                p.tune(fuse_limit=0)
                _step(p, t, M, False)
                p.tune(fuse_limit=limit)
        assert _step(good, a, M, sgd=k == 2) == [0, 0]
        given_up = _step(bad, b, M, sgd=k == 2)
        # with no budget every segment of a block of several tiles gives up
        if spin == 0 and ((offs[1:] - 1) // T > offs[:-1] // T).any():
            assert min(given_up) > 0
        torch.cuda.synchronize()
        for key in a:
            assert torch.equal(a[key].view(torch.int32), b[key].view(torch.int32)), "%s M=%d call %d: %s" % (name, M, k, key)


@pytest.mark.parametrize("name", ["whole_tiles", "few_segments", "dense"])
def test_what_waits_leave_is_finished_by_many(name):
    """Thousands of waits that run out cost thousands of tiles' second pass, shared out, not one after the other: a workgroup
    moves a parked tile (32 KiB) in about 10 us, END_WGS = 16 of them in less than 1 us a tile; one wavefront alone takes 28."""
    offs = np.concatenate([[0], np.cumsum(LAYOUTS[name])])
    plan = ef.ef_plan_create(offs, 1)
    plan.set_persistent(False)
    plan.tune(spin_limit=0)
    t = _tensors(offs, 1, 3)
    took, parked = [], 0
    for _ in range(4):
        begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        begin.record()
        ef.ef_worker_step(plan, t["g"], t["m"], t["e"], 0.9, 0.1, 0.05, t["ws"], t["wc"])
        end.record()
        parked = plan.last_fallbacks()[0]
        took.append(begin.elapsed_time(end) * 1e3)
    assert parked > 900
    assert min(took) < 300 + 1.0 * parked, (took, parked)


@pytest.mark.parametrize("M", [2, 9])
def test_every_parked_tile_is_counted(M):
    """ef_plan_last_fallbacks counts tiles, whether a workgroup has one or two of them and whoever ends the call."""
    offs = np.concatenate([[0], np.cumsum(LAYOUTS["whole_tiles"])])
    plan, t = ef.ef_plan_create(offs, M), _tensors(offs, M, 7)
    plan.set_persistent(False)
    assert plan.server_pairs(M)
    plan.tune(spin_limit=0)
    assert _step(plan, t, M, False) == [M * int(offs[-1]) // T, int(offs[-1]) // T]


@pytest.mark.parametrize("names", [("whole_tiles", "few_segments"), ("dense", "whole_tiles"), ("few_segments", "dense")])
def test_plans_whose_calls_overlap(names):
    """Calls on two plans and two streams, more workgroups than are resident: workgroups of one wait in slots that the other's need, and with
    few polls some give up.  Every result has the bits of the same calls one after the other."""
    M, calls = 2, 6
    streams = [torch.cuda.Stream() for _ in names]
    want, got, plans = [], [], []
    for k, name in enumerate(names):
        offs = np.concatenate([[0], np.cumsum(LAYOUTS[name])])
        alone, plan = ef.ef_plan_create(offs, M), ef.ef_plan_create(offs, M)
        for p in (alone, plan):
            p.set_persistent(False)
        t = _tensors(offs, M, 11 + k)
        for _ in range(3 * calls):
            _step(alone, t, M, False)
        want.append(t)
        got.append(_tensors(offs, M, 11 + k))
        plans.append(plan)
    torch.cuda.synchronize()
    for spin in (2048, 8, 0):
        for p in plans:
            p.tune(spin_limit=spin)
        for _ in range(calls):
            for p, t, stream in zip(plans, got, streams):
                with torch.cuda.stream(stream):
                    ef.ef_worker_step(p, t["g"], t["m"], t["e"], 0.9, 0.1, 0.05, t["ws"], t["wc"])
                    ef.ef_server_step(p, M, t["ws"], t["wc"], t["te"], 0.1, 0.05, t["ss"], t["sc"])
        torch.cuda.synchronize()
    for name, a, b in zip(names, want, got):
        for key in a:
            assert torch.equal(a[key].view(torch.int32), b[key].view(torch.int32)), (name, key)
