"""The native marshalling of the step calls (csrc/ef_binding.cpp) against the path through ctypes: the same bits for every call and
every form of its arguments (one row or several, padded rows, signed and unsigned words, integer and NumPy scalars), and
the same exceptions for what neither takes."""
import numpy as np
import pytest
import torch

import paper_1905_10936_amd as ef

pytestmark = pytest.mark.gpu

T = 4096
OFFS = np.concatenate([[0], np.cumsum([3 * T + 7, 50, 1, 2 * T, 999])])
D = int(OFFS[-1])


def _state(plan, n, pad, seed=1):
    gen = torch.Generator("cuda").manual_seed(seed)
    ds = (D + 3) // 4 * 4 + 4 * pad
    shape = (D,) if n == 1 and pad < 0 else (n, ds)
    t = {k: torch.randn(shape, device="cuda", generator=gen) for k in ("g", "m", "e")}
    t["te"], t["x"], t["dm"] = (torch.randn(D, device="cuda", generator=gen) for _ in range(3))
    words = torch.uint64 if pad == 1 else torch.int64
    t["ws"], t["ss"] = torch.zeros(n, plan.W, dtype=words, device="cuda"), torch.zeros(plan.W, dtype=words, device="cuda")
    t["wc"], t["sc"] = torch.zeros(n, plan.B, device="cuda"), torch.zeros(plan.B, device="cuda")
    t["msg"], t["out"] = (torch.zeros(k * ef.ef_payload_bytes(plan), dtype=torch.uint8, device="cuda") for k in (n, 1))
    t["q"] = torch.zeros(n, 2, dtype=torch.float64, device="cuda")
    return t


class _Recorder:
    """A native module, and which of its calls answered."""

    def __init__(self, native):
        self.native, self.answers = native, []

    def __getattr__(self, name):
        def call(*args):
            rc = getattr(self.native, name)(*args)
            self.answers.append((name, rc is not None))
            return rc
        return call


def _run(n, pad, number, stream=None):
    plan = ef.ef_plan_create(OFFS, n)
    t = _state(plan, n, pad)
    a, b, c = number(0.9), number(0.1), number(0.05)
    if stream is not None:
        torch.cuda.synchronize()
    ef.ef_worker_step(plan, t["g"], t["m"], t["e"], a, b, c, t["ws"], t["wc"], stream=stream)
    ef.ef_server_step(plan, n, t["ws"], t["wc"], t["te"], b, c, t["ss"], t["sc"], stream)
    ef.ef_apply(plan, t["x"], t["ss"], t["sc"], c, stream)
    if stream is not None:
        torch.cuda.synchronize()
    ef.ef_apply_wd(plan, t["x"], t["dm"], t["ss"], t["sc"], c, a, number(0.01))
    ef.ef_worker_step_sgd(plan, t["g"], t["e"], b, c, t["ws"], t["wc"])
    ef.ef_worker_step_fused(plan, t["g"], t["m"], t["e"], a, b, c, t["msg"])
    ef.ef_server_step_fused(plan, n, t["msg"], t["te"], b, c, t["out"])
    ef.ef_apply_fused(plan, t["x"], t["out"], c)
    ef.ef_compressor_quality(plan, t["g"], t["q"])
    st = ef.ef_state_create(plan, n)
    ef.ef_worker_step_state(plan, st, t["g"], a, b, c, t["ws"], t["wc"])
    ef.ef_server_step_state(plan, st, n, t["ws"], t["wc"], b, c, t["ss"], t["sc"])
    torch.cuda.synchronize()
    st.close()
    plan.close()
    return t


@pytest.mark.parametrize("n,pad,number", [(1, -1, float), (1, 0, float), (3, 0, float), (3, 1, np.float64), (3, 2, np.float32),
                                          (2, 0, lambda v: torch.tensor(v, dtype=torch.float64))])
def test_the_same_bits_as_through_ctypes(n, pad, number, monkeypatch):
    ef.lib()
    native = ef._native
    assert not isinstance(native, ef._ThroughCtypes)
    recorder = _Recorder(native)
    monkeypatch.setattr(ef, "_native", recorder)
    got = _run(n, pad, number)
    # Python's numbers, NumPy's doubles (they are floats) and no stream: taken there, every one of the eleven; anything else: no number taken
    taken = number in (float, np.float64)
    assert len({name for name, _ in recorder.answers}) == len(ef._NATIVE_CALLS)
    assert all(answered == (taken or name == "compressor_quality") for name, answered in recorder.answers)
    monkeypatch.setattr(ef, "_native", ef._ThroughCtypes())
    want = _run(n, pad, number)
    for k in want:
        assert torch.equal(got[k].view(torch.uint8), want[k].view(torch.uint8)), k
    recorder = _Recorder(native)
    monkeypatch.setattr(ef, "_native", recorder)
    again = _run(n, pad, number, torch.cuda.Stream())       # a stream given: through ctypes
    assert [answered for _, answered in recorder.answers[:3]] == [False] * 3
    for k in want:
        assert torch.equal(again[k].view(torch.uint8), want[k].view(torch.uint8)), k


def _bad_calls(plan, t):
    n = 3
    args = [t["g"], t["m"], t["e"], 0.9, 0.1, 0.05, t["ws"], t["wc"]]

    def worker(**change):
        a = list(args)
        for k, v in change.items():
            a[int(k[1:])] = v
        return lambda: ef.ef_worker_step(plan, *a)

    return {
        "cpu": worker(a0=t["g"].cpu()), "dtype": worker(a1=t["m"].double()), "not_contiguous": worker(a0=t["g"][:, ::2]),
        "shape": worker(a1=t["m"][:2]), "words": worker(a6=t["ws"][:2]), "scales": worker(a7=t["wc"][:, :-1]),
        "mu": worker(a3=1.5), "mu_text": worker(a3="much"), "none": worker(a2=None), "eta": worker(a5=0.0),
        "overlap": worker(a0=t["m"]), "workers": lambda: ef.ef_server_step(plan, 4, t["ws"], t["wc"], t["te"], 0.1, 0.1, t["ss"], t["sc"]),
        "three_dims": worker(a0=t["g"][None]), "alignment": lambda: ef.ef_apply(plan, torch.zeros(D + 1, device="cuda")[1:], t["ss"], t["sc"], 0.1),
        "server_err": lambda: ef.ef_server_step(plan, n, t["ws"], t["wc"], t["te"][:-1], 0.1, 0.1, t["ss"], t["sc"]),
        "message": lambda: ef.ef_apply_fused(plan, t["x"], t["out"][:-1], 0.1), "quality": lambda: ef.ef_compressor_quality(plan, t["g"], t["q"][:2]),
    }


def test_the_same_exceptions_as_through_ctypes(monkeypatch):
    plan = ef.ef_plan_create(OFFS, 3)
    t = _state(plan, 3, 0)
    ef.lib()
    native, answers = ef._native, []
    for module in (native, ef._ThroughCtypes()):
        monkeypatch.setattr(ef, "_native", module)
        seen = {}
        for name, call in _bad_calls(plan, t).items():
            with pytest.raises(Exception) as e:
                call()
            seen[name] = (type(e.value), str(e.value))
        answers.append(seen)
    assert answers[0] == answers[1]
    monkeypatch.setattr(ef, "_native", native)
    plan.close()
    with pytest.raises(ef.EfError):
        ef.ef_apply(plan, t["x"], t["ss"], t["sc"], 0.1)
