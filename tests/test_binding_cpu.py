"""The native marshalling takes nothing it cannot vouch for: without a GPU every call is left to the path through ctypes."""
import inspect
import os
import shutil
import struct

import pytest
import torch

import paper_1905_10936_amd as ef
from paper_1905_10936_amd import build


def test_calls_it_cannot_vouch_for_are_left_to_ctypes():
    ef.lib()
    if not os.path.exists(build.BINDING):
        pytest.skip("ef_binding.cpp could not be built here")
    n = ef._native
    key, t = struct.pack("Pqqqq", 0, 64, 1, 1, 16), torch.zeros(64)
    w, c = torch.zeros(1, dtype=torch.int64), torch.zeros(1)
    assert n.apply(key, t, w, c, 0.1, None) is None                  # host tensors
    assert n.apply(b"", t, w, c, 0.1, None) is None                  # a closed plan
    assert n.apply(key, t, w, c, 0.1) is None and n.apply() is None  # another number of arguments
    assert n.apply(key, None, w, c, 0.1, None) is None and n.apply(None, t, w, c, 0.1, None) is None
    assert n.apply(key, t, w, c, 0.1, torch) is None                 # a stream of its own
    # each with a call's own arguments, one of which is not on the GPU
    f, state, m = 0.1, struct.pack("Pq", 0, 1), torch.zeros(16, dtype=torch.uint8)
    calls = {"worker_step": (key, t, t, t, f, f, f, w, c), "worker_step_sgd": (key, t, t, f, f, w, c),
             "worker_step_fused": (key, t, t, t, f, f, f, m), "worker_step_state": (key, state, t, f, f, f, w, c),
             "server_step": (key, 1, w, c, t, f, f, w, c), "server_step_state": (key, state, 1, w, c, f, f, w, c),
             "server_step_fused": (key, 1, m, t, f, f, m), "apply": (key, t, w, c, f), "apply_wd": (key, t, t, w, c, f, f, f),
             "apply_fused": (key, t, m, f), "compressor_quality": (key, t, torch.zeros(2, dtype=torch.float64))}
    assert len(calls) == len(ef._NATIVE_CALLS)
    for name, args in calls.items():
        # the wrapper's own call has as many
        wrapper = inspect.signature(getattr(ef, "ef_" + name)).parameters
        expected = [k for k in wrapper if k != "static_scratch"]
        assert len(args) + 1 == len(expected), name
        assert getattr(n, name)(*args, None) is None, name
    with pytest.raises(TypeError):
        n.bind(1)


@pytest.mark.parametrize("what", ["no library", "other sources", "another torch"])
def test_a_binding_that_cannot_be_used_leaves_the_library_usable(what, tmp_path, monkeypatch):
    L = ef.lib()
    if not os.path.exists(build.BINDING):
        pytest.skip("ef_binding.cpp could not be built here")
    place = str(tmp_path / "_ef_binding.so")
    shutil.copy(build.BINDING, place)
    monkeypatch.setitem(build.TARGETS, place, build.TARGETS[build.BINDING])
    monkeypatch.setattr(build, "BINDING", place)
    monkeypatch.setattr(ef, "_native", ef._ThroughCtypes())
    if what == "no library":
        with open(place, "wb") as f:
            f.write(b"not a library")
    elif what == "other sources":
        header = str(tmp_path / "ef.h")
        shutil.copy(build.TARGETS[place][1][0], header)
        with open(header, "a") as f:
            f.write("int ef_one_more(void);\n")
        monkeypatch.setitem(build.TARGETS, place, (build.TARGETS[place][0], [header]))
    else:
        monkeypatch.setattr(torch, "__version__", "0.0")
    with pytest.warns(RuntimeWarning, match="calls go through ctypes"):
        ef._load_native(L)
    assert isinstance(ef._native, ef._ThroughCtypes) and ef._native.apply() is None
    assert ef.ef_strerror(-3)
