"""The native marshalling takes nothing it cannot vouch for: without a GPU every call is left to the path through ctypes."""
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
    for name in ("worker_step", "worker_step_sgd", "worker_step_fused", "worker_step_state", "server_step", "server_step_state",
                 "server_step_fused", "apply_wd", "apply_fused", "compressor_quality"):
        assert getattr(n, name)(key, t, t, t, 0.1, 0.1, 0.1, w, c, None) is None, name
    with pytest.raises(TypeError):
        n.bind(1)


@pytest.mark.parametrize("what", ["no library", "old", "another torch or header"])
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
    elif what == "old":
        os.utime(place, (1, 1))
    else:
        monkeypatch.setattr(build, "binding_built_for", lambda: "torch 0.0, ef.h 0")
    with pytest.warns(RuntimeWarning, match="calls go through ctypes"):
        ef._load_native(L)
    assert isinstance(ef._native, ef._ThroughCtypes) and ef._native.apply() is None
    assert ef.ef_strerror(-3)
