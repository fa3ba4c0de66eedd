"""A release writes the L2 back, and what it releases may be announced only when that is over.  The wait that belongs to the
compiler's fence goes missing where it knows of nothing on its way, the write-back itself not counted: then the announcement can be
there before the data.  No run can be relied on to show it, so this follows the control flow of the built kernels: on every path from
a write-back to a store or an atomic stands a wait for it."""
import os

import pytest

import paper_1905_10936_amd as ef
from tests.test_state_read_before_count import OBJDUMP, _kernels


def early_announcements(start, code):
    """Addresses of stores and atomics that can be reached from a write-back without a wait."""
    index = {at: i for i, (at, _, _) in enumerate(code)}
    bad = []
    todo = [i + 1 for i, (_, text, _) in enumerate(code) if text.startswith("buffer_wbl2")]
    seen = set()
    while todo:
        i = todo.pop()
        while i not in seen:
            seen.add(i)
            at, text, target = code[i]
            op = text.split()[0]
            if op == "s_waitcnt" and "vmcnt(0)" in text or op == "s_endpgm":
                break
            if op.startswith(("global_store", "global_atomic", "flat_store", "flat_atomic", "buffer_store", "buffer_atomic")):
                bad.append((at, text))
                break
            if op == "s_branch" or op.startswith("s_cbranch"):
                to = index[start + int(target.group(1) or "0", 16)]
                if op == "s_branch":
                    i = to
                    continue
                todo.append(to)
            i += 1
    return bad


def test_no_announcement_ahead_of_the_wait(tmp_path):
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    ef.lib()
    releasing = 0
    for name, (start, code) in _kernels(tmp_path).items():
        releasing += any(text.startswith("buffer_wbl2") for _, text, _ in code)
        assert not early_announcements(start, code), name
    assert releasing > 0


def test_the_check_sees_what_it_is_for():
    def run(*lines):
        return early_announcements(0, [(4 * i, text, None) for i, text in enumerate(lines)])

    back, wait, store, end = "buffer_wbl2 sc1", "s_waitcnt vmcnt(0)", "global_store_dwordx2 v1, v[2:3], s[8:9] sc1", "s_endpgm"
    assert not run(store, back, wait, store, end)
    assert run(wait, back, store, end)
    assert run(wait, back, "s_waitcnt lgkmcnt(0)", store, end)
