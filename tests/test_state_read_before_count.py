"""A workgroup may count itself in only once all of its wavefronts have read the call state: the last one to be counted steps the
state.  That needs a barrier between every wavefront's read and the count, and the read has to be over at the barrier.
No run can be relied on to show a count that is too early, so this follows the control flow of the built kernels: on no path
from a kernel's entry to a count may the barrier be missing, nor a scalar load be on its way at the first one.  A count is an
atomic whose address has the lane number of a full mask added to it (arrive()): the compiler makes another mask for its own."""
import os
import re
import shutil
import subprocess

import pytest

import paper_1905_10936_amd as ef

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
# the kernels that may end their call, by what their mangled names contain: not those with dense and other tiles (tiles<.., 2, ..>),
# the server's pairs of more than eight workers and the mixed ones built without it, which leave that to k_tail
ENDING = ("k_worker_small", "k_server_small", "k_worker_tilesILb[01]ELi[01]E", "k_worker_mixedILb[01]ELb[01]ELb1E", "k_server_mixed",
          "k_server_tilesILi[01]ELb0E", "k_server_tilesILi[01]ELb1ELb0E")
COUNT_SPAN = 24         # instructions ahead of a count's atomic in which its address is formed


def _kernels(tmp):
    lib = shutil.copy(ef.LIB_PATH, os.path.join(str(tmp), "libef.so"))
    subprocess.run([OBJDUMP, "--offloading", lib], cwd=str(tmp), check=True, capture_output=True)
    image = [f for f in os.listdir(str(tmp)) if f.endswith("gfx950")]
    assert len(image) == 1
    text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", os.path.join(str(tmp), image[0])], check=True, capture_output=True,
                          text=True).stdout
    kernels, body = {}, None
    for line in text.splitlines():
        head = re.match(r"([0-9a-f]+) <(\w+)>:", line)
        if head:
            body = kernels[head.group(2)] = (int(head.group(1), 16), [])
        elif body is not None and "//" in line:
            code, _, place = line.partition("//")
            body[1].append((int(place.split(":")[0], 16), code.strip(), re.search(r"<\w+(?:\+0x([0-9a-f]+))?>\s*$", place)))
    return kernels


def is_count(code, i):
    if not code[i][1].startswith("global_atomic_add"):
        return False
    return any(re.match(r"v_mbcnt_lo_u32_b32\w* v\d+, -1, 0", text) for _, text, _ in code[max(0, i - COUNT_SPAN):i])


def early_counts(start, code):
    """Addresses of counts that can be reached without a barrier, and of first barriers that a scalar load may be outstanding at."""
    index = {at: i for i, (at, _, _) in enumerate(code)}
    seen, todo, bad = set(), [(0, False)], []
    while todo:
        i, loading = todo.pop()
        while (i, loading) not in seen:
            seen.add((i, loading))
            at, text, target = code[i]
            op = text.split()[0]
            if op.startswith(("s_setpc", "s_swappc", "s_call")):
                raise AssertionError("a call at %x: this test does not follow it" % at)
            if op.startswith("s_load"):
                loading = True
            elif op == "s_waitcnt" and "lgkmcnt(0)" in text:
                loading = False
            elif is_count(code, i):
                bad.append((at, text))
                break
            elif op == "s_barrier":
                if loading:
                    bad.append((at, "s_barrier with a scalar load on its way"))
                break
            if op == "s_endpgm":
                break
            if op == "s_branch" or op.startswith("s_cbranch"):
                to = index[start + int(target.group(1) or "0", 16)]
                if op == "s_branch":
                    i = to
                    continue
                todo.append((to, loading))
            i += 1
    return bad


def test_no_count_ahead_of_the_barrier(tmp_path):
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    ef.lib()
    kernels = {name: k for name, k in _kernels(tmp_path).items() if any(re.search(e, name) for e in ENDING)}
    for e in ENDING:
        assert any(re.search(e, name) for name in kernels), e
    for name, (start, code) in kernels.items():
        assert any(is_count(code, i) for i in range(len(code))), name
        assert not early_counts(start, code), name


def test_the_check_sees_what_it_is_for():
    def run(*lines):
        code = [(4 * i, text, re.search(r"<\w+(?:\+0x([0-9a-f]+))?>\s*$", text)) for i, text in enumerate(lines)]
        return early_counts(0, code)

    load, wait, barrier, end = "s_load_dwordx8 s[4:11], s[0:1], 0x0", "s_waitcnt lgkmcnt(0)", "s_barrier", "s_endpgm"
    lane, count = "v_mbcnt_lo_u32_b32 v1, -1, 0", "global_atomic_add v1, v0, v1, s[0:1] sc0"
    assert not run(lane, load, wait, barrier, count, end)
    assert run(lane, load, wait, count, barrier, end)
    assert run(lane, load, barrier, count, end)
    assert run(lane, load, wait, "s_cbranch_vccz 1 <k+0x14>", barrier, count, end)      # one of two paths
    assert not run(lane, load, wait, "s_cbranch_vccz 1 <k+0x18>", barrier, count, end)
    assert not run(load, wait, count, barrier, end)                                     # an atomic, but no count
