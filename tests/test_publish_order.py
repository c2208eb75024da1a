"""The block kernel's values that cross workgroups, in the built code (no GPU needed).

With two solver blocks per workgroup two threads of different waves publish
block scalars with agent-scope stores, and one thread counts the workgroup in.
A barrier does not wait for another wave's global stores, so each publishing
wave has to wait for its own (vmcnt(0)) before the last barrier ahead of the
counter's atomic; otherwise the last workgroup to arrive may read old scalars.
This walks the control flow of the built kernel from every such store."""
import os
import re
import shutil
import subprocess

import pytest

import paper_1306_1970_amd as flr

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
SO = os.path.join(os.path.dirname(os.path.abspath(flr.__file__)), "libflr.so")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    d = str(tmp_path_factory.mktemp("code"))
    shutil.copy(SO, d)
    subprocess.check_call([OBJDUMP, "--offloading", "libflr.so"], cwd=d, stdout=subprocess.DEVNULL)
    out = {}
    for f in sorted(os.listdir(d)):
        if "gfx950" not in f:
            continue
        text = subprocess.check_output([OBJDUMP, "-d", "--no-show-raw-insn", os.path.join(d, f)], text=True)
        name = None
        for line in text.splitlines():
            head = re.match(r"([0-9a-f]+) <(\S+)>:", line)
            ins = re.match(r"\s+(\S.*?)\s*// ([0-9A-F]+):(.*)", line)
            if head:
                name, base = head.group(2), int(head.group(1), 16)
                out[name] = []
            elif ins and name:
                # "<kernel+0x1a2c>" after a branch: its target
                to = re.search(r"<%s(?:\+0x([0-9a-f]+))?>" % re.escape(name), ins.group(3) + ins.group(1))
                out[name].append((int(ins.group(2), 16), ins.group(1),
                                  base + int(to.group(1) or "0", 16) if to else None))
    return out


def _successors(code):
    at = {a: i for i, (a, _, _) in enumerate(code)}
    nxt = []
    for i, (_, text, to) in enumerate(code):
        op = text.split()[0]
        s = []
        if op.startswith("s_branch") or op.startswith("s_cbranch"):
            s.append(at[to])
        if not op.startswith(("s_branch", "s_endpgm")) and i + 1 < len(code):
            s.append(i + 1)
        nxt.append(s)
    return nxt


def _reach(starts, nxt, stop):
    """Instructions reachable from the successors of starts; a stopping one is reached but not passed."""
    seen, todo = set(), [s for i in starts for s in nxt[i]]
    while todo:
        i = todo.pop()
        if i in seen:
            continue
        seen.add(i)
        if not stop(i):
            todo += nxt[i]
    return seen


def unordered_publications(code):
    """(stores, offending barriers): stores to the coherence point, and the barriers just ahead of a counting
    atomic that one of them reaches without its wave having waited for it."""
    nxt = _successors(code)
    text = [t for _, t, _ in code]
    barrier = [i for i, t in enumerate(text) if t.startswith("s_barrier")]
    atomic = {i for i, t in enumerate(text) if t.startswith("global_atomic_add")}
    stores = [i for i, t in enumerate(text) if t.startswith("global_store") and " sc1" in t]
    assert barrier and atomic, "not a publishing kernel"
    bad = []
    for b in barrier:
        if not _reach([b], nxt, lambda i: text[i].startswith("s_barrier")) & atomic:
            continue  # not the last barrier before a count
        for s in stores:
            if b in _reach([s], nxt, lambda i: text[i].startswith("s_waitcnt") and "vmcnt(0)" in text[i]):
                bad.append((code[s][0], code[b][0]))
    return stores, bad


def test_two_publishers_wait_for_their_stores(kernels):
    names = [n for n in kernels if re.search(r"k_blockILi2ELb0E", n) and not n.endswith(".kd")]
    assert len(names) == 1, names
    stores, bad = unordered_publications(kernels[names[0]])
    print("  %s: %d publishing stores, %d reach an arrival unordered" % (names[0], len(stores), len(bad)))
    assert len(stores) >= 9  # six scalars of a step, three more at an MM boundary
    assert not bad
