"""Device-scope stores are waited for where other work-groups rely on their
order, shown on the machine code of the built library.

A work-group's release fence and barrier wait for LDS only: a store to memory
may still be on its way when a later one, to another address, has arrived.
Where the order matters the code has to wait on the vector-memory counter, on
every path and in every wave.  Timing hides a missing wait, so no run shows
it; here the kernels' control flow graphs are walked instead."""
import os
import re
import subprocess

import pytest

import paper_1502_00355_amd as sl

OBJDUMP = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-objdump")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """Kernel name -> [(address, instruction, branch target or None)]."""
    sl.lib()   # (refuses a library that was built from other sources)
    d = tmp_path_factory.mktemp("code")
    os.symlink(sl.LIB_PATH, d / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=d, check=True, stdout=subprocess.PIPE)
    out = {}
    for f in sorted(os.listdir(d)):
        if "gfx950" not in f:
            continue
        text = subprocess.run([OBJDUMP, "-d", f], cwd=d, check=True, stdout=subprocess.PIPE, text=True).stdout
        cur, base = None, 0
        for ln in text.splitlines():
            m = re.match(r"([0-9a-f]+) <(\S+)>:", ln)
            if m:
                cur, base = out.setdefault(m.group(2), []), int(m.group(1), 16)
                continue
            m = re.match(r"\t(.*?)\s*// ([0-9A-F]+):", ln)
            if not m or cur is None:
                continue
            ins, target = m.group(1).strip(), None
            if ins.startswith(("s_branch", "s_cbranch")):
                t = re.search(r"<[^+>]+(?:\+0x([0-9a-f]+))?>$", ln)
                target = base + (int(t.group(1), 16) if t.group(1) else 0)
            cur.append((int(m.group(2), 16), ins, target))
    return out


def walk(code, step):
    """Runs `step(state, instruction) -> state` over every path (states are
    sets, joined by union) and returns the state before each instruction."""
    index = {addr: k for k, (addr, _, _) in enumerate(code)}
    before = [None] * len(code)
    work = [(0, frozenset())]
    while work:
        k, s = work.pop()
        while k < len(code):
            s = s if before[k] is None else before[k] | s
            if s == before[k]:
                break
            before[k] = s
            _, ins, target = code[k]
            if ins.startswith("s_endpgm"):
                break
            s = step(s, ins)
            if target is not None:
                work.append((index[target], s))
                if ins.startswith("s_branch"):
                    break
            k += 1
    return before


def waits_for_all(ins):
    return ins.startswith("s_waitcnt") and "vmcnt(0)" in ins


def is_exchange_store(ins):
    return ins.startswith("global_store_dwordx2") and ins.endswith("sc1")


def test_exchange_stores_are_waited_for(kernels):
    """The flow kernels set a published position's slot back two versions
    ahead.  Before a wave publishes after a barrier, its stores from before
    that barrier are done."""
    names = [n for n in kernels if "k_sweep_flow" in n]
    assert len(names) == 20

    def step(s, ins):
        if waits_for_all(ins):
            return frozenset()
        if ins.startswith("s_barrier"):
            return frozenset("old" for _ in s)
        return s | {"new"} if is_exchange_store(ins) else s

    for n in names:
        code = kernels[n]
        at = [k for k, (_, ins, _) in enumerate(code) if is_exchange_store(ins)]
        assert len(at) >= 4, n
        before = walk(code, step)
        for k in at:
            assert before[k] is None or "old" not in before[k], "%s at %x" % (n, code[k][0])


def test_folds_are_waited_for_before_a_group_is_counted(kernels):
    """A launch's last work-group reads what the others left: a group's
    stores and atomics are done before the atomic that counts it."""
    def is_fold(ins):
        return (ins.startswith("global_store") and ins.endswith("sc1")) or \
               (ins.startswith("global_atomic") and not ins.endswith("sc0"))

    def step(s, ins):
        if waits_for_all(ins):
            return frozenset()
        return s | {"store"} if is_fold(ins) else s

    found = 0
    for n, code in kernels.items():
        if not re.search(r"k_sweep(_split|_lanes|_tile|_class)?I", n):
            continue
        # (in the tile kernel the others are the counters that deal the tiles)
        at = [k for k, (_, ins, _) in enumerate(code) if ins.startswith("global_atomic_add ") and ins.endswith("sc0") and
              ("k_sweep_tile" not in n or "offset:1152" in ins)]
        assert at, n
        found += 1
        before = walk(code, step)
        for k in at:
            assert not before[k], "%s at %x" % (n, code[k][0])
    assert found > 50
