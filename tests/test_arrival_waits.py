"""Workgroups that hand results to one another through an arrival counter (the merge of context splits inside the
decode kernels, the sums of a group's workgroups in the centroid learning): before a wavefront reaches the barrier in
front of the count, all its device-scope stores and atomics must have been carried out.  Neither a barrier nor
__syncthreads() waits for global memory on gfx950, so the kernels need a wait of their own.  Checked on the machine
code of the built library, along every path of every kernel; no GPU is touched."""
import glob
import os
import re
import shutil
import subprocess

import pytest

import paper_2405_03917_amd as cq
from paper_2405_03917_amd import build as cq_build

OBJDUMP = os.path.join(os.path.dirname(os.path.realpath(cq_build.HIPCC)), "..", "lib", "llvm", "bin", "llvm-objdump")
OBJDUMP = next((p for p in (OBJDUMP, "/opt/rocm/llvm/bin/llvm-objdump") if os.path.exists(p)), None)

ATOMIC = re.compile(r"global_atomic_|flat_atomic_|buffer_atomic_")
STORE = re.compile(r"(global|flat|buffer)_store_")
TARGET = re.compile(r"<[^>]*?(?:\+0x([0-9a-f]+))?>")


def kernels(listing):
    """name -> [(offset in the kernel, text)] of a disassembly."""
    out, name, base = {}, None, 0
    for line in listing.splitlines():
        m = re.match(r"([0-9a-f]{16}) <(.*)>:", line)
        if m:
            name, base = m.group(2), int(m.group(1), 16)
            out[name] = []
            continue
        m = re.match(r"\t(.*?)\s*// ([0-9A-F]{12}):(.*)", line)
        if m and name is not None:
            out[name].append((int(m.group(2), 16) - base, (m.group(1) + " " + m.group(3)).strip()))
    return out


def unwaited(code):
    """(counts, faults) of a kernel: how many arrival counts it has, and the offsets of counts, and of the barriers in
    front of them, that a wavefront can reach while a device-scope store or atomic of its own is still under way."""
    at = {off: i for i, (off, _) in enumerate(code)}
    ops = [t.split()[0] for _, t in code]
    counts = {i for i, (_, t) in enumerate(code) if ATOMIC.match(t) and re.search(r"\bsc0\b", t)}      # (sc0: returns the old value)

    def successors(i):
        if ops[i] == "s_branch" or ops[i].startswith("s_cbranch"):
            yield at[int(TARGET.search(code[i][1]).group(1) or "0", 16)]
        if ops[i] not in ("s_branch", "s_endpgm") and i + 1 < len(code):
            yield i + 1

    def counted_behind(barrier):
        seen, todo = set(), list(successors(barrier))
        while todo:
            i = todo.pop()
            if i in seen or ops[i] == "s_barrier":
                continue
            if i in counts:
                return True
            seen.add(i)
            todo += successors(i)
        return False

    ends = counts | {i for i, op in enumerate(ops) if op == "s_barrier" and counted_behind(i)}
    seen, faults, todo = set(), set(), [(0, False)] if counts else []
    while todo:
        state = todo.pop()
        if state in seen:
            continue
        seen.add(state)
        i, pending = state
        if i in ends and pending:
            faults.add(code[i][0])
            continue
        if ops[i] == "s_waitcnt" and "vmcnt(0)" in code[i][1]:
            pending = False
        elif i not in counts and (ATOMIC.match(ops[i]) or (STORE.match(ops[i]) and re.search(r"\bsc1\b", code[i][1]))):
            pending = True
        todo += [(j, pending) for j in successors(i)]
    return len(counts), sorted(faults)


def test_the_walk_follows_both_sides_of_a_branch():
    store, count = "global_store_dword v0, v1, s[0:1] sc1", "global_atomic_add v0, v1, v2, s[2:3] sc0"

    def run(*text):
        return unwaited([(4 * i, t) for i, t in enumerate(text)])

    assert run(store, "s_waitcnt vmcnt(0)", "s_barrier", count, "s_endpgm") == (1, [])
    assert run(store, "s_waitcnt vmcnt(1)", "s_barrier", count, "s_endpgm") == (1, [8])
    assert run("s_cbranch_scc1 1 <k+0x8>", store, "s_waitcnt vmcnt(0)", "s_barrier", count, "s_endpgm") == (1, [])
    assert run(store, "s_cbranch_scc1 1 <k+0xc>", "s_waitcnt vmcnt(0)", "s_barrier", count, "s_endpgm") == (1, [12])
    assert run(store, "s_waitcnt vmcnt(0)", "s_barrier", "s_cbranch_execz 1 <k+0x14>", count, store, "s_barrier", "s_endpgm") == (1, [])
    assert run("s_barrier", store, count, "s_endpgm") == (1, [8])
    assert run("global_atomic_add_x2 v[0:1], v[2:3], off", "s_barrier", count, "s_endpgm") == (1, [4])


@pytest.mark.skipif(OBJDUMP is None, reason="no llvm-objdump")
def test_partials_are_written_before_their_workgroup_is_counted(tmp_path):
    cq.load()
    lib = shutil.copy(cq_build.LIB, tmp_path / "libcq.so")
    subprocess.check_call([OBJDUMP, "--offloading", lib], stdout=subprocess.DEVNULL)
    found, bad = {}, {}
    for obj in glob.glob(str(tmp_path / "libcq.so.*gfx950*")):
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", obj], check=True, capture_output=True, text=True).stdout
        for name, code in kernels(text).items():
            n, faults = unwaited(code)
            if n:
                found[name] = n
            if faults:
                bad[name] = [hex(f) for f in faults]
    families = {f: sum(f in n for n in found) for f in ("decode_split_kernel", "decode_pair_kernel", "kmeans_lloyd_kernel")}
    assert all(families.values()), families              # (the kernels that count are the ones looked at)
    assert not bad, bad
