"""The order of loads and stores in the built kernels: every streaming load of a tile is issued before the wait
that precedes the tile's stores, also where a lane mask guards those stores."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2609_34645_amd import build, emu

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
INSN = re.compile(r"^\t(\S+)([^/]*)// ([0-9A-F]+):")
TARGET = re.compile(r"<[^>]*\+0x([0-9a-f]+)>")


def masked_loads(body):
    """The streaming vector loads of a kernel's listing that sit in a block run under a narrowed lane mask: one
    that is entered, right after the mask is narrowed, by falling through s_cbranch_execz or from an
    s_cbranch_execnz above it (backwards, that branch closes a loop)."""
    insns = [(m[1], m[2], int(m[3], 16), line) for line in body.splitlines() if (m := INSN.match(line))]
    first = insns[0][2]
    targets, guarded = set(), set()
    for i, (op, _, at, line) in enumerate(insns):
        if "branch" not in op:
            continue
        t = TARGET.search(line)
        to = first + int(t[1], 16) if t else None
        targets.add(to)
        if not i or "saveexec" not in insns[i - 1][0]:
            continue
        if op == "s_cbranch_execz" and i + 1 < len(insns):
            guarded.add(insns[i + 1][2])
        elif op == "s_cbranch_execnz" and to is not None and to > at:
            guarded.add(to)
    out, inside = [], False
    for i, (op, args, at, _) in enumerate(insns):
        if at in guarded:
            inside = True
        elif at in targets or (i and "branch" in insns[i - 1][0]):
            inside = False
        if inside and re.match(r"(global|buffer)_load_dwordx[24]$", op) and re.search(r"\bnt\b", args):
            out.append(op + args)
    return out


def test_masked_loads_reads_a_listing():
    """The listing of a guarded store with its load behind the wait, and with the load ahead of it."""
    def listing(*ops):
        return "\n".join(f"\t{op:60}// {4 * i:012X}: 00000000" + (f" <k+0x{to:x}>" if to else "")
                         for i, (op, to) in enumerate(ops))

    load, store, wait = "global_load_dwordx4 v[0:3], v4, s[0:1] nt", "global_store_dwordx4 v4, v[0:3], s[2:3] nt", "s_waitcnt vmcnt(0)"
    mask, guard = "s_and_saveexec_b64 s[4:5], vcc", "s_cbranch_execz 3"
    assert len(masked_loads(listing((wait, 0), (mask, 0), (guard, 20), (load, 0), (store, 0), ("s_endpgm", 0)))) == 1
    assert masked_loads(listing((load, 0), (wait, 0), (mask, 0), (guard, 20), (store, 0), ("s_endpgm", 0))) == []
    assert masked_loads(listing((mask, 0), (guard, 12), (store, 0), (load, 0), (wait, 0), ("s_endpgm", 0))) == []


@pytest.mark.skipif(not shutil.which(OBJDUMP), reason="no llvm-objdump")
def test_no_streaming_load_under_a_lane_mask(tmp_path):
    """A load that only a guarded store uses is moved into the store's block by the compiler where nothing holds
    it above: it then starts after the wait for the others, and the piece takes two memory latencies."""
    if not os.path.exists(emu.LIB_PATH):
        build.build()
    lib = shutil.copy(emu.LIB_PATH, tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", lib], cwd=tmp_path, check=True, capture_output=True)
    code = [p for p in os.listdir(tmp_path) if "gfx950" in p]
    assert len(code) == 1
    text = subprocess.run([OBJDUMP, "-d", code[0]], cwd=tmp_path, check=True, capture_output=True, text=True).stdout
    kernels = dict(re.findall(r"^[0-9a-f]+ <(\S*k_(?:reshard|buckets)\S*)>:\n(.*?)(?=^\S|\Z)", text, re.S | re.M))
    assert len(kernels) > 100
    assert sum(len(re.findall(r"_load_dwordx[24] .*\bnt\b", b)) for b in kernels.values()) > 1000
    bad = {n: m for n, b in kernels.items() if (m := masked_loads(b))}
    assert not bad, f"{len(bad)} of {len(kernels)} kernels, e.g. {next(iter(bad.items()))}"
