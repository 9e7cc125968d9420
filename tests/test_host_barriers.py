"""CPU check of the built kernels: at every workgroup barrier a wave has waited
for its LDS operations, whichever way it came there.

Waves hand each other data through LDS with a barrier between, and a barrier
does not wait for LDS operations by itself: the wait is an instruction before
it, which the compiler places. The test walks the instructions of the library's
gfx950 code (an LDS operation is in flight until an s_waitcnt lgkmcnt(0); what
is in flight at a join is so if it is on any path) and names every barrier that
can be reached with one in flight. Lane exchanges (ds_bpermute and the like)
touch no memory and do not count.
"""
import glob
import os
import re
import shutil
import subprocess

import pytest

from paper_2201_05213_amd import _lib
from paper_2201_05213_amd import build as nxbuild

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
INSTR = re.compile(r"^\t(\S+)(.*?)\s*// ([0-9A-F]+):")
TARGET = re.compile(r"<.*\+0x([0-9a-f]+)>$")


def functions(listing):
    """(name, [(address, mnemonic, operands, branch offset from the function's start)])"""
    name, code = None, []
    for line in listing:
        m = re.match(r"^[0-9a-f]+ <(\w+)>:", line)
        if m:
            if name:
                yield name, code
            name, code = m.group(1), []
            continue
        m = INSTR.match(line)
        if m and name:
            t = TARGET.search(line.rstrip()) if m.group(1).startswith(("s_branch", "s_cbranch")) else None
            code.append((int(m.group(3), 16), m.group(1), m.group(2), int(t.group(1), 16) if t else 0))
    if name:
        yield name, code


def undrained_barriers(code):
    start, index = code[0][0], {a: k for k, (a, _, _, _) in enumerate(code)}
    entered = [0] * len(code)  # bits: reached with nothing in flight (1), with an LDS operation (2)
    work, bad = [(0, 1)], set()
    while work:
        k, state = work.pop()
        while k < len(code) and not entered[k] & state:
            entered[k] |= state
            _, op, args, target = code[k]
            if op.startswith("ds_") and not re.match(r"ds_(bpermute|permute|swizzle|nop)", op):
                state = 2
            elif op == "s_waitcnt" and re.search(r"lgkmcnt\(0\)|^\s*0\s*$", args):
                state = 1
            elif op == "s_barrier" and state == 2:
                bad.add(code[k][0] - start)
            if op.startswith(("s_branch", "s_cbranch")):
                work.append((index[start + target], state))
            if op in ("s_branch", "s_endpgm", "s_setpc_b64"):
                break
            k += 1
    return sorted(bad)


def test_lds_operations_end_before_barriers(tmp_path):
    if not os.path.exists(_lib.LIB_PATH):
        nxbuild.build()
    lib = shutil.copy(_lib.LIB_PATH, tmp_path)
    subprocess.run([OBJDUMP, "--offloading", lib], check=True, capture_output=True, cwd=tmp_path)
    objects = sorted(glob.glob(str(tmp_path / "*gfx950*")))
    if len(objects) != 3:
        pytest.fail(f"gfx950 code objects of three sources expected: {objects}")
    found, barriers = {}, 0
    for obj in objects:
        out = subprocess.run([OBJDUMP, "-d", obj], check=True, capture_output=True, text=True).stdout
        for name, code in functions(out.splitlines()):
            n = sum(op == "s_barrier" for _, op, _, _ in code)
            if n:
                barriers += n
                bad = undrained_barriers(code)
                if bad:
                    found[name] = [hex(b) for b in bad]
    assert barriers > 100
    assert not found, found
