"""CPU check of the built row decoder: a wave that stores pixels waits for its
stores before the workgroup's next barrier.

A band of a lane reads the rows above it from the image, where another
workgroup, possibly on another XCD, has stored them; that one publishes its
steps with a release at agent scope. The release waits for the stores of its own
wave (s_waitcnt vmcnt(0)), and a workgroup barrier waits for none: a wave that
leaves pixels to be published by another could have them in flight when the
step is published. The test walks the instructions of the gfx950 code (a byte
store is in flight until an s_waitcnt vmcnt(0); the row decoder stores bytes
to the image alone) and names every barrier that one is in flight at.
"""
import glob
import os
import re
import shutil
import subprocess

import pytest

from test_host_barriers import OBJDUMP, functions

from paper_2201_05213_amd import _lib
from paper_2201_05213_amd import build as nxbuild


def barriers_with_pixels_in_flight(code):
    start, index = code[0][0], {a: k for k, (a, _, _, _) in enumerate(code)}
    entered = [0] * len(code)  # bits: reached with nothing in flight (1), with a pixel store (2)
    work, bad = [(0, 1)], set()
    while work:
        k, state = work.pop()
        while k < len(code) and not entered[k] & state:
            entered[k] |= state
            _, op, args, target = code[k]
            if re.match(r"(flat|global|buffer)_store_byte", op):
                state = 2
            elif op == "s_waitcnt" and re.search(r"vmcnt\(0\)|^\s*0\s*$", args):
                state = 1
            elif op == "s_barrier" and state == 2:
                bad.add(code[k][0] - start)
            if op.startswith(("s_branch", "s_cbranch")):
                work.append((index[start + target], state))
            if op in ("s_branch", "s_endpgm", "s_setpc_b64"):
                break
            k += 1
    return sorted(bad)


def test_row_decoder_pixels_reach_memory_before_they_are_published(tmp_path):
    if not os.path.exists(_lib.LIB_PATH):
        nxbuild.build()
    lib = shutil.copy(_lib.LIB_PATH, tmp_path)
    subprocess.run([OBJDUMP, "--offloading", lib], check=True, capture_output=True, cwd=tmp_path)
    kernels, found = 0, {}
    for obj in sorted(glob.glob(str(tmp_path / "*gfx950*"))):
        out = subprocess.run([OBJDUMP, "-d", obj], check=True, capture_output=True, text=True).stdout
        for name, code in functions(out.splitlines()):
            if "k_decode_rows" not in name:
                continue
            kernels += 1
            assert any("store_byte" in op for _, op, _, _ in code), name
            assert any(op == "buffer_wbl2" for _, op, _, _ in code), name
            bad = barriers_with_pixels_in_flight(code)
            if bad:
                found[name] = [hex(b) for b in bad]
    if kernels == 0:
        pytest.fail("no row decoder in the library")
    assert not found, found
