"""No loop over lanes around a buffer access in the library's kernels (CPU).

A buffer descriptor that the compiler cannot keep in scalar registers is read
lane by lane in a loop around its access.  The plane marches of the single-pass
kernels once had such loops with register spills inside, and gave wrong values;
their descriptors are scalars by construction now, and this test reads the
AMD assembly of the built library to see that none has come back with a
change of source or compiler.  A kernel with a descriptor per lane, compiled
here and never run, shows that the reading finds one.
"""
import os
import re
import shutil
import subprocess

import pytest

from paper_2609_30039_amd import build as B

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"

pytestmark = pytest.mark.skipif(not (os.path.exists(OBJDUMP) and os.path.exists(B.HIPCC)), reason="no ROCm tools")

LOOPED = r"""
#include <hip/hip_runtime.h>
__global__ void k_looped(const char* base, const int* which, unsigned* out) {
    const char* p = base + 4096 * which[threadIdx.x];
    auto r = __builtin_amdgcn_make_buffer_rsrc((void*)p, 0, 4096, 0x00027000);
    out[threadIdx.x] = __builtin_amdgcn_raw_buffer_load_b32(r, 4 * threadIdx.x, 0, 0);
}
__global__ void k_plain(const char* base, unsigned* out) {
    auto r = __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, 4096, 0x00027000);
    out[threadIdx.x] = __builtin_amdgcn_raw_buffer_load_b32(r, 4 * threadIdx.x, 0, 0);
}
"""


def _code_objects(lib, tmp):
    """The device code of a library built here, one file per translation unit."""
    path = shutil.copy(lib, tmp)
    subprocess.run([OBJDUMP, "--offloading", path], check=True, capture_output=True, cwd=tmp)
    return sorted(os.path.join(tmp, f) for f in os.listdir(tmp) if "amdgcn" in f and f.startswith(os.path.basename(lib)))


def _lane_loops(code):
    """(functions read, functions with a loop over lanes around a buffer access): the
    loop takes the descriptor of its first lane, masks the lanes that share it,
    makes the access and branches back while lanes are left."""
    text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", code], check=True, capture_output=True, text=True).stdout
    name, rows, seen, found = None, [], 0, []

    def scan():
        at = {a: n for n, (a, _) in enumerate(rows)}
        for n, (a, ins) in enumerate(rows):
            m = re.match(r"s_cbranch_(?:execnz|execz|scc[01]|vccnz|vccz) .*?<.*?\+(0x[0-9a-f]+)>|"
                         r"s_cbranch_(?:execnz|execz|scc[01]|vccnz|vccz) .*", ins)
            if not m or not m.group(1):
                continue
            to = at.get(rows[0][0] + int(m.group(1), 16))
            if to is None or to >= n or n - to > 120:
                continue
            body = [i for _, i in rows[to:n]]
            if (any("saveexec" in i for i in body) and any(i.startswith("buffer_") for i in body) and
                    any(re.match(r"v_cmp_eq_u(32|64)", i) for i in body) and
                    sum(i.startswith("v_readfirstlane_b32") for i in body) >= 2):
                found.append((name, body))
                return

    for line in text.splitlines():
        m = re.match(r"^([0-9a-f]+) <(.+)>:$", line)
        if m:
            if rows:
                scan()
            name, rows, seen = m.group(2), [], seen + 1
            continue
        m = re.match(r"^\s+(\S.*?)\s*//\s*([0-9A-Fa-f]+):(.*)$", line)
        if m and name:
            rows.append((int(m.group(2), 16), (m.group(1) + " " + m.group(3)).strip()))
    if rows:
        scan()
    return seen, found


def test_the_reading_finds_a_lane_loop(tmp_path):
    src, lib = tmp_path / "looped.hip", str(tmp_path / "liblooped.so")
    src.write_text(LOOPED)
    subprocess.run([B.HIPCC, "-x", "hip", *B.FLAGS, "-shared", str(src), "-o", lib], check=True, capture_output=True)
    out = tmp_path / "out"
    out.mkdir()
    names = [n for code in _code_objects(lib, str(out)) for n, _ in _lane_loops(code)[1]]
    assert len(names) == 1 and "k_looped" in names[0], names


def test_no_lane_loops_in_the_library(tmp_path):
    if not os.path.exists(B.LIB):
        B.build()
    seen, bad = 0, []
    for code in _code_objects(B.LIB, str(tmp_path)):
        n, found = _lane_loops(code)
        seen += n
        bad += [name for name, _ in found]
    assert seen > 100 and not bad, bad
