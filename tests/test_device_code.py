"""Checks of the compiled gfx950 kernels of libtacg.so (CPU only): what the sources assume of their own machine code and
the compiler does not promise.  Skipped only where the library is not built."""
import os
import re
import shutil
import subprocess

import pytest

import paper_2606_01007_amd as tacg
from paper_2606_01007_amd import build

LLVM = os.path.join(os.path.dirname(os.path.realpath(build.HIPCC)), "..", "llvm", "bin")
if not os.path.isdir(LLVM):
    LLVM = "/opt/rocm/llvm/bin"


def _tool(name, *args):
    r = subprocess.run([os.path.join(LLVM, name), *args], capture_output=True, text=True, check=True)
    return r.stdout


@pytest.fixture(scope="module")
def code_objects(tmp_path_factory):
    """The gfx950 code objects of the built library, one file per translation unit."""
    if not os.path.exists(tacg.LIB_PATH):
        pytest.skip("libtacg.so not built")
    d = tmp_path_factory.mktemp("code")
    so = str(d / "libtacg.so")
    shutil.copy(tacg.LIB_PATH, so)
    _tool("llvm-objdump", "--offloading", so)
    out = sorted(str(p) for p in d.iterdir() if p.name.endswith("gfx950"))
    assert out
    return out


def _registers(text):
    regs = set()
    for m in re.finditer(r"\bv\[(\d+):(\d+)\]|\bv(\d+)\b", text):
        lo = int(m.group(1) or m.group(3))
        regs.update(range(lo, int(m.group(2) or lo) + 1))
    return regs


def _touched_in_flight(listing, issue):
    """Instructions that touch a result register of an `issue` instruction before a wait has covered it.  The LDS returns a
    wave's results in order: s_waitcnt lgkmcnt(n) covers an operation once n or more have been issued behind it."""
    kernels, found, name = {}, [], None
    pending, behind = set(), 0
    for line in listing.splitlines():
        m = re.match(r"^[0-9a-f]+ <(\S+)>:", line)
        if m:
            name, pending, behind = m.group(1), set(), 0
            continue
        ins = line.split("//")[0].strip()
        if not ins or name is None:
            continue
        op, _, rest = ins.partition(" ")
        if op.startswith(issue):
            kernels[name] = kernels.get(name, 0) + 1
            dst, _, src = rest.partition(",")
            if _registers(src) & pending:
                found.append((name, ins))
            pending |= _registers(dst)
            behind = 0
            continue
        if op == "s_waitcnt":
            m = re.search(r"lgkmcnt\((\d+)\)", rest)
            if m and int(m.group(1)) <= behind:
                pending = set()
            continue
        if pending and op.startswith("ds_"):
            behind += 1
        if pending & _registers(rest):
            found.append((name, ins))
    return kernels, found


def test_waits_cover_the_lds_exchanges(code_objects):
    """The decayed-load scoring issues its LDS exchanges in inline assembly and waits for them later: until that wait no
    instruction of the built kernels may read, move or overwrite a result."""
    kernels, found = {}, []
    for path in code_objects:
        k, f = _touched_in_flight(_tool("llvm-objdump", "-d", "--no-show-raw-insn", path), "ds_wrxchg2st64_rtn_b32")
        kernels.update(k)
        found += f
    assert len(kernels) == 16 * 4 * 2 and all("on_main" in k for k in kernels)
    assert not found, f"{len(found)} instructions, the first: {found[:5]}"


# static LDS that a launch with dynamic LDS above 64 KB counts in (bytes); the bit planes address theirs from 0
STATIC_LDS = {"ev_planes": 0, "ev_main": 0, "on_main": 0, "group_objective_kernel": 0, "coact_hist_kernel": 0,
              "coact_reduce_kernel": 0, "rw_graph": 0, "rw_pref": 512}


def test_static_lds_is_what_the_launches_assume(code_objects):
    seen = {}
    for path in code_objects:
        for m in re.finditer(r"\.group_segment_fixed_size:\s*(\d+)(?:(?!\.group_segment_fixed_size).)*?\.name:\s*(\S+)",
                             _tool("llvm-readelf", "--notes", path), re.S):
            for name in STATIC_LDS:
                if re.search(rf"\d{name}(?![a-z_])", m.group(2)):
                    seen.setdefault(name, set()).add(int(m.group(1)))
    assert seen == {name: {size} for name, size in STATIC_LDS.items()}


def test_the_check_of_waits_sees_a_missing_one():
    head = "0000000000001000 <k>:\n\tds_wrxchg2st64_rtn_b32 v[2:3], v9, v1, v1 offset1:1\n\tds_add_u32 v9, v8\n"
    use = "\tv_cvt_f64_u32_e32 v[4:5], v3\n"
    assert _touched_in_flight(head + use + "\ts_waitcnt lgkmcnt(1)\n", "ds_wrxchg2st64_rtn")[1]
    assert _touched_in_flight(head + "\ts_waitcnt lgkmcnt(2)\n" + use, "ds_wrxchg2st64_rtn")[1]
    assert not _touched_in_flight(head + "\ts_waitcnt vmcnt(0) lgkmcnt(1)\n" + use, "ds_wrxchg2st64_rtn")[1]
