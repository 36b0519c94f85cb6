"""The whole-run kernel's exchange stores, in the code that was built for gfx950.

A 128-bit store reads its data registers a little after it is issued; an instruction right behind it
that overwrites them needs a wait state.  The compiler inserts one only where the store's scalar
offset is not a register (with a register there it sees no hazard), and with a register the exchange
has been seen to publish the next word's payload under this word's tag.  So every such store of the
kernel has the constant offset 0, and none is followed by a write of its data registers."""
import re
import shutil
import struct
import subprocess

import pytest

from paper_2301_05518_amd import build

OBJDUMP = shutil.which("llvm-objdump", path="/opt/rocm/llvm/bin:/opt/rocm/lib/llvm/bin")
OBJCOPY = shutil.which("llvm-objcopy", path="/opt/rocm/llvm/bin:/opt/rocm/lib/llvm/bin")


def code_objects(fatbin: bytes):
    """The gfx950 code objects of the library's offload bundles."""
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = fatbin.find(magic)
    while at >= 0:
        (n,) = struct.unpack_from("<Q", fatbin, at + 24)
        p = at + 32
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", fatbin, p)
            ident = fatbin[p + 24:p + 24 + idlen].decode()
            p += 24 + idlen
            if "gfx950" in ident and size:
                yield fatbin[at + off:at + off + size]
        at = fatbin.find(magic, at + 24)


def registers(operand: str) -> set:
    m = re.fullmatch(r"v\[(\d+):(\d+)\]", operand)
    if m:
        return set(range(int(m[1]), int(m[2]) + 1))
    m = re.fullmatch(r"v(\d+)", operand)
    return {int(m[1])} if m else set()


def written(line: str) -> set:
    """Vector registers an instruction writes at once (loads write theirs much later)."""
    words = line.split(None, 1)
    if not words or not words[0].startswith("v_") or words[0].startswith("v_cmp") or len(words) < 2:
        return set()
    return registers(words[1].split(",")[0].strip())


def check(disassembly: str):
    """(kernel instances, 128-bit buffer stores, offending lines) of the whole-run kernel."""
    kernels, stores, bad = 0, 0, []
    inside, data = False, None
    for raw in disassembly.splitlines():
        if raw.endswith(">:"):
            inside = "smear_run" in raw
            kernels += inside
            data = None
            continue
        line = raw.split("//")[0].strip()
        if not inside or not line:
            continue
        if data is not None and written(line) & data:
            bad.append(f"data of the store before: {line}")
        data = None
        if line.startswith("buffer_store_dwordx4"):
            stores += 1
            ops = [o.strip() for o in line.split(None, 1)[1].split(",")]
            data = registers(ops[0])
            # vdata, vaddr, srsrc, soffset and modifiers
            if not re.match(r"0\b", ops[3]):
                bad.append(line)
    return kernels, stores, bad


def test_reads_the_forms_that_matter():
    """The check itself: a scalar offset in a register and an overwrite right behind are found."""
    good = "0 <_Zsmear_run>:\n buffer_store_dwordx4 v[2:5], v1, s[0:3], 0 offen sc1 // x\n s_nop 0\n v_mov_b32_e32 v2, v9\n"
    assert check(good) == (1, 1, [])
    assert len(check(good.replace(", 0 offen", ", s7 offen"))[2]) == 1
    assert len(check(good.replace(" s_nop 0\n", ""))[2]) == 1
    assert check(good.replace("v2, v9", "v6, v9").replace(" s_nop 0\n", ""))[2] == []
    assert check(good.replace("smear_run", "other"))[1] == 0


@pytest.mark.skipif(not OBJDUMP or not OBJCOPY, reason="no llvm-objdump")
def test_exchange_stores(tmp_path):
    fat = tmp_path / "fatbin"
    subprocess.run([OBJCOPY, f"--dump-section=.hip_fatbin={fat}", build.LIB, str(tmp_path / "copy.so")], check=True)
    kernels = stores = 0
    bad = []
    for k, obj in enumerate(code_objects(fat.read_bytes())):
        if b"smear_run" not in obj:
            continue
        f = tmp_path / f"obj{k}"
        f.write_bytes(obj)
        res = subprocess.run([OBJDUMP, "-d", "--mcpu=gfx950", str(f)], check=True, capture_output=True, text=True)
        a, b, c = check(res.stdout)
        kernels, stores, bad = kernels + a, stores + b, bad + c
    assert kernels == 32 and stores > 0        # four formats, one to four RHS, cut and whole cells
    assert not bad, bad[:5]
