"""The built library's device code, disassembled, for a distance between instructions that the compiler does not keep by itself; and what
inline assembly has to tell it."""
import glob
import os
import re
import shutil
import struct
import subprocess

import pytest

LLVM = "/opt/rocm/llvm/bin"
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2402_19427_amd", "librglru.so")
OBJDUMP = shutil.which("llvm-objdump", path=LLVM)


def code_objects(blob):
    """gfx950 code objects of the offload bundles in a host library (magic, count, then offset, size and name of each entry)."""
    magic, at = b"__CLANG_OFFLOAD_BUNDLE__", 0
    while (at := blob.find(magic, at)) >= 0:
        pos = at + len(magic)
        (n,) = struct.unpack_from("<Q", blob, pos)
        pos += 8
        for _ in range(n if n < 16 else 0):
            off, size, length = struct.unpack_from("<QQQ", blob, pos)
            name = blob[pos + 24:pos + 24 + length]
            pos += 24 + length
            if b"gfx950" in name and size:
                yield blob[at + off:at + off + size]
        at += len(magic)


def registers(text):
    out = set()
    for a, b in re.findall(r"\bv\[(\d+):(\d+)\]", text):
        out |= set(range(int(a), int(b) + 1))
    return out | {int(a) for a in re.findall(r"\bv(\d+)\b", text)}


@pytest.fixture(scope="module")
def listings(tmp_path_factory):
    """The instructions of every code object, one a line."""
    if OBJDUMP is None or not os.path.exists(LIB):
        pytest.skip("no disassembler, or the library is not built")
    out, where = [], tmp_path_factory.mktemp("code")
    for i, obj in enumerate(code_objects(open(LIB, "rb").read())):
        path = where / ("%d.co" % i)
        path.write_bytes(obj)
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(path)], stdout=subprocess.PIPE, text=True, check=True).stdout
        out.append([l.split("//")[0].strip() for l in text.split("\n") if l.startswith("\t")])
    return out


def test_data_of_wide_stores_with_a_scalar_offset_is_left_alone(listings):
    """Behind a buffer store of 16 bytes whose offset is a scalar register, no vector instruction writes into its data registers
    for two cycles (an s_nop counts for its operand and one more)."""
    stores, bad = 0, []
    for lines in listings:
        for k, line in enumerate(lines):
            m = re.match(r"buffer_store_dwordx[34] (v\[\d+:\d+\]), v\d+, s\[\d+:\d+\], s\d+\b", line)
            if not m:
                continue
            stores += 1
            data, gap = registers(m.group(1)), 0
            for nxt in lines[k + 1:k + 3]:
                if gap >= 2:
                    break
                if nxt.startswith("s_nop"):
                    gap += int(nxt.split()[1], 0)
                elif re.match(r"v_(?!cmp)", nxt):
                    ops = nxt.split(None, 1)[1]
                    if registers(ops if "swap" in nxt else ops.split(",")[0]) & data:
                        bad.append((line, nxt))
                gap += 1
    assert stores > 0
    assert not bad, bad


def test_inline_assembly_names_m0_where_it_writes_it():
    """The compiler sets m0 in front of loads of its own: inline assembly that writes it has to say so, or it may be moved between."""
    found = 0
    for path in sorted(glob.glob(os.path.join(ROOT, "paper_2402_19427_amd", "csrc", "*.h*"))):
        for asm in re.findall(r"\basm(?: volatile)?\((.*?)\);", open(path).read(), re.S):
            if re.search(r"\b(s_mov_b32|s_add_u32|s_movk_i32) m0\b", asm):
                found += 1
                assert asm.rpartition(":")[2].count('"m0"') == 1, (path, asm)
    assert found > 0
