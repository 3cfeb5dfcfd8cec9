"""The built library's device code, disassembled: distances between instructions that the compiler does not keep by itself."""
import os
import re
import shutil
import struct
import subprocess

import pytest

LLVM = "/opt/rocm/llvm/bin"
LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2402_19427_amd", "librglru.so")
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
    """(name, instructions) of every function."""
    if OBJDUMP is None or not os.path.exists(LIB):
        pytest.skip("no disassembler, or the library is not built")
    out, where = [], tmp_path_factory.mktemp("code")
    for i, obj in enumerate(code_objects(open(LIB, "rb").read())):
        path = where / ("%d.co" % i)
        path.write_bytes(obj)
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(path)], stdout=subprocess.PIPE, text=True, check=True).stdout
        for fn in re.split(r"\n(?=[0-9a-f]{16} <)", text)[1:]:
            name, _, body = fn.partition("\n")
            out.append((name, [l.split("//")[0].strip() for l in body.split("\n") if l.startswith("\t")]))
    return out


def test_data_of_wide_stores_with_a_scalar_offset_is_left_alone(listings):
    """Behind a buffer store of 16 bytes whose offset is a scalar register, no vector instruction writes into its data registers
    for two cycles (an s_nop counts for its operand and one more)."""
    stores, bad = 0, []
    for _, lines in listings:
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


def test_loads_written_out_restore_m0(listings):
    """The direct-to-LDS loads written out by hand (those of the kernels in tiles) put back what m0 held: the compiler does not know
    that they write it."""
    loads, bad = 0, []
    for name, lines in listings:
        if not re.search("(bwd|fwd)_tile_kernel|tile_wgrad_kernel", name):
            continue
        for k, line in enumerate(lines):
            if not re.match(r"buffer_load_dwordx4 .*\blds$", line):
                continue
            loads += 1
            saved = re.match(r"s_mov_b32 (s\d+), m0$", lines[k - 3])
            if not saved or lines[k + 1] != "s_mov_b32 m0, " + saved.group(1):
                bad.append(lines[k - 3:k + 2])
    assert loads > 0
    assert not bad, bad[:4]
