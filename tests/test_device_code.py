"""The device code of the built library, disassembled: what the compiler leaves to chance on gfx950.

A store of more than 8 bytes to a lane reads its data registers after it is issued, and a vector instruction that comes too soon can
replace them.  The compiler leaves two wait states in between, but none after a buffer store with an offset in a scalar
register, where this chip needs them too: values of 16 lanes then come from what the register held next."""
import os
import re
import shutil
import struct
import subprocess

import pytest

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2409_12517_amd", "libssg.so")
OBJDUMP = shutil.which("llvm-objdump") or "/opt/rocm/llvm/bin/llvm-objdump"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"
WAIT_STATES = 2


def code_objects(path):
    """The gfx950 code objects in a library's offload bundles: magic, count, then (offset, size, name length, name) of each."""
    data = open(path, "rb").read()
    at = data.find(MAGIC)
    while at >= 0:
        pos = at + len(MAGIC)
        (count,) = struct.unpack_from("<Q", data, pos)
        pos += 8
        for _ in range(count):
            offset, size, n = struct.unpack_from("<QQQ", data, pos)
            name = data[pos + 24:pos + 24 + n].decode()
            pos += 24 + n
            if name.endswith("gfx950") and size:
                yield data[at + offset:at + offset + size]
        at = data.find(MAGIC, at + len(MAGIC))


def registers(operand):
    """The vector registers of an operand such as v7, v[4:7] or a[0:3] (accumulation registers); empty: something else."""
    m = re.fullmatch(r"([va])(?:(\d+)|\[(\d+):(\d+)\])", operand)
    if not m:
        return set()
    numbers = [int(m[2])] if m[2] else range(int(m[3]), int(m[4]) + 1)
    return {(m[1], n) for n in numbers}


def early_overwrites(lines):
    """(store, overwriting instruction) pairs that are fewer than WAIT_STATES apart, in order of the listing."""
    found, open_stores = [], []                               # open: [store, its data registers, wait states left]
    for line in lines:
        m = re.match(r"\s+([a-z]\w+)\s*([^/]*)", line)
        if not m:
            if line.rstrip().endswith(":"):                   # another function
                open_stores = []
            continue
        op, operands = m[1], [x.strip() for x in m[2].strip().split(",")]
        if op.startswith("v_"):
            written = registers(operands[0].split()[0]) if operands[0] else set()
            found += [(s, line.strip()) for s, data, _ in open_stores if data & written]
        states = int(operands[0], 0) + 1 if op == "s_nop" else 1
        open_stores = [(s, data, left - states) for s, data, left in open_stores if left > states]
        if re.fullmatch(r"(buffer|global|flat|scratch)_store_dwordx[34]", op):
            data = registers(operands[0] if op.startswith("buffer") else operands[1])
            open_stores.append((line.strip(), data, WAIT_STATES))
    return found


def test_finder():
    scalar = "\tbuffer_store_dwordx4 v[2:5], v6, s[0:3], s10 offen sc1 // 000"
    assert early_overwrites([scalar, "\tv_add_f32_e32 v3, s4, v2 // 000"])
    assert early_overwrites([scalar, "\ts_add_i32 s1, s1, 4", "\tv_pk_mul_f32 v[4:5], v[8:9], v[10:11]"])
    assert not early_overwrites([scalar, "\tv_add_f32_e32 v6, s4, v2", "\tv_mov_b32_e32 v7, v2", "\tv_mov_b32_e32 v2, v7"])
    assert not early_overwrites([scalar, "\ts_nop 1", "\tv_mov_b32_e32 v2, v7"])
    assert early_overwrites(["\tglobal_store_dwordx4 v[18:19], v[2:5], off", "\tv_mov_b32_e32 v5, v7"])
    assert early_overwrites(["\tglobal_store_dwordx4 v[18:19], a[2:5], off", "\tv_accvgpr_write_b32 a3, v7"])
    assert not early_overwrites(["\tglobal_store_dwordx4 v[18:19], a[2:5], off", "\tv_mov_b32_e32 v3, v7"])
    assert not early_overwrites(["\tglobal_store_dwordx2 v[18:19], v[2:3], off", "\tv_mov_b32_e32 v2, v7"])


def test_no_store_data_is_overwritten_early(tmp_path):
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    objects = list(code_objects(LIB))
    assert objects, "no gfx950 code in the library"
    stores, bad = 0, []
    for i, code in enumerate(objects):
        path = tmp_path / f"{i}.co"
        path.write_bytes(code)
        text = subprocess.run([OBJDUMP, "-d", "--mcpu=gfx950", str(path)], capture_output=True, text=True, check=True).stdout
        lines = text.splitlines()
        stores += sum("_store_dwordx4" in x for x in lines)
        bad += early_overwrites(lines)
    assert stores > 100, "the listing was not understood"
    assert not bad, f"{len(bad)} stores, the first: {bad[0]}"
