"""The device code of the built library: what its sources rely on and no compiler checks.

Wait states.  The compiler does not look into an inline assembly statement when it places them.  The CDNA instruction set asks
for five between a vector instruction that writes a scalar register (v_readfirstlane, v_cmp) and a memory instruction that reads
it; with fewer the memory instruction may take the register's old value, here the address of a copy into LDS.

LDS addresses.  The staged gather's multi-probe form reads its rows at addresses counted from zero (it flips their bits), so the
dynamic LDS must start there: the kernel has no static one.
"""
import re
import shutil
import struct
import subprocess

import pytest

from paper_2403_07221_amd import build

OBJDUMP = shutil.which("llvm-objdump") or "/opt/rocm/lib/llvm/bin/llvm-objdump"
READELF = shutil.which("llvm-readelf") or "/opt/rocm/lib/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"
VALU_TO_VMEM = 5  # wait states

SGPRS = re.compile(r"\bs\[(\d+):(\d+)\]|\bs(\d+)\b|\b(vcc)\b")


def sgprs(operands):
    regs = set()
    for first, last, one, vcc in SGPRS.findall(operands):
        if vcc:
            regs.add("vcc")
        elif one:
            regs.add(int(one))
        else:
            regs |= set(range(int(first), int(last) + 1))
    return regs


def scalar_results(op, operands):
    """Scalar registers that the vector instruction writes."""
    if op.startswith(("v_readfirstlane", "v_readlane", "v_cmp")):
        return sgprs(operands[0])
    if "_co_" in op or op.startswith("v_div_scale"):
        return sgprs(operands[1])
    return set()


def code_objects():
    data = build.LIB.read_bytes()
    at = data.find(MAGIC)
    while at >= 0:
        (count,) = struct.unpack_from("<Q", data, at + len(MAGIC))
        entry = at + len(MAGIC) + 8
        for _ in range(count):
            offset, size, name = struct.unpack_from("<QQQ", data, entry)
            if b"gfx950" in data[entry + 24:entry + 24 + name]:
                yield data[at + offset:at + offset + size]
            entry += 24 + name
        at = data.find(MAGIC, at + 1)


def too_early(listing):
    """Memory instructions that read a scalar register sooner than VALU_TO_VMEM wait states after a vector instruction wrote it,
    following the code in the order it stands."""
    kernel, recent, found = "", [], []   # recent: (registers written, wait states of the instruction), newest last
    for line in listing.splitlines():
        if line.endswith(">:"):
            kernel = line.split("<")[1][:-2]
            recent = []
            continue
        text = line.split("//")[0].strip()
        if not text or not line.startswith("\t"):
            continue
        op, _, rest = text.partition(" ")
        operands = [o.strip() for o in rest.split(",")]
        if op.startswith(("global_", "buffer_", "flat_")):
            reads, states = sgprs(rest), 0
            for written, waits in reversed(recent):
                if states >= VALU_TO_VMEM:
                    break
                if written & reads:
                    found.append(f"{kernel}: {text} after {states} wait states")
                    break
                states += waits
        recent.append((scalar_results(op, operands) if op.startswith("v_") else set(), int(rest, 0) + 1 if op == "s_nop" else 1))
        del recent[:-VALU_TO_VMEM - 1]
    return found


def test_the_check_sees_a_missing_wait():
    head = "0000000000001000 <kernel>:\n\tv_readfirstlane_b32 s8, v1\n\ts_mov_b32 m0, s9\n"
    load = "\tglobal_load_lds_dwordx4 v46, s[8:9]\n"
    assert len(too_early(head + "\ts_nop 1\n" + load)) == 1
    assert len(too_early(head + "\ts_nop 2\n" + load)) == 1
    assert too_early(head + "\ts_nop 3\n" + load) == []
    assert too_early(head + "\tglobal_load_lds_dwordx4 v46, s[10:11]\n") == []


@pytest.mark.skipif(not shutil.which(OBJDUMP), reason="llvm-objdump not found")
def test_memory_instructions_wait_for_their_scalar_operands(tmp_path):
    objects = list(code_objects())
    assert len(objects) == build.N_PARTS
    copies = 0
    for i, code in enumerate(objects):
        path = tmp_path / f"{i}.co"
        path.write_bytes(code)
        listing = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(path)], capture_output=True, text=True, check=True).stdout
        copies += listing.count("global_load_lds")
        assert too_early(listing) == []
    assert copies > 100


@pytest.mark.skipif(not shutil.which(READELF), reason="llvm-readelf not found")
def test_staged_gather_has_no_static_lds(tmp_path):
    sizes = []
    for i, code in enumerate(code_objects()):
        path = tmp_path / f"{i}.co"
        path.write_bytes(code)
        notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
        sizes += [int(size) for size, name in re.findall(r"\.group_segment_fixed_size: (\d+).*?\.name: +(_Z\w+)", notes, re.S)
                  if "gather_lds_kernel" in name]
    assert len(sizes) > 100 and set(sizes) == {0}


@pytest.mark.skipif(not shutil.which(READELF), reason="llvm-readelf not found")
def test_deep_direct_gather_is_built_as_it_is_launched(tmp_path):
    """(row type, row pieces a token, mode, depth): weighted at either depth for every row type, plain for fp32 rows."""
    path, forms = tmp_path / "a.co", set()
    for code in code_objects():
        path.write_bytes(code)
        notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
        forms |= {tuple(map(int, m)) for m in re.findall(r"_ZN4lffn13gather_kernelILi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)EEE", notes)}
    deep = {f for f in forms if f[3]}
    assert deep == {(t, w, 1, d) for t in (0, 1, 2) for w in (4, 8, 16) for d in (8, 16)} | {(0, w, 0, 16) for w in (4, 8, 16)}
