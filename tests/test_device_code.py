"""What the compiler made of the kernels, read from the library as built: the instructions and the resources that correctness or
speed rest on and that no test of results would show.  Needs no GPU."""
import os
import re
import struct
import subprocess

import pytest

from paper_2507_01004_amd import zeco

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


def code_objects():
    """The gfx950 code objects in the library, one per source file with kernels."""
    if not os.path.exists(zeco.LIB_PATH):
        from paper_2507_01004_amd.build import build_lib
        build_lib()
    data = open(zeco.LIB_PATH, "rb").read()
    out = []
    for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", data):
        entries, at = struct.unpack_from("<Q", data, m.start() + 24)[0], m.start() + 32
        for _ in range(entries):
            offset, size, n = struct.unpack_from("<QQQ", data, at)
            if b"gfx950" in data[at + 24:at + 24 + n]:
                out.append(data[m.start() + offset:m.start() + offset + size])
            at += 24 + n
    assert out
    return out


def kernels():
    """Name -> metadata of every kernel in the library (the ELF note the runtime itself launches by)."""
    msgpack = pytest.importorskip("msgpack")
    out = {}
    for obj in code_objects():
        table, = struct.unpack_from("<Q", obj, 0x28)
        size, count = struct.unpack_from("<HH", obj, 0x3a)
        for at in range(table, table + size * count, size):
            kind, = struct.unpack_from("<I", obj, at + 4)
            offset, = struct.unpack_from("<Q", obj, at + 24)
            if kind == 7:   # SHT_NOTE: one note, name padded to four bytes
                name, desc = struct.unpack_from("<II", obj, offset)
                start = offset + 12 + (name + 3) // 4 * 4
                for k in msgpack.unpackb(obj[start:start + desc], strict_map_key=False)["amdhsa.kernels"]:
                    out[k[".name"]] = k
    assert out
    return out


def instructions(obj, path):
    """(kernel, mnemonic, operands) of every instruction of a code object."""
    path.write_bytes(obj)
    text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(path)], check=True, capture_output=True, text=True).stdout
    kernel = None
    for line in text.splitlines():
        if line.endswith(">:"):
            kernel = line.split("<")[1][:-2]
        elif line.startswith("\t"):
            yield (kernel,) + tuple((line.split("//")[0].strip() + " ").split(" ", 1))


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no disassembler")
def test_fetches_to_lds_wait_for_their_base(tmp_path):
    """A vector-memory instruction may read a scalar register five wait states after a vector instruction wrote it, and the compiler,
    which restores scalars from vector lanes, does not know of the loads inside an asm block: each has to bring the wait along, or
    share the base of a load just before it."""
    seen = 0
    for obj in code_objects():
        before = []
        for _, op, args in instructions(obj, tmp_path / "code.elf"):
            if op.startswith("global_load_lds"):
                seen += 1
                base = args.split(",")[1].strip()
                assert before[-1][0] == "s_nop"
                if before[-2][0] == "s_mov_b32":   # first of a group
                    assert before[-2][1].startswith("m0") and int(before[-1][1]) >= 3
                else:
                    assert before[-2][0] == "s_add_u32" and before[-2][1].startswith("m0")
                    assert before[-3][0].startswith("v_add_u32")
                    assert before[-4][0].startswith("global_load_lds") and before[-4][1].split(",")[1].strip() == base
            before = (before + [(op, args)])[-4:]
    assert seen > 0


def test_chunk_kernels_keep_their_registers():
    """A spilled register of the chunk kernel is reloaded in its loop, and the wait for it is a wait for the rows fetched ahead as well.
    Two or three, saved around the loop's tail, are what the twelve-wave forms need at their 168 registers."""
    spilled = {n: k[".vgpr_spill_count"] for n, k in kernels().items() if "gla_chunk_bf16_kernel" in n}
    assert len(spilled) > 100
    assert {n: v for n, v in spilled.items() if v > 3} == {}


def test_two_workgroups_of_the_narrow_dq_pass_share_a_compute_unit():
    """Six waves of a workgroup on four SIMDs: a second one fits for certain at four waves a SIMD, 128 registers.  (Its LDS is asserted
    at compile time.)"""
    found = [k for n, k in kernels().items() if re.search(r"gla_bwd_bf16_kernelILi64ELi64ELi[12]ELb0ELi[012]ELb0E", n)]
    assert len(found) == 10   # gate layouts, siblings (not with per-head gates), cache hints
    for k in found:
        assert k[".vgpr_count"] <= 128 and k[".vgpr_spill_count"] == 0


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no disassembler")
def test_what_key_channel_siblings_share_is_not_streamed(tmp_path):
    """Two workgroups that own half of the key channels each read the same v, and the same g with one decay per head.  Read with the
    non-temporal hint these come from HBM twice: only the four-byte g and the rows of k are told apart here, by width and number."""
    hinted, plain = {}, {}
    for obj in code_objects():
        for kernel, op, args in instructions(obj, tmp_path / "code.elf"):
            if op.startswith("global_load") and re.search(r"gla_chunk_bf16_kernelILi64ELi\d+ELi1ELi2ELi[13]ELb[01]ELi2EE", kernel):
                (hinted if args.split()[-1] == "nt" else plain).setdefault(kernel, []).append(op)
    assert len(plain) == 8   # two widths of v, forward and backward states, two ranges of gates
    for kernel, ops in plain.items():
        assert set(hinted[kernel]) == {"global_load_dwordx2"}, kernel
        assert len(hinted[kernel]) < ops.count("global_load_dwordx2"), kernel


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no disassembler")
def test_scan_stores_its_end_states_twice_only_where_asked(tmp_path):
    """The second copy of the end states (a forward that saves its states) has kernels of its own: a pointer tested at the end of the
    others would cost every scan its load."""
    stores = {}
    for obj in code_objects():
        for kernel, op, _ in instructions(obj, tmp_path / "code.elf"):
            m = kernel and re.search(r"state_scan_kernelILi(\d+)ELi\d+ELb1ELi0ELb0ELb([01])E", kernel)
            if m and op.startswith("global_store"):
                key = (m.group(1), m.group(2))
                stores[key] = stores.get(key, 0) + 1
    for v in ("4", "2", "1"):
        assert stores[v, "1"] == stores[v, "0"] + 1
