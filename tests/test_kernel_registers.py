"""Register use of the product kernels in the built library, from its own code objects' metadata and instructions (no GPU)."""
import os
import re
import subprocess
import struct

import msgpack
import pytest

import paper_2503_02550_amd as S

LIB = os.path.join(os.path.dirname(S.__file__), "libspecinf.so")


def _notes(elf):
    """The metadata maps of an ELF code object's notes."""
    shoff, = struct.unpack_from("<Q", elf, 40)
    entsize, count = struct.unpack_from("<HH", elf, 58)
    for i in range(count):
        kind, _, _, at, size = struct.unpack_from("<IQQQQ", elf, shoff + i * entsize + 4)
        end = at + size
        while kind == 7 and at < end:      # SHT_NOTE
            namesz, descsz, note = struct.unpack_from("<III", elf, at)
            desc = at + 12 + (namesz + 3) // 4 * 4
            if note == 32:                 # AMDGPU metadata, MessagePack
                yield msgpack.unpackb(elf[desc:desc + descsz], strict_map_key=False)
            at = desc + (descsz + 3) // 4 * 4


def _code_objects():
    with open(LIB, "rb") as f:
        lib = f.read()
    magic, at = b"__CLANG_OFFLOAD_BUNDLE__", 0
    while (at := lib.find(magic, at)) >= 0:
        n, = struct.unpack_from("<Q", lib, at + len(magic))
        pos = at + len(magic) + 8
        for _ in range(n if n < 16 else 0):
            off, size, name = struct.unpack_from("<QQQ", lib, pos)
            if b"gfx950" in lib[pos + 24:pos + 24 + name] and size:
                yield lib[at + off:at + off + size]
            pos += 24 + name
        at += len(magic)


def _kernels():
    return {k[".name"]: k for elf in _code_objects() for notes in _notes(elf) for k in notes["amdhsa.kernels"]}


@pytest.mark.parametrize("kernel", ["gemm_ring_kernel", "gemm_fed_kernel", "gemm_pp_kernel"])
def test_product_kernels_leave_room_for_the_bubbles_wait(kernel):
    """Two of their wavefronts on a SIMD and the one that waits for the bubble's end share its 512 registers, so a block of
    any product runs on the CU that holds that wait; and none is kept in scratch memory (a reload inside the main loop waits
    for every fetch in flight)."""
    kernels = _kernels()
    wait = max(k[".vgpr_count"] for n, k in kernels.items() if "bubble" in n)
    found = {n: k for n, k in kernels.items() if kernel in n}
    assert len(found) >= 4
    for name, k in found.items():
        granule = lambda r: (r + 7) // 8 * 8
        assert 2 * granule(k[".vgpr_count"]) + granule(wait) <= 512, (name, k[".vgpr_count"], wait)
        assert k[".vgpr_spill_count"] == 0, name


def test_only_the_fetches_use_m0(tmp_path):
    """The fetch into LDS is an assembly statement that writes M0.  The compiler reserves that register and cannot be told
    of the write; it would set M0 itself right before an instruction that reads it, and a fetch could come to stand between
    the two.  So no kernel with such fetches may contain another use of M0."""
    objdump = "/opt/rocm/llvm/bin/llvm-objdump"
    if not os.path.exists(objdump):
        pytest.skip("no disassembler")
    fetches = 0
    for i, elf in enumerate(_code_objects()):
        if b"gemm_ring_kernel" not in elf:
            continue
        (tmp_path / f"{i}.co").write_bytes(elf)
        text = subprocess.run([objdump, "-d", "--no-show-raw-insn", "--mcpu=gfx950", tmp_path / f"{i}.co"], capture_output=True, text=True, check=True).stdout
        for part in re.split(r"\n[0-9a-f]+ <", text)[1:]:
            name, body = part.split(">:\n", 1)
            code = [line.split("//")[0].strip() for line in body.splitlines()]
            for k, line in enumerate(code):
                if "m0" in line:
                    assert re.match(r"s_mov_b32 m0, s\d+$", line) and code[k + 1] == "s_nop 0" and re.match(r"buffer_load_dwordx4 .* lds$", code[k + 2]), (name, code[k:k + 3])
                    fetches += 1
    assert fetches > 100


def _kernel_code(tmp_path, having, comments=False):
    """(name, instructions) of every kernel in the code objects that hold `having`; comments: with their addresses behind them."""
    objdump = "/opt/rocm/llvm/bin/llvm-objdump"
    if not os.path.exists(objdump):
        pytest.skip("no disassembler")
    for i, elf in enumerate(_code_objects()):
        if having not in elf:
            continue
        (tmp_path / f"{i}.co").write_bytes(elf)
        text = subprocess.run([objdump, "-d", "--no-show-raw-insn", "--mcpu=gfx950", tmp_path / f"{i}.co"], capture_output=True, text=True, check=True).stdout
        for part in re.split(r"\n[0-9a-f]+ <", text)[1:]:
            name, body = part.split(">:\n", 1)
            yield name, [line.strip() if comments else line.split("//")[0].strip() for line in body.splitlines()]


def _reached(code, successors, begin, without=()):
    """The instructions that can follow one of `begin`, on paths that touch none of `without`."""
    seen, todo = set(), [j for i in begin for j in successors[i]]
    while todo:
        i = todo.pop()
        if i not in seen and i not in without:
            seen.add(i)
            todo += successors[i]
    return seen


def test_product_kernels_stamp_their_end_behind_their_results(tmp_path):
    """The end of a launch is the clock read behind the block's results.  On no path from a fetch of operands to that read (a clock
    read that a count of blocks leads to) may a wavefront be without a barrier that the stores of the results lead to: those that
    only fetch wait there for the others."""
    kernels = 0
    for name, code in _kernel_code(tmp_path, b"gemm_ring_kernel", comments=True):
        if not re.search("gemm_(ring|fed|pp)_kernel", name) or not any(line.startswith("buffer_store") for line in code):
            continue                       # (the rare epilogues store to plain addresses; their kernels are the same otherwise)
        at = {int(re.search(r"// ([0-9A-F]+):", line)[1], 16): i for i, line in enumerate(code) if "// " in line}
        first = min(at)
        successors = []
        for i, line in enumerate(code):
            to = re.search(r"<\S+?(?:\+0x([0-9a-f]+))?>$", line) if re.match("s_c?branch", line) else None
            successors.append([] if line.startswith("s_endpgm") else ([i + 1] if not line.startswith("s_branch") and i + 1 < len(code) else []) + ([at[first + int(to[1] or "0", 16)]] if to else []))
        having = lambda pattern: [i for i, line in enumerate(code) if re.match(pattern, line)]      # noqa: E731
        counts = [i for i in having(r"(global|flat)_atomic_add v.* sc0 ") if any("0x801" in line for line in code[max(0, i - 24):i])]
        ends = set(having("s_memrealtime")) & _reached(code, successors, counts)
        barriers = set(having("s_barrier")) & _reached(code, successors, having("buffer_store"))
        assert counts and ends, name
        assert not ends & _reached(code, successors, having(r"buffer_load_dwordx4 .* lds"), without=barriers), name
        kernels += 1
    assert kernels >= 40


def test_block_0_is_counted_behind_the_words_it_left(tmp_path):
    """Block 0 takes a kernel's start off the sum of the times, and the block found to be the last reads that sum.  So the count of a
    block (the atomic whose counter is chosen by the number of blocks, 0x801 being the border between two levels) stands behind a
    wait for everything outstanding, under a branch on the block's number."""
    counts = 0
    for name, code in _kernel_code(tmp_path, b"gfx950"):
        if not any(line.startswith("global_atomic_add_x2") for line in code):
            continue
        for i, line in enumerate(code):
            window = code[max(0, i - 32):i]
            if re.match(r"(global|flat)_atomic_add v.* sc0$", line) and any(re.match(r"s_cmpk_\w+ s\d+, 0x801$", w) for w in window[-24:]):
                assert any(re.match(r"s_cmp_\w+ s\d+, 0$", a) and b.startswith("s_cbranch") and w == "s_waitcnt vmcnt(0)"
                           for a, b, w in zip(window, window[1:], window[2:])), (name, window)
                counts += 1
    assert counts > 100
