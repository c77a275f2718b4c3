"""What the compiler made of the kernels, read from the code objects of the library that was built here."""
import os
import re
import struct
import subprocess

import pytest

from paper_2601_12150_amd import build as nb_build

READELF, OBJDUMP = "/opt/rocm/llvm/bin/llvm-readelf", "/opt/rocm/llvm/bin/llvm-objdump"


def code_objects(tmp_path):
    """Every gfx950 code object in libnsattn.so, as a file."""
    data = open(nb_build.LIB, "rb").read()
    for m in re.finditer(b"\x7fELF", data):
        at = m.start()
        if at == 0 or struct.unpack_from("<H", data, at + 18)[0] != 224:      # EM_AMDGPU
            continue
        shoff, = struct.unpack_from("<Q", data, at + 40)
        shentsize, shnum = struct.unpack_from("<HH", data, at + 58)
        path = tmp_path / ("%d.o" % at)
        path.write_bytes(data[at:at + shoff + shentsize * shnum])
        yield path


def kernels(tmp_path):
    """{kernel name: spilled vector registers}."""
    found = {}
    for path in code_objects(tmp_path):
        notes = subprocess.run([READELF, "--notes", str(path)], stdout=subprocess.PIPE, text=True, check=True).stdout
        for entry in notes.split("- .agpr_count:")[1:]:
            name = re.search(r"\.name:\s+(\S+)", entry).group(1)
            found[name] = int(re.search(r"\.vgpr_spill_count:\s+(\d+)", entry).group(1))
    return found


@pytest.mark.skipif(not (os.path.exists(nb_build.LIB) and os.path.exists(READELF)), reason="needs the built library and llvm-readelf")
def test_no_kernel_spills_vector_registers(tmp_path):
    """The attention kernels count their own memory requests: a reload of a spilled register in a key loop waits for
    every transfer in flight, tile by tile."""
    found = kernels(tmp_path)
    assert sum("attn_sweep_kernel" in n for n in found) == 6 and sum("attn_block16_kernel" in n for n in found) == 3
    assert {n: c for n, c in found.items() if c} == {}


def registers(text):
    """{"v12", "a3", ..} named in a piece of an instruction."""
    found = set()
    for kind, first, last, one in re.findall(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+)\b)", text):
        found.update(kind + str(i) for i in (range(int(first), int(last) + 1) if first else [int(one)]))
    return found


def hazards(lines):
    """Where a disassembly has a v_mfma_f32_16x16x32_bf16 within two wait states of the vector instruction that wrote one of its
    operands, or an instruction other than a product of the same accumulator within eleven of the product whose result it names (the
    wait states that the instruction set's manual asks of the program), over every path through its branches."""
    code, at = [], {}                          # (opcode, operands, target); address -> index
    for ln in lines:
        m = re.match(r"\s+(\w+)\s*(.*?)\s*// ([0-9A-F]{8,}): [0-9A-F ]+(?:<\S+?\+0x([0-9a-f]+)>)?", ln)
        k = re.match(r"([0-9a-f]+) <\S+>:", ln)
        if k:
            start = int(k.group(1), 16)
        elif m:
            at[int(m.group(3), 16)] = len(code)
            code.append((m.group(1), m.group(2), start + int(m.group(4), 16) if m.group(4) else None))
    product = [op == "v_mfma_f32_16x16x32_bf16" for op, _, _ in code]
    split = [ops.split(", ") for _, ops, _ in code]

    def following(i, states):
        """Instructions that may run at most that many wait states after instruction i."""
        todo, seen = [(i, states)], {}
        while todo:
            j, left = todo.pop()
            op, _, target = code[j]
            if j != i:
                left -= 1 + int(split[j][0]) if op == "s_nop" else 1
            if op == "s_endpgm" or left < 0:
                continue
            nxt = ([at[target]] if op.startswith(("s_cbranch", "s_branch")) and target in at else []) + ([] if op == "s_branch" else [j + 1])
            for n in nxt:
                if n < len(code) and seen.get(n, -1) < left:
                    seen[n] = left
                    todo.append((n, left))
        return [n for n, left in seen.items() if left > 0]

    for i, (op, ops, _) in enumerate(code):
        if product[i]:
            result = registers(split[i][0])
            for j in following(i, 11):
                named = registers(code[j][1])
                if named & result and not (product[j] and split[j][0] == split[i][0] and not registers(split[j][1] + " " + split[j][2]) & result):
                    yield "%s %s: its result is named by %s %s" % (op, ops, code[j][0], code[j][1])
        elif op.startswith("v_") and not op.startswith(("v_cmp", "v_readfirstlane", "v_readlane")):
            written = registers(split[i][0] + (" " + split[i][1] if "swap" in op else ""))
            for j in following(i, 2):
                if product[j] and written & registers(code[j][1]):
                    yield "%s %s: written right before %s %s" % (op, ops, code[j][0], code[j][1])


PRODUCT = "\tv_mfma_f32_16x16x32_bf16 a[0:3], v[4:7], v[8:11], a[0:3]"
CASES = [  # instructions around a product, and whether they are a fault
    (["\tv_mov_b32_e32 v9, v20", PRODUCT], True), (["\tv_mov_b32_e32 v9, v20", "\ts_nop 0", PRODUCT], True),
    (["\tv_mov_b32_e32 v9, v20", "\ts_nop 1", PRODUCT], False), (["\tv_accvgpr_write_b32 a3, 0", PRODUCT], True),
    (["\tds_read_b128 v[4:7], v30", "\ts_waitcnt lgkmcnt(0)", PRODUCT], False), ([PRODUCT, PRODUCT], False),
    ([PRODUCT, "\ts_nop 9", "\tv_accvgpr_read_b32 v1, a2"], True), ([PRODUCT, "\ts_nop 10", "\tv_accvgpr_read_b32 v1, a2"], False),
    ([PRODUCT, "\ts_nop 3", "\tds_write_b128 v1, a[0:3]"], True), ([PRODUCT, "\tv_mov_b32_e32 v4, v20"], False),
]


@pytest.mark.parametrize("lines,fault", CASES)
def test_hazards_are_found(lines, fault):
    text = ["0000000000000100 <k>:"] + ["%s // %012X: 00000000" % (ln, 256 + 4 * i) for i, ln in enumerate(lines + ["\ts_endpgm"])]
    assert bool(list(hazards(text))) == fault


def test_hazards_across_a_loops_end_are_found():
    lines = [PRODUCT, "\tv_mov_b32_e32 v30, v31", "\tv_mov_b32_e32 v8, v31", "\ts_cbranch_scc1 65532"]
    text = ["0000000000000100 <k>:"] + ["%s // %012X: BF85FFFC%s" % (ln, 256 + 4 * i, " <k+0x0>" if "branch" in ln else "") for i, ln in enumerate(lines)]
    assert list(hazards(text))


@pytest.mark.skipif(not (os.path.exists(nb_build.LIB) and os.path.exists(OBJDUMP)), reason="needs the built library and llvm-objdump")
def test_products_written_in_asm_keep_their_distance(tmp_path):
    """The 256 x 256 linear maps' products are asm, for which the compiler pads nothing: no move of an operand may stand right before one,
    inside the loop or in the slices behind it, and nothing may touch a result that is on its way."""
    for path in code_objects(tmp_path):
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(path)], stdout=subprocess.PIPE, text=True, check=True).stdout
        if "gemm256_bf16_kernel" in text:
            assert text.count("v_mfma_f32_16x16x32_bf16") > 20000
            assert list(hazards(text.splitlines())) == []
            return
    assert False, "no code object with the kernel"
