"""The FP8 products of the 256-column tiles are asm statements, which the compiler does not know as matrix instructions: it keeps no
distance between them and other instructions that touch their registers.  What is built is therefore looked at: no other instruction
reads or writes an accumulator within 18 wait states of a product that writes it, no vector instruction writes an operand within two
in front of one, and nothing is spilled (a spill would be such an instruction, wherever the compiler puts it)."""
import os
import re
import subprocess

import pytest

from paper_2409_11155_amd import build

PRODUCT = "v_mfma_f32_16x16x128_f8f6f4"
BEHIND, IN_FRONT = 18, 2


def registers(operands):
    """Vector registers named in an operand list."""
    found = set()
    for a, lo, hi in re.findall(r"\bv(?:(\d+)\b|\[(\d+):(\d+)\])", operands):
        found |= {int(a)} if a else set(range(int(lo), int(hi) + 1))
    return found


def findings(lines):
    """Places where an instruction comes too close to a product, over every path of `lines` (one kernel's instructions)."""
    code, at_label = [], {}
    for line in lines:
        line = line.split(";")[0].strip()
        if re.match(r"[.\w$]+:$", line):
            at_label[line[:-1]] = len(code)
        elif line and not line.startswith("."):
            op, _, rest = line.partition(" ")
            operands = [o for o in re.split(r",\s*(?![^\[]*\])", rest)]
            code.append((op, rest.strip(), registers(operands[0]), set().union(*(registers(o) for o in operands[1:])) if operands[1:] else set()))
    bad, done = [], set()

    def scan(start, product, vector, limit):
        """`product`, `vector`: wait states since a product / another vector instruction wrote a register."""
        for n, (op, rest, first, others) in enumerate(code[start:start + limit]):
            if op == PRODUCT:
                near = {r for r in first | others if vector.get(r, 99) < IN_FRONT}
            else:
                near = {r for r in first | others if product.get(r, 99) < BEHIND}
            if near:
                bad.append((start + n, op, rest, sorted(near)))
            step = int(rest) + 1 if op == "s_nop" else 1
            product = {r: a + step for r, a in product.items() if a + step < BEHIND}
            vector = {r: a + step for r, a in vector.items() if a + step < IN_FRONT}
            if op == PRODUCT:
                product.update({r: 0 for r in first})
            elif op.startswith("v_"):
                vector.update({r: 0 for r in first})
            if op.startswith(("s_cbranch", "s_branch")) and (start + n) not in done:
                done.add(start + n)
                scan(at_label[rest], product, vector, BEHIND + 1)
            if op in ("s_endpgm", "s_branch"):
                product, vector = {}, {}

    scan(0, {}, {}, len(code))
    return bad


def test_the_check_finds_what_it_looks_for():
    product = PRODUCT + " v[0:3], v[8:15], v[16:23], v[0:3]"
    assert not findings([product, product, "s_nop 15", "s_nop 1", "v_mul_f32 v0, v1, v2"])
    assert not findings(["v_mov_b32 v8, v30", "s_nop 1", product])
    for code in ([product, "s_nop 15", "v_mul_f32 v40, v1, v2"], [product, "v_mov_b32 v3, 0"], ["v_mov_b32 v9, v30", product],
                 [product, "ds_write_b128 v50, v[0:3]"], [product, "scratch_store_dword off, v2, off"],
                 [".L1:", "v_add_f32 v40, v0, v0", "s_nop 7", product, "s_cbranch_scc0 .L1", "s_endpgm"]):
        assert findings(code), code


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("isa") / "gemm_pp.s")
    subprocess.run([build.hipcc(), *build.DEVICE_FLAGS, "--offload-device-only", "-S", "-o", out, os.path.join(build.CSRC, "gemm_pp.hip")],
                   check=True, capture_output=True)
    with open(out) as f:
        return f.read()


def test_nothing_comes_near_the_accumulators_of_the_fp8_products(assembly):
    kernels = {}
    for m in re.finditer(r"^(\w*gemm_pp_kernel\w*):.*?^\.Lfunc_end\d+:", assembly, re.S | re.M):
        if PRODUCT in m.group(0):
            kernels[m.group(1)] = m.group(0).splitlines()[1:-1]
    assert len(kernels) == 18                     # three heights, six epilogues
    for name, lines in kernels.items():
        assert findings(lines) == [], name


def test_the_tiles_spill_nothing(assembly):
    spills = re.findall(r"\.name:\s+(\S*gemm_pp_kernel\S*)\n(?:.*\n)*?\s+\.vgpr_spill_count:\s+(\d+)", assembly)
    assert len(spills) == 36
    assert {n: int(c) for n, c in spills if int(c)} == {}
