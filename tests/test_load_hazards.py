"""CPU: what the compiler made of the loads, in the code objects of the built library.  Those into LDS are written as assembly
(load_to_lds): between a vector instruction that writes a scalar register and a load that reads it the hardware wants five wait
states, and the compiler does not count them in front of these loads."""
import glob
import os
import re
import shutil
import subprocess

import pytest

import paper_2201_13195_amd as rmm

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


def scalars(operand):
    m = re.fullmatch(r"s(?:\[(\d+):(\d+)\]|(\d+))", operand.strip())
    return set() if m is None else set(range(int(m[1]), int(m[2]) + 1)) if m[1] else {int(m[3])}


def written(instruction):
    """Scalar registers that a vector instruction writes."""
    op, _, rest = instruction.partition(" ")
    if not op.startswith("v_"):
        return set()
    operands = rest.split(",")
    two = op.startswith(("v_mad_u64", "v_mad_i64", "v_div_scale")) or "_co_" in op       # (their carry is a second result)
    return set().union(*[scalars(o) for o in operands[:2 if two else 1]])


def early_writes(text):
    """(loads into LDS, those whose scalar registers a vector instruction writes in the five wait states before them), in
    program order."""
    code = [re.sub(r"\s+", " ", line.split("//")[0]).strip() for line in text.split("\n")]
    code = [c for c in code if c and not c.endswith(":")]
    loads = [i for i, c in enumerate(code) if c.startswith("buffer_load") and c.endswith(" lds")]
    bad = []
    for i in loads:
        operands = code[i].split(" ", 1)[1].split(",")
        need, states, j = scalars(operands[1]) | scalars(operands[2].split(" offen")[0]), 0, i - 1
        while states < 5 and j >= 0:
            if written(code[j]) & need:
                bad.append(code[j:i + 1])
                break
            states += int(code[j].split()[1], 0) + 1 if code[j].startswith("s_nop") else 1
            j -= 1
    return len(loads), bad


def test_the_scan_sees_a_write():
    settled = "v_readfirstlane_b32 s10, v1\n s_nop 4\n s_mov_b32 m0, s2\n s_nop 0\n buffer_load_dwordx4 v1, s[8:11], s4 offen lds\n"
    assert early_writes(settled) == (1, [])
    for w in ("v_add_u32 v2, s10, v3", "s_mov_b32 s10, s53", "v_readlane_b32 s9, v9, 3\n s_nop 2", "v_mov_b32 v10, v4"):
        assert early_writes(settled.replace("v_readfirstlane_b32 s10, v1\n s_nop 4", w)) == (1, []), w
    for w in ("v_readlane_b32 s4, v9, 3", "v_mad_u64_u32 v[2:3], s[8:9], v4, v5, 0", "v_readlane_b32 s9, v9, 3\n s_nop 1"):
        assert len(early_writes(settled.replace("s_nop 4", w))[1]) == 1, w


@pytest.fixture(scope="module")
def code(tmp_path_factory):
    """The disassembly of every code object."""
    if not os.path.exists(OBJDUMP):
        pytest.skip("no disassembler")
    where = str(tmp_path_factory.mktemp("objects"))
    shutil.copy(rmm.lib_path(), os.path.join(where, "librmm.so"))
    subprocess.run([OBJDUMP, "--offloading", "librmm.so"], cwd=where, check=True, capture_output=True)
    objects = glob.glob(os.path.join(where, "*gfx950"))
    assert objects
    return [subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", path], capture_output=True, text=True, check=True).stdout for path in objects]


def test_scalar_registers_of_a_load_have_settled(code):
    total = 0
    for text in code:
        loads, bad = early_writes(text)
        assert not bad, (len(bad), bad[0])
        total += loads
    assert total > 1000


def test_a_sketch_tile_asks_for_its_operand_before_it_generates(code):
    """The loads of a tile's first step stand in front of the generator's first multiplication."""
    kernels = [(name, body) for text in code for name, body in re.findall(r"<(\S*sketch_kernel\S*)>:\n(.*?)(?=\n\n|\Z)", text, re.S)]
    assert len(kernels) == 12
    for name, body in kernels:
        columns = int(re.search(r"ShapeILi\d+ELi(\d+)E", name)[1])
        before = body[:re.search(r"v_mad_u64_u32 (\S+ ){4}0\b", body).start()]        # (with a third operand they make addresses)
        assert before.count(" lds") == columns // 64, name          # 1 KB each, of 64 tokens, from eight waves


def loops(body):
    """The text of the loops of a kernel that are up to 1500 instructions long."""
    lines = [line for line in body.split("\n") if "//" in line]
    at = [int(line.split("//")[1].split(":")[0], 16) for line in lines]
    for i, line in enumerate(lines):
        back = re.match(r"\s*s_cbranch\S+ (\d+)", line)
        if back and int(back[1]) >= 1 << 15:
            start = at[i] + 4 + 4 * (int(back[1]) - (1 << 16))
            if start in at and i - at.index(start) < 1500:
                yield "\n".join(lines[at.index(start):i])


def test_a_plain_tile_keeps_a_request_in_flight(code):
    """No step of a loop over tiles waits for every load: the newer of the two requests would be waited for right behind its issue."""
    total = 0
    for text in code:
        for name, body in re.findall(r"<(\S*plain_(?:pass|tn)_kernel\S*)>:\n(.*?)(?=\n\n|\Z)", text, re.S):
            for loop in loops(body):
                if "v_mfma" in loop and "buffer_load" in loop:
                    assert "vmcnt(0)" not in loop, name
                    total += 1
    assert total >= 20


def test_an_fp32_tile_of_columns_waits_for_no_load_between_its_products_and_the_barrier(code):
    kernels = [(name, body) for text in code
               for name, body in re.findall(r"<(\S*plain_tn_kernelIffNS\S*PlainShapeILi32E\S*)>:\n(.*?)(?=\n\n|\Z)", text, re.S)]
    assert len(kernels) >= 2
    for name, body in kernels:
        marks = re.findall(r"v_mfma|buffer_load|vmcnt|s_barrier", body)
        assert not re.search(r"v_mfma(vmcnt)+s_barrier", "".join(marks)), name
        assert marks.count("s_barrier") >= 4
