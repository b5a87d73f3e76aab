"""Wait states of the LDS DMAs in the built library.

An LDS DMA takes its LDS address from M0, and the ISA asks for one wait state between a scalar write
of M0 and the DMA; a vector-memory instruction that takes its base from scalar registers needs five
after a vector instruction wrote them.  The hardware checks neither, and the compiler inserts no wait
states inside inline assembly, so the disassembly is checked here."""
import os
import re
import shutil
import subprocess

import pytest

import paper_2608_16157_amd as ftm

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
DMA = re.compile(r"(global|buffer)_load\S*_lds_|buffer_load\S* .*\blds\b")


@pytest.fixture(scope="module")
def instructions(tmp_path_factory):
    """The instructions of every gfx950 kernel of the library, in layout order."""
    d = tmp_path_factory.mktemp("dis")
    lib = shutil.copy(os.environ.get("FTMOE_LIBRARY", ftm.LIB_PATH), d / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", lib], check=True, capture_output=True, cwd=d)
    text = []
    for obj in sorted(d.glob("lib.so.*gfx950")):
        out = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", obj], check=True, capture_output=True, text=True).stdout
        # a line of a kernel's name, "0000 <name>:", or of an instruction
        text += [line.split("//")[0].strip() for line in out.splitlines() if line.startswith("\t") or line.endswith(">:")]
    assert sum(bool(DMA.match(t)) for t in text) > 1000   # the GEMV's and the GEMM's DMAs are all there
    return text


def sgprs(operand):
    """Numbers of the scalar registers of one operand."""
    if m := re.fullmatch(r"s(\d+)", operand):
        return {int(m[1])}
    if m := re.fullmatch(r"s\[(\d+):(\d+)\]", operand):
        return set(range(int(m[1]), int(m[2]) + 1))
    return set()


def operands(text):
    return [t.strip() for t in text.split(None, 1)[1].split(",")] if " " in text else []


def wait_states(text):
    return int(text.split()[1], 0) + 1 if text.startswith("s_nop") else 1


def test_m0_write_is_not_adjacent(instructions):
    bad = [i for i in range(1, len(instructions))
           if DMA.match(instructions[i]) and re.match(r"s_\w+ m0,", instructions[i - 1])]
    assert not bad, f"{len(bad)} LDS DMAs directly behind a write of M0, the first: {instructions[bad[0] - 1:bad[0] + 1]}"


def test_m0_belongs_to_the_assembly_dmas(instructions):
    """The assembly cannot declare M0 as clobbered, so in the kernels that hold it nothing but the DMAs,
    each with a write of its own, uses M0."""
    kernel, seen = "", 0
    for i, text in enumerate(instructions):
        if text.endswith(">:"):
            kernel = text
        elif "grouped_gemm" in kernel or "skinny_gemm" in kernel:
            if DMA.match(text):
                assert re.match(r"s_mov_b32 m0,", instructions[i - 2]) and instructions[i - 1] == "s_nop 0", (kernel, text)
                seen += 1
            elif re.search(r"\bm0\b", text):
                assert DMA.match(instructions[i + 2]), (kernel, text)
            else:
                assert not re.match(r"ds_gws|s_sendmsg|s_movrel|ds_\w+_addtid", text), (kernel, text)
    assert seen > 1000


def test_scalar_base_is_settled(instructions):
    bad = []
    for i, text in enumerate(instructions):
        if not DMA.match(text):
            continue
        base = set().union(*(sgprs(o.split()[0]) for o in operands(text) if o))
        states, j = 0, i - 1
        while base and j >= 0 and states < 5:
            prev = instructions[j]
            if prev.startswith("v_"):
                # the destination and, where there is one, the carry-out
                n_dest = 2 if re.match(r"v_(mad_[iu]64|add_co|sub_co|addc|subb|div_scale)", prev) else 1
                if any(base & sgprs(o) for o in operands(prev)[:n_dest]):
                    bad.append((prev, text))
                    break
            states += wait_states(prev)
            j -= 1
    assert not bad, f"{len(bad)} LDS DMAs whose base a vector instruction wrote just before, the first: {bad[0]}"
