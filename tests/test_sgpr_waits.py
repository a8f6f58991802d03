"""The built kernels keep the wait states gfx950 asks for between a vector instruction that writes a scalar
register and a vector instruction that reads it (two).  The compiler sees to this in its own code but does
not look into inline assembly, so the library's machine code is read back and checked as a whole."""
import os
import re
import shutil
import subprocess

import pytest

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
WAIT_STATES = 2


def scalar_registers(operand):
    """Names of the 32-bit scalar registers an operand stands for."""
    m = re.fullmatch(r"s\[(\d+):(\d+)\]", operand)
    if m:
        return {f"s{i}" for i in range(int(m[1]), int(m[2]) + 1)}
    if re.fullmatch(r"s\d+", operand):
        return {operand}
    return {"vcc": {"vcc_lo", "vcc_hi"}, "vcc_lo": {"vcc_lo"}, "vcc_hi": {"vcc_hi"}}.get(operand, set())


def too_close(lines):
    """Pairs (writer, reader) of vector instructions with fewer wait states between them than needed."""
    recent, found = [], []                      # (instruction, registers it wrote, wait states since)
    for line in lines:
        text = line.split("//")[0].strip()
        if not text or text.endswith(":"):
            continue
        name, _, rest = text.partition(" ")
        if name in ("s_branch", "s_endpgm", "s_setpc_b64"):     # what follows is not reached from here
            recent = []
            continue
        ops = [o.strip() for o in rest.split(",")]
        vector = name.startswith("v_")
        if vector:
            two = name.startswith(("v_add_co", "v_sub_co", "v_subrev_co", "v_addc_co", "v_subb_co", "v_div_scale",
                                   "v_mad_u64", "v_mad_i64"))   # a vector result, then a scalar one
            read = set().union(*(scalar_registers(o.split(" ")[0]) for o in ops[2 if two else 1:]), set())
            found += [(w, text) for w, regs, gap in recent if gap < WAIT_STATES and regs & read]
        states = int(ops[0], 0) + 1 if name == "s_nop" else 1
        recent = [(w, r, g + states) for w, r, g in recent if g + states < WAIT_STATES]
        if vector:
            wrote = scalar_registers(ops[0]) | (scalar_registers(ops[1]) if two else set())
            if wrote:
                recent.append((text, wrote, 0))
    return found


def test_the_check_sees_a_missing_wait():
    pair = ["v_readlane_b32 s7, v1, s2", "v_cndmask_b32_e64 v0, v1, v2, s[6:7]"]
    assert len(too_close(pair)) == 1
    assert len(too_close([pair[0], "s_nop 0", pair[1]])) == 1
    assert not too_close([pair[0], "s_nop 1", pair[1]])
    assert not too_close([pair[0], "s_add_u32 s1, s1, 1", "v_mov_b32_e32 v9, v8", pair[1]])
    assert not too_close([pair[0], "s_add_u32 s6, s7, 1"])           # scalar readers are interlocked


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no disassembler")
def test_vector_reads_of_scalar_registers_wait_for_vector_writes(tmp_path):
    from paper_2206_04746_amd import binding
    lib = shutil.copy(binding.LIB_PATH, tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", str(lib)], cwd=tmp_path, check=True, capture_output=True)
    objects = sorted(tmp_path.glob("lib.so.*gfx950"))
    assert objects
    readers = 0
    for obj in objects:
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--no-leading-addr", str(obj)], check=True,
                              capture_output=True, text=True).stdout
        kernel = ""
        for part in re.split(r"\n(?=<[^>]+>:)", text):
            kernel = part.split("\n", 1)[0]
            readers += part.count("v_cndmask")
            close = too_close(part.split("\n")[1:])
            assert not close, (kernel, len(close), close[0])
    assert readers > 100                          # the parser reads what it thinks it reads
