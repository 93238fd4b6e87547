"""The built library's own machine code: rules of the target that the compiler keeps for the
instructions it emits and nobody keeps inside inline assembly."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2505_21889_amd import build as B


def objdump():
    for cand in ("/opt/rocm/llvm/bin/llvm-objdump", shutil.which("llvm-objdump")):
        if cand and os.path.exists(cand):
            return cand
    pytest.skip("llvm-objdump not found")


@pytest.fixture(scope="module")
def listing(tmp_path_factory):
    """Disassembly of every gfx950 code object in the library."""
    tool = objdump()
    if not os.path.exists(B.LIB_PATH):
        B.build_library()
    folder = tmp_path_factory.mktemp("code")
    shutil.copy(B.LIB_PATH, folder)
    subprocess.run([tool, "--offloading", os.path.basename(B.LIB_PATH)], cwd=folder, check=True, capture_output=True)
    text = [subprocess.run([tool, "-d", "--no-show-raw-insn", name], cwd=folder, check=True, capture_output=True,
                           text=True).stdout
            for name in sorted(os.listdir(folder)) if name.endswith("gfx950")]
    assert any("extend_attention_kernel" in t for t in text)
    return "\n".join(text)


def scalar_registers(operand):
    """Scalar register numbers that an operand names (vcc as two numbers of its own)."""
    operand = operand.strip()
    if operand.startswith("vcc"):
        return {-1, -2}
    m = re.fullmatch(r"s\[(\d+):(\d+)\]", operand)
    if m:
        return set(range(int(m[1]), int(m[2]) + 1))
    m = re.fullmatch(r"s(\d+)", operand)
    return {int(m[1])} if m else set()


def short_waits(text):
    """Vector instructions that read a scalar register or VCC less than two wait states -- memory
    instructions less than five -- behind the vector instruction that wrote it, in program order."""
    found, written, function = [], {}, ""
    for line in text.splitlines():
        m = re.match(r"[0-9a-f]+ <(.*)>:", line)
        if m:
            function, written = m[1], {}
            continue
        m = re.match(r"\s+(\S+)\s*([^/]*)", line)
        if not m:
            continue
        op, operands = m[1], [x.strip() for x in re.split(r",\s*(?![^\[]*\])", m[2].strip())]
        if op in ("s_branch", "s_endpgm", "s_setpc_b64"):
            written = {}
            continue
        states = int(operands[0], 0) + 1 if op == "s_nop" else 1
        if op.startswith("v_"):
            compare = op.startswith("v_cmp")
            # what it writes: the first operand, and the carry or flag behind it
            two = "_co_" in op or op.startswith(("v_div_scale", "v_mad_u64", "v_mad_i64"))
            outputs = operands[:2] if two else operands[:1]
            inputs = operands[len(outputs):]
            if compare and not any(scalar_registers(x) for x in outputs) and "exec" not in outputs[0]:
                outputs, inputs = ["vcc"], operands
            read = set().union(*(scalar_registers(x) for x in inputs)) if inputs else set()
            if op.startswith("v_div_fmas"):
                read |= {-1, -2}
            if any(written.get(r, 2) < 2 for r in read):
                found.append("%s: %s" % (function[:60], line.split("//")[0].strip()))
            written = {r: n + states for r, n in written.items()}
            for x in outputs:
                for r in scalar_registers(x):
                    written[r] = 0
        else:
            if op.startswith(("global_", "buffer_", "flat_", "scratch_")):
                read = set().union(set(), *(scalar_registers(x.split(" ")[0]) for x in operands))
                if any(written.get(r, 5) < 5 for r in read):
                    found.append("%s: %s" % (function[:60], line.split("//")[0].strip()))
            written = {r: n + states for r, n in written.items()}
            for x in operands[:1]:  # a scalar instruction that writes the register ends the matter
                for r in scalar_registers(x) if op.startswith("s_") else ():
                    written.pop(r, None)
    return found


@pytest.mark.parametrize("code,count", [
    ("v_cmp_gt_i32_e32 vcc, v1, v2\n\tv_cndmask_b32_e32 v3, v4, v5, vcc", 1),
    ("v_cmp_gt_i32_e32 vcc, v1, v2\n\ts_nop 0\n\tv_cndmask_b32_e32 v3, v4, v5, vcc", 1),
    ("v_cmp_gt_i32_e32 vcc, v1, v2\n\ts_nop 1\n\tv_cndmask_b32_e32 v3, v4, v5, vcc", 0),
    ("v_cmp_gt_i32_e64 s[2:3], v1, v2\n\tv_mov_b32_e32 v9, v8\n\tv_cndmask_b32_e64 v3, v4, v5, s[2:3]", 1),
    ("v_cmp_gt_i32_e64 s[2:3], v1, v2\n\tv_cmp_gt_i32_e64 s[4:5], v1, v2\n\tv_mov_b32_e32 v9, v8\n\t"
     "v_cndmask_b32_e64 v3, v4, v5, s[2:3]", 0),
    ("v_readfirstlane_b32 s2, v1\n\ts_mov_b32 m0, s9\n\ts_nop 0\n\tglobal_load_lds_dwordx4 v3, s[2:3] offset:1024", 1),
    ("v_readfirstlane_b32 s2, v1\n\ts_mov_b32 m0, s9\n\ts_nop 3\n\tglobal_load_lds_dwordx4 v3, s[2:3] offset:1024", 0),
])
def test_the_rule_finds_its_cases(code, count):
    assert len(short_waits("0 <f>:\n\t" + code)) == count


def test_vector_reads_of_fresh_scalar_results_keep_their_wait_states(listing):
    assert short_waits(listing) == []
