"""Wait states around the prefill kernels' inline-assembly loads (CPU only).

A vector instruction that writes a scalar register (v_readlane, a compare,
a carry) must be followed by 5 wait states before a vector memory instruction
reads that register; the hardware does not check.  The compiler keeps the
distance for its own loads but does not look into inline assembly.  The test
builds the kernels' assembly with the library's flags and walks back from
every vector memory instruction over every path that leads to it."""

import os
import re
import subprocess

import pytest

from paper_2609_33536_amd import build

WAIT_STATES = 5
_SREG = re.compile(r"^-?\|?s(?:(\d+)|\[(\d+):(\d+)\])\|?$")
_MEMORY = ("global_", "buffer_", "flat_", "scratch_")
_TWO_RESULTS = ("v_add_co_", "v_addc_co_", "v_sub_co_", "v_subb_co_", "v_subrev_co_", "v_subbrev_co_", "v_div_scale_",
                "v_mad_u64_u32", "v_mad_i64_i32")


def _sregs(operand):
    m = _SREG.match(operand)
    if m:
        lo = int(m.group(1) or m.group(2))
        return {f"s{i}" for i in range(lo, int(m.group(3) or lo) + 1)}
    return {"vcc"} if operand in ("vcc", "vcc_lo", "vcc_hi") else set()


def _parse(text):
    """Instructions and labels in order: (mnemonic, operands, line), ('label:', [name], line)."""
    out = []
    for n, line in enumerate(text.splitlines(), 1):
        line = line.split(";")[0].split("//")[0].strip()
        if not line or (line.startswith(".") and not line.endswith(":")):
            continue
        if line.endswith(":"):
            out.append(("label:", [line[:-1]], n))
            continue
        op, *args = [t for t in re.split(r"[,\s]+", line) if t]
        out.append((op, args, n))
    return out


def _vector_writes(op, args):
    """Scalar registers that a vector instruction writes."""
    if not op.startswith("v_") or not args:
        return set()
    if op.startswith("v_cmp"):
        return _sregs(args[0]) if _sregs(args[0]) else {"vcc"}
    regs = _sregs(args[0])
    if op.startswith(_TWO_RESULTS) and len(args) > 1:
        regs = regs | _sregs(args[1])
    return regs


def too_close(text):
    """(states between, writer's line, reader's line) of every pair below the required distance, and how
    many vector memory instructions with a scalar operand were looked at."""
    code = _parse(text)
    jumps = {}
    for i, (op, args, _) in enumerate(code):
        if op.startswith(("s_branch", "s_cbranch")):
            jumps.setdefault(args[-1], []).append(i)
    found, looked = [], 0

    def back(i, states, regs, reader):   # instruction i was executed `states` wait states before the reader
        while i >= 0 and states < WAIT_STATES:
            op, args, line = code[i]
            if op == "label:":
                for j in jumps.get(args[0], []):
                    back(j - 1, states + 1, regs, reader)
            elif op in ("s_endpgm", "s_branch", "s_setpc_b64"):
                return                                            # nothing falls through it
            elif _vector_writes(op, args) & regs:
                found.append((states, line, code[reader][2]))
                return
            else:
                states += int(args[0], 0) + 1 if op == "s_nop" else 1
            i -= 1

    for i, (op, args, _) in enumerate(code):
        if op.startswith(_MEMORY):
            regs = set().union(*map(_sregs, args))
            if regs:
                looked += 1
                back(i - 1, 0, regs, i)
    return found, looked


def test_the_walk_itself():
    load = "global_load_lds_dwordx4 v1, s[4:5]\n"
    assert too_close("v_readlane_b32 s5, v2, s3\ns_mov_b32 m0, s9\ns_nop 0\n" + load) == ([(2, 1, 4)], 1)
    assert too_close("v_readlane_b32 s5, v2, s3\ns_mov_b32 m0, s9\ns_nop 3\n" + load) == ([], 1)
    assert too_close("v_readlane_b32 s6, v2, s3\n" + load) == ([], 1)                       # another register
    assert too_close("v_cmp_gt_i32_e64 s[4:5], v2, v3\n" + load) == ([(0, 1, 2)], 1)
    assert too_close("v_readfirstlane_b32 s4, v2\ns_branch .L1\ns_nop 7\n.L1:\n" + load)[0] == [(1, 1, 5)]
    assert too_close("v_readfirstlane_b32 s4, v2\ns_branch .L2\n.L1:\n" + load)[0] == []   # not on its path


@pytest.mark.parametrize("source", ["prefill.hip", "transition.hip"])
def test_scalar_operands_of_memory_instructions(source, tmp_path):
    try:
        cc = build.hipcc()
    except RuntimeError:
        pytest.skip("hipcc missing")
    asm = tmp_path / "kernels.s"
    p = subprocess.run([cc, *build.FLAGS, "--cuda-device-only", "-S", os.path.join(build.CSRC, source), "-o", str(asm)],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert p.returncode == 0, p.stdout[-3000:]
    found, looked = too_close(asm.read_text())
    assert looked > 10
    assert not found, f"{len(found)} of {looked} too close (wait states, writer's line, reader's line): {found[:8]}"
