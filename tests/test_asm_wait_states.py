"""Wait states around inline assembly, in the built library (CPU only).

Two distances that the hardware does not check, and that the compiler keeps
for its own instructions but not around inline assembly:
 - a vector instruction that writes a scalar register (v_readlane, a compare,
   a carry) and a vector memory instruction that reads it: 5 wait states;
 - a vector store of more than 8 bytes and a vector instruction that overwrites
   its data registers: 2 wait states.
The test disassembles the library's device code and walks back from every
vector memory instruction, and forward from every such store, over every path."""

import glob
import os
import re
import shutil
import subprocess

import pytest

from paper_2609_33536_amd import ekv

READ_STATES, STORE_STATES = 5, 2
_SREG = re.compile(r"^-?\|?s(?:(\d+)|\[(\d+):(\d+)\])\|?$")
_VREG = re.compile(r"^v(?:(\d+)|\[(\d+):(\d+)\])$")
_MEMORY = ("global_", "buffer_", "flat_", "scratch_")
_TWO_RESULTS = ("v_add_co_", "v_addc_co_", "v_sub_co_", "v_subb_co_", "v_subrev_co_", "v_subbrev_co_", "v_div_scale_",
                "v_mad_u64_u32", "v_mad_i64_i32")
_TO_SCALAR = ("v_readlane", "v_readfirstlane", "v_cmp")
_ENDS = ("s_endpgm", "s_branch", "s_setpc_b64")


def _regs(pattern, operand, name):
    m = pattern.match(operand)
    if not m:
        return {"vcc"} if name == "s" and operand in ("vcc", "vcc_lo", "vcc_hi") else set()
    lo = int(m.group(1) or m.group(2))
    return {f"{name}{i}" for i in range(lo, int(m.group(3) or lo) + 1)}


def _sregs(operand):
    return _regs(_SREG, operand, "s")


def _vregs(operand):
    return _regs(_VREG, operand, "v")


def _parse(text):
    """Functions as lists of (mnemonic, operands, line), labels as ('label:', [name], line)."""
    functions = [[]]
    for n, line in enumerate(text.splitlines(), 1):
        if re.match(r"^[0-9a-f]+ <.*>:$", line):
            functions.append([])
            continue
        line = line.split("//")[0].split(";")[0].strip()
        label = re.match(r"^<?([.\w]+)>?:$", line)
        if label:
            functions[-1].append(("label:", [label.group(1)], n))
        elif line and not line.startswith(".") and "file format" not in line and "Disassembly" not in line:
            op, *args = [t for t in re.split(r"[,\s]+", line) if t]
            functions[-1].append((op, args, n))
    return functions


def _scalar_writes(op, args):
    """Scalar registers that a vector instruction writes."""
    if not op.startswith("v_") or not args:
        return set()
    if op.startswith("v_cmp"):
        return _sregs(args[0]) or {"vcc"}
    regs = _sregs(args[0])
    if op.startswith(_TWO_RESULTS) and len(args) > 1:
        regs = regs | _sregs(args[1])
    return regs


def _states(op, args):
    return int(args[0], 0) + 1 if op == "s_nop" else 1


def too_close(text):
    """(states between, writer's line, reader's line) of every pair below its distance, and how many vector
    memory instructions with a scalar operand and how many wide stores were looked at."""
    found, reads, stores = [], 0, 0
    for code in _parse(text):
        jumps, labels = {}, {}
        for i, (op, args, _) in enumerate(code):
            if op.startswith(("s_branch", "s_cbranch")):
                jumps.setdefault(args[-1], []).append(i)
            elif op == "label:":
                labels[args[0]] = i

        def back(i, states, regs, reader):   # instruction i was executed `states` wait states before the reader
            while i >= 0 and states < READ_STATES:
                op, args, line = code[i]
                if op == "label:":
                    for j in jumps.get(args[0], []):
                        back(j - 1, states + 1, regs, reader)
                elif op in _ENDS:
                    return                                            # nothing falls through it
                elif _scalar_writes(op, args) & regs:
                    found.append((states, line, code[reader][2]))
                    return
                else:
                    states += _states(op, args)
                i -= 1

        def forward(i, states, data, store):   # instruction i is executed `states` wait states after the store
            while i < len(code) and states < STORE_STATES:
                op, args, line = code[i]
                if op.startswith("v_") and args and not op.startswith(_TO_SCALAR) and _vregs(args[0]) & data:
                    found.append((states, code[store][2], line))
                    return
                if op.startswith(("s_branch", "s_cbranch")) and args[-1] in labels:
                    forward(labels[args[-1]], states + 1, data, store)
                if op in _ENDS:
                    return
                states += 0 if op == "label:" else _states(op, args)
                i += 1

        for i, (op, args, _) in enumerate(code):
            if op.startswith(_MEMORY):
                regs = set().union(*map(_sregs, args))
                if regs:
                    reads += 1
                    back(i - 1, 0, regs, i)
                if re.search(r"_store_dwordx[34]$", op):
                    stores += 1
                    forward(i + 1, 0, _vregs(args[0 if op.startswith("buffer_") else 1]), i)
    return found, reads, stores


def test_the_walk_itself():
    load = "global_load_lds_dwordx4 v1, s[4:5]\n"
    assert too_close("v_readlane_b32 s5, v2, s3\ns_mov_b32 m0, s9\ns_nop 0\n" + load) == ([(2, 1, 4)], 1, 0)
    assert too_close("v_readlane_b32 s5, v2, s3\ns_mov_b32 m0, s9\ns_nop 3\n" + load) == ([], 1, 0)
    assert too_close("v_readlane_b32 s6, v2, s3\n" + load) == ([], 1, 0)                       # another register
    assert too_close("v_cmp_gt_i32_e64 s[4:5], v2, v3\n" + load) == ([(0, 1, 2)], 1, 0)
    assert too_close("v_readfirstlane_b32 s4, v2\ns_branch L1\ns_nop 7\n<L1>:\n" + load)[0] == [(1, 1, 5)]
    assert too_close("v_readfirstlane_b32 s4, v2\ns_branch L2\n<L1>:\n" + load)[0] == []        # not on its path
    store = "global_store_dwordx4 v[4:5], v[8:11], off sc1\n"
    assert too_close(store + "v_mov_b32_e32 v9, v1\n") == ([(0, 1, 2)], 0, 1)
    assert too_close(store + "s_nop 0\nv_mov_b32_e32 v9, v1\n") == ([(1, 1, 3)], 0, 1)
    assert too_close(store + "s_nop 1\nv_mov_b32_e32 v9, v1\n") == ([], 0, 1)
    assert too_close(store + "v_mov_b32_e32 v5, v9\nv_readlane_b32 s9, v8, 0\n") == ([], 0, 1)  # address; a read
    assert too_close(store + "s_cbranch_scc1 L1\ns_nop 7\n<L1>:\nv_mov_b64_e32 v[8:9], v[2:3]\n")[0] == [(1, 1, 5)]


def test_distances_in_the_library(tmp_path):
    objdump = "/opt/rocm/llvm/bin/llvm-objdump"
    if not os.path.exists(objdump):
        pytest.skip("llvm-objdump missing")
    from __graft_entry__ import _ensure_built
    _ensure_built()
    shutil.copy(ekv.LIB_PATH, tmp_path / "lib.so")
    subprocess.run([objdump, "--offloading", "lib.so"], cwd=tmp_path, check=True, stdout=subprocess.PIPE)
    found, reads, stores = [], 0, 0
    for path in sorted(glob.glob(str(tmp_path / "lib.so.*gfx950"))):
        text = subprocess.run([objdump, "-d", "--symbolize-operands", "--no-show-raw-insn", path], check=True,
                              stdout=subprocess.PIPE, text=True).stdout
        f, r, s = too_close(text)
        found, reads, stores = found + [(os.path.basename(path),) + x for x in f], reads + r, stores + s
    assert reads > 10000 and stores > 1000
    assert not found, f"{len(found)} too close (code object, wait states, lines of the two): {found[:8]}"
