"""The built device code keeps the wait states that inline assembly hides.

A matrix instruction (MFMA, structured-sparse MFMA) may read a register only two
wait states after a vector-ALU instruction wrote it, and a vector memory
instruction a scalar register (its base address) only five after.  The compiler
sees to that for its own instructions, not for those in inline assembly, in
front of which it is free to place the move of an operand.  This test reads the
listing of the library's gfx950 code objects (built here from these sources) and
looks at every such instruction, across branches.  CPU only.
"""
import os
import re
import shutil
import subprocess

import pytest

from paper_2501_08582_amd import _lib

OBJDUMP = shutil.which("llvm-objdump") or "/opt/rocm/llvm/bin/llvm-objdump"
MATRIX_WAIT, BASE_WAIT = 2, 5
MATRIX = ("v_mfma", "v_smfmac")
MEMORY = ("global_", "buffer_", "flat_", "scratch_")


def _regs(text):
    out = set()
    for m in re.finditer(r"\b([vas])\[(\d+):(\d+)\]|\b([vas])(\d+)\b", text):
        if m.group(1):
            out |= {m.group(1) + str(i) for i in range(int(m.group(2)), int(m.group(3)) + 1)}
        else:
            out.add(m.group(4) + m.group(5))
    return out


def _operands(text):
    return [o.strip() for o in re.split(r",(?![^\[]*\])", text)] if text else []


def _functions(listing):
    """{name: [(mnemonic, operands, address, branch target)]}; the target is an offset in the function."""
    out, cur = {}, None
    for line in listing.split("\n"):
        m = re.match(r"^[0-9a-f]+ <(.*)>:$", line)
        if m:
            cur = out.setdefault(m.group(1), [])
            continue
        m = re.match(r"^\s+(\S+)\s*(.*?)\s*// ([0-9A-F]+):.*?(?:<\S+\+0x([0-9a-f]+)>)?$", line)
        if m and cur is not None:
            cur.append((m.group(1), m.group(2), int(m.group(3), 16), m.group(4)))
    return out


def _written(mn, ops):
    """Registers that a vector-ALU instruction writes (its first operand; the second one too of a swap or
    where it takes a carry or a mask)."""
    if not mn.startswith("v_") or mn.startswith(MATRIX + ("v_nop",)):
        return set()
    o = _operands(ops)
    two = mn.startswith(("v_swap", "v_mad_u64", "v_mad_i64", "v_div_scale")) or "_co_" in mn
    return set().union(*(_regs(x) for x in o[:2 if two else 1]))


def _violations(code):
    bad, start = [], code[0][2] if code else 0
    at = {a - start: i for i, (_, _, a, _) in enumerate(code)}
    jumps = {}
    for i, (mn, _, _, target) in enumerate(code):
        if target and mn.startswith(("s_branch", "s_cbranch")):
            jumps.setdefault(at.get(int(target, 16)), []).append(i)

    def back(i, need, left, want, of):
        before = [] if i == 0 or code[i - 1][0] in ("s_branch", "s_endpgm") else [i - 1]
        for p in before + jumps.get(i, []):
            mn, ops = code[p][:2]
            if _written(mn, ops) & want:
                bad.append(f"{mn} {ops} -> {code[of][0]} {code[of][1]}: {need - left} wait states")
                continue
            states = int(ops, 0) + 1 if mn == "s_nop" else 1
            if states < left:
                back(p, need, left - states, want, of)

    for i, (mn, ops, _, _) in enumerate(code):
        o = _operands(ops)
        if mn.startswith(MATRIX):
            read = o if mn.startswith("v_smfmac") else o[1:]  # smfmac accumulates into its first operand
            back(i, MATRIX_WAIT, MATRIX_WAIT, set().union(*(_regs(x) for x in read)), i)
        elif mn.startswith(MEMORY):
            base = {r for r in _regs(ops) if r[0] == "s"}
            if base:
                back(i, BASE_WAIT, BASE_WAIT, base, i)
    return bad


def test_the_reader_sees_a_missing_wait():
    def listing(*lines):
        out = "0000 <f>:\n"
        for i, line in enumerate(lines):  # "mnemonic operands", with "@target" for a branch
            text, _, target = line.partition("@")
            out += f"\t{text} // {4 * i:012X}: 00000000" + (f" <f+{target}>" if target else "") + "\n"
        return out

    def bad(*lines):
        return _violations(_functions(listing(*lines))["f"])

    mfma = "v_mfma_f32_32x32x16_bf16 v[2:17], v[46:49], v[94:97], 0"
    assert bad("v_mov_b32_e32 v94, v19", mfma) and bad("v_mov_b32_e32 v94, v19", "s_nop 0", mfma)
    assert bad("v_accvgpr_mov_b32 a48, a0", "v_smfmac_f32_32x32x32_bf16 a[48:63], v[0:3], v[4:11], v12")
    assert not bad("v_mov_b32_e32 v94, v19", "s_nop 1", mfma)
    assert not bad("v_mov_b32_e32 v2, v19", mfma) and not bad("ds_read_b64 v[94:95], v2", mfma)
    # over a branch: the move at the end of a loop, the product at its head
    assert bad("s_nop 7", mfma, "v_mov_b32_e32 v94, v19", "s_cbranch_scc1 65532@0x4")
    load = "global_load_lds_dwordx4 v131, s[16:17]"
    assert bad("v_readfirstlane_b32 s16, v1", "s_mov_b32 m0, s36", "s_nop 0", load)
    assert not bad("v_readfirstlane_b32 s16, v1", "s_nop 4", load)
    assert not bad("s_mov_b32 s16, s2", load) and not bad("v_readfirstlane_b32 s18, v1", load)


def test_instructions_wait_for_their_operands(tmp_path):
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    if not os.path.exists(_lib.LIB_PATH):
        pytest.fail("liblors.so is not built (python -m paper_2501_08582_amd.build)")
    shutil.copy(_lib.LIB_PATH, tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=tmp_path, check=True, capture_output=True)
    seen, bad = 0, []
    for name in sorted(os.listdir(tmp_path)):
        if "gfx950" not in name:
            continue
        text = subprocess.run([OBJDUMP, "-d", name], cwd=tmp_path, check=True, capture_output=True, text=True).stdout
        for fn, code in _functions(text).items():
            seen += sum(mn.startswith(MATRIX) for mn, *_ in code)
            bad += [f"{fn}: {b}" for b in _violations(code)]
    assert seen > 5000, "the library's matrix instructions were not found"
    assert not bad, f"{len(bad)} instructions read an operand too early:\n" + "\n".join(bad[:10])
