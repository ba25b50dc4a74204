"""Static check of the hand-written DPP instructions in the device assembly.

A DPP instruction reads its first source through the cross-lane DPP network.
On gfx9-family GPUs (gfx950 included) the hardware does not interlock that
read: two wait states must separate a VALU write of the VGPR from the DPP
read, and five a VALU write of EXEC from any DPP instruction; a matrix (MFMA)
result needs far more before any VALU reads it.  The compiler inserts these
for the DPP instructions it generates.  The fused row-broadcast FMACs of the
factorisation are inline assembly, so the compiler does not see their DPP
operand; this module verifies on the assembly of each build that none of
them reads a register written too recently.  Nor does the compiler count a
write inside inline assembly as one before its own DPP and permlane-swap
instructions: their sources must be two wait states away from such a write.

Wait states are counted as the ISA does: one per instruction issued in
between, N + 1 for ``s_nop N``.  The walk back stops at a basic-block label,
where the requirement must already be met (a label can have predecessors
other than the fall-through); for a read outside inline assembly it goes on
through the fall-through and every branch to the label.

    python -m paper_1808_04473_amd.isa_check <file.s> ...
"""
from __future__ import annotations

import re
import sys

DPP_SRC_WAIT = 2     # VALU writes VGPR -> DPP reads it
DPP_EXEC_WAIT = 5    # VALU writes EXEC -> any DPP instruction
MFMA_READ_WAIT = 19  # any MFMA result -> VALU read (largest pass count, conservative)

_REG = re.compile(r"^[-|]*(?:neg\()?\|?([va])(?:(\d+)|\[(\d+):(\d+)\])")


def _regs(operand: str) -> set[tuple[str, int]]:
    m = _REG.match(operand.strip())
    if not m:
        return set()
    kind = m.group(1)
    if m.group(2) is not None:
        return {(kind, int(m.group(2)))}
    return {(kind, r) for r in range(int(m.group(3)), int(m.group(4)) + 1)}


def _split(line: str) -> tuple[str, list[str]]:
    body = line.split(";")[0].strip()
    if not body:
        return "", []
    parts = body.split(None, 1)
    op = parts[0]
    if len(parts) == 1:
        return op, []
    # operands end where the first modifier (word with ':' or a bare keyword) starts
    ops = []
    for tok in parts[1].split(","):
        tok = tok.strip()
        ops.append(tok.split()[0] if tok else tok)
    return op, ops


def _wait_states(op: str, ops: list[str]) -> int:
    if op == "s_nop":
        return int(ops[0], 0) + 1 if ops else 1
    return 1


def _valu_writes(op: str, ops: list[str]) -> tuple[set[tuple[str, int]], bool]:
    """(VGPR/AGPR written, EXEC written) of a vector-ALU instruction."""
    if not op.startswith("v_") or not ops:
        return set(), False
    if op.startswith("v_cmpx"):
        return set(), True
    if op.startswith(("v_cmp", "v_readlane", "v_readfirstlane")):
        return set(), False
    return _regs(ops[0]), False


def _is_label(line: str) -> bool:
    return bool(re.match(r"^[.\w]+:", line))


def _cross_lane_sources(op: str, ops: list[str]) -> set[tuple[str, int]]:
    """Registers that a DPP or permlane-swap instruction reads across lanes."""
    if "_dpp" in op and len(ops) >= 2:
        return _regs(ops[1])
    if op.startswith("v_permlane") and "swap" in op and len(ops) >= 2:
        return _regs(ops[0]) | _regs(ops[1])
    return set()


def _check_outside(lines: list[str]) -> list[str]:
    """Cross-lane reads outside inline assembly of registers that a vector
    instruction inside it wrote less than two wait states before."""
    errors = []
    inside, jumps, in_asm = [], {}, False
    for n, raw in enumerate(lines):
        s = raw.strip()
        if s.startswith(";;#ASMSTART"):
            in_asm = True
        elif s.startswith(";;#ASMEND"):
            in_asm = False
        inside.append(in_asm)
        op, ops = _split(raw)
        if op.startswith(("s_branch", "s_cbranch")) and ops:
            jumps.setdefault(ops[0], []).append(n)

    def writer(k, src, waited):
        while k >= 0 and waited < DPP_SRC_WAIT:
            s = lines[k].strip()
            if _is_label(s):
                for j in jumps.get(s.split(":")[0], []):
                    w = writer(j, src, waited)
                    if w is not None:
                        return w
            else:
                op, ops = _split(lines[k])
                if op and not op.startswith("."):
                    if op in ("s_endpgm", "s_setpc_b64"):
                        return None
                    if inside[k] and _valu_writes(op, ops)[0] & src:
                        return k
                    waited += _wait_states(op, ops)
            k -= 1
        return None

    for n, raw in enumerate(lines):
        if inside[n]:
            continue
        src = _cross_lane_sources(*_split(raw))
        k = writer(n - 1, src, 0) if src else None
        if k is not None:
            errors.append(f"line {n + 1}: {raw.strip()!r} reads across lanes what inline assembly wrote at line {k + 1}")
    return errors


def check_lines(lines: list[str]) -> list[str]:
    """Returns one message per hazard found in the inline-assembly DPP
    instructions of the given assembly listing, and in the cross-lane reads of
    what inline assembly wrote."""
    errors = _check_outside(lines)
    in_asm = False
    for n, raw in enumerate(lines):
        s = raw.strip()
        if s.startswith(";;#ASMSTART"):
            in_asm = True
            continue
        if s.startswith(";;#ASMEND"):
            in_asm = False
            continue
        if not in_asm:
            continue
        op, ops = _split(raw)
        if "_dpp" not in op or len(ops) < 2:
            continue
        src0 = _regs(ops[1])
        every = set()
        for o in ops[1:]:
            every |= _regs(o)
        waited = 0
        k = n - 1
        while k >= 0 and waited < MFMA_READ_WAIT:
            prev = lines[k].strip()
            if _is_label(prev):
                if waited < DPP_EXEC_WAIT:
                    errors.append(f"line {n + 1}: {s!r} follows block label {prev!r} "
                                  f"after only {waited} wait states")
                break
            pop, pops = _split(lines[k])
            if pop and not pop.startswith("."):
                wr, wexec = _valu_writes(pop, pops)
                if "mfma" in pop and wr & every:
                    errors.append(f"line {n + 1}: {s!r} reads an MFMA result of line {k + 1} "
                                  f"after {waited} wait states")
                elif waited < DPP_SRC_WAIT and wr & src0:
                    errors.append(f"line {n + 1}: {s!r} reads its DPP source written at line "
                                  f"{k + 1} ({prev!r}) after {waited} wait states")
                if wexec and waited < DPP_EXEC_WAIT:
                    errors.append(f"line {n + 1}: {s!r} follows an EXEC write at line {k + 1} "
                                  f"after {waited} wait states")
                waited += _wait_states(pop, pops)
            k -= 1
    return errors


def check_file(path: str) -> list[str]:
    with open(path) as f:
        return [f"{path}: {e}" for e in check_lines(f.read().split("\n"))]


def main(argv=None) -> int:
    errs = []
    for p in (argv if argv is not None else sys.argv[1:]):
        errs += check_file(p)
    for e in errs:
        print(e)
    return 1 if errs else 0


if __name__ == "__main__":
    sys.exit(main())
