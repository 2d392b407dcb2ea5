"""Scan gfx950 assembly for vector instructions that read a register too soon after a matrix
instruction wrote it.

The matrix pipeline delivers its result some cycles after issue and the hardware does not
interlock a following vector-ALU read; the compiler pads with wait states.  It was seen to
leave a path uncovered (matrix instruction, two branches, a register copy of the accumulator:
3 to 4 wait states instead of 8), which gave wrong numbers in one build and not in the next.
This walks every control-flow path from each matrix instruction for NEED wait states and
reports vector-ALU reads of its destination inside that window.  `s_nop k` counts k + 1, any
other instruction 1; a register that is overwritten drops out of the dependence.
"""
import re

NEED = 8  # wait states between a 4-pass matrix instruction and a vector-ALU read of its result: what the compiler keeps on gfx950, nowhere fewer
_REG = re.compile(r"\bv\[(\d+):(\d+)\]|\bv(\d+)\b")


def _regs(text):
    out = set()
    for m in _REG.finditer(text):
        if m.group(1):
            out.update(range(int(m.group(1)), int(m.group(2)) + 1))
        else:
            out.add(int(m.group(3)))
    return out


def _blocks(lines):
    blocks, order, cur = {"__entry": []}, ["__entry"], "__entry"
    for ln in lines:
        ln = ln.split(";")[0].rstrip()
        if not ln.strip():
            continue
        m = re.match(r"^(\.LBB[0-9_]+):", ln)
        if m:
            cur = m.group(1)
            blocks[cur] = []
            order.append(cur)
        elif not ln.lstrip().startswith("."):
            blocks[cur].append(ln.strip())
    return blocks, order


def scan(asm_text, name_filter="decode_kernel", need=NEED):
    """Returns [(kernel, block, matrix instruction, reader, wait states between them)]."""
    text = asm_text.split("\n")
    findings, kernels = [], 0
    i = 0
    while i < len(text):
        m = re.match(r"^(_Z\S+):", text[i])
        if not (m and name_filter in m.group(1)):
            i += 1
            continue
        j = i + 1
        while j < len(text) and "s_endpgm" not in text[j]:
            j += 1
        kernels += 1
        blocks, order = _blocks(text[i + 1 : j + 1])
        fallthrough = {}
        for bi, b in enumerate(order):
            ends_in_jump = bool(blocks[b]) and blocks[b][-1].startswith("s_branch")
            fallthrough[b] = order[bi + 1] if not ends_in_jump and bi + 1 < len(order) else None
        for b in order:
            for k, x in enumerate(blocks[b]):
                if not x.startswith("v_mfma"):
                    continue
                dst = frozenset(_regs(x.split()[1].rstrip(",")))
                seen, stack = set(), [(b, k + 1, 0, dst)]
                while stack:
                    bb, pos, ws, live = stack.pop()  # live: registers of the result not overwritten since
                    if ws >= need or not live or (bb, pos, live) in seen:
                        continue
                    seen.add((bb, pos, live))
                    ins, ended = blocks[bb], False
                    while pos < len(ins) and ws < need and live:
                        y = ins[pos]
                        op = y.split()[0]
                        nop = re.match(r"s_nop\s+(\d+)", y)
                        if nop:
                            ws += int(nop.group(1)) + 1
                            pos += 1
                            continue
                        parts = [p.strip() for p in y[len(op):].split(",")]
                        if op.startswith("v_") and not op.startswith("v_mfma"):
                            srcs = set()
                            for p in parts[1:]:
                                srcs |= _regs(p)
                            if srcs & live:
                                findings.append((m.group(1), bb, x, y, ws))
                                ended = True
                                break
                            if parts:
                                live = live - _regs(parts[0])
                        t = re.match(r"s_cbranch_\w+\s+(\S+)", y)
                        if t and t.group(1) in blocks:
                            stack.append((t.group(1), 0, ws + 1, live))
                        t = re.match(r"s_branch\s+(\S+)", y)
                        if t:
                            if t.group(1) in blocks:
                                stack.append((t.group(1), 0, ws + 1, live))
                            ended = True
                            break
                        ws += 1
                        pos += 1
                    if not ended and pos >= len(ins) and ws < need and live and fallthrough[bb]:
                        stack.append((fallthrough[bb], 0, ws, live))
        i = j
    return findings, kernels


NEED_SCALAR = 5  # wait states between a vector-ALU write of a scalar register and a memory instruction that reads it
_SREG = re.compile(r"\bs\[(\d+):(\d+)\]|\bs(\d+)\b")


def _scalar_regs(text):
    out = set()
    for m in _SREG.finditer(text):
        if m.group(1):
            out.update(range(int(m.group(1)), int(m.group(2)) + 1))
        else:
            out.add(int(m.group(3)))
    return out


def scan_scalar_addresses(asm_text, name_filter="decode_kernel", need=NEED_SCALAR):
    """Memory instructions that read a scalar register too soon after a vector-ALU instruction wrote it (v_readlane of a
    spilled register, v_readfirstlane, a compare), along every path.  The compiler keeps the distance between its own instructions
    but does not look inside inline assembly.  Returns [(kernel, block, writer, reader, wait states)], number of kernels."""
    text = asm_text.split("\n")
    findings, kernels, i = [], 0, 0
    while i < len(text):
        m = re.match(r"^(_Z\S+):", text[i])
        if not (m and name_filter in m.group(1)):
            i += 1
            continue
        j = i + 1
        while j < len(text) and "s_endpgm" not in text[j]:
            j += 1
        kernels += 1
        blocks, order = _blocks(text[i + 1 : j + 1])
        follows = {b: order[k + 1] if k + 1 < len(order) else None for k, b in enumerate(order)}
        for b in order:
            for k, x in enumerate(blocks[b]):
                op, _, operands = x.partition(" ")
                if not op.startswith("v_") or op.startswith("v_mfma"):
                    continue
                # (a carry or compare result is the second operand of some instructions)
                written = frozenset(r for p in operands.split(",")[: 2 if "_co_" in op or "div_scale" in op else 1] for r in _scalar_regs(p))
                seen, stack = set(), [(b, k + 1, 0, written)]
                while stack:
                    bb, pos, ws, live = stack.pop()
                    if ws >= need or not live or (bb, pos, ws, live) in seen:
                        continue
                    seen.add((bb, pos, ws, live))
                    if pos >= len(blocks[bb]):
                        if follows[bb]:
                            stack.append((follows[bb], 0, ws, live))
                        continue
                    y = blocks[bb][pos]
                    yop, _, yargs = y.partition(" ")
                    if yop == "s_nop":
                        stack.append((bb, pos + 1, ws + int(yargs) + 1, live))
                        continue
                    if re.match(r"(global|flat|buffer|scratch|tbuffer)_", yop) and _scalar_regs(yargs) & live:
                        findings.append((m.group(1), bb, x, y, ws))
                        continue
                    if yop.startswith("s_") and not re.match(r"s_(cmp|bitcmp|cbranch|branch|waitcnt|barrier|setprio|store|dcache)", yop):
                        live = live - _scalar_regs(yargs.split(",")[0])
                    t = re.match(r"s_c?branch(?:_\w+)?\s+(\S+)", y)
                    if t and t.group(1) in blocks:
                        stack.append((t.group(1), 0, ws + 1, live))
                    if not yop.startswith("s_branch"):
                        stack.append((bb, pos + 1, ws + 1, live))
        i = j
    return findings, kernels
