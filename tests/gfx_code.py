"""Reads back the gfx950 code of the library built here (llvm-objdump), for tests of what the source leaves to the compiler:
the instructions of every kernel as a control-flow graph, and two facts about them that hold on all paths."""
import os
import re
import shutil
import subprocess

OBJDUMP = os.environ.get("FLEXCO_OBJDUMP", "/opt/rocm/llvm/bin/llvm-objdump")


def kernels(lib, tmp):
    """{mangled name: [(address, mnemonic, operands)]} of the device code in `lib`; `tmp`: an empty directory"""
    copy = os.path.join(tmp, "lib.so")
    shutil.copy(lib, copy)
    subprocess.run([OBJDUMP, "--offloading", copy], check=True, capture_output=True, cwd=tmp)
    out = {}
    for f in sorted(os.listdir(tmp)):
        if not f.endswith("gfx950"):
            continue
        text = subprocess.run([OBJDUMP, "-d", "--mcpu=gfx950", "--no-show-raw-insn", os.path.join(tmp, f)], check=True,
                              capture_output=True, text=True).stdout
        code = None
        for line in text.splitlines():
            head = re.match(r"^[0-9a-f]+ <(.*)>:", line)
            if head:
                code = out.setdefault(head.group(1), [])
                continue
            m = re.match(r"^\s+(\S+)\s*(.*?)\s*//\s*([0-9A-Fa-f]+):", line)
            if m and code is not None:
                code.append((int(m.group(3), 16), m.group(1), [a.strip() for a in m.group(2).split(",")]))
    return out


def successors(code):
    at = {ins[0]: k for k, ins in enumerate(code)}
    succ = []
    for k, (addr, op, args) in enumerate(code):
        nxt = [k + 1] if k + 1 < len(code) else []
        if op in ("s_endpgm", "s_setpc_b64"):
            nxt = []
        elif op == "s_branch" or op.startswith("s_cbranch"):
            off = int(args[0], 0) & 0xffff
            target = at[addr + 4 + 4 * (off - 0x10000 if off & 0x8000 else off)]
            nxt = [target] if op == "s_branch" else nxt + [target]
        succ.append(nxt)
    return succ


def _fixpoint(code, start, step, join):
    """state on entry of every instruction, the join over all paths (`None`: not reached)"""
    succ, state = successors(code), [None] * len(code)
    state[0], work = start, [0]
    while work:
        k = work.pop()
        out = step(state[k], code[k])
        for n in succ[k]:
            new = out if state[n] is None else join(state[n], out)
            if new != state[n]:
                state[n] = new
                work.append(n)
    return state


def lds_reads_at_barriers(code):
    """[(reads still on their way that were issued since the previous barrier, and before it)] per s_barrier, upper bounds
    over all paths.  LDS reads return in order, so a wait for lgkmcnt(n) leaves the n youngest."""
    CAP = 64

    def step(st, ins):
        young, old = st
        _, op, args = ins
        if op.startswith("ds_"):
            return min(young + 1, CAP), old
        if op == "s_waitcnt":
            m = re.search(r"lgkmcnt\((\d+)\)", " ".join(args))
            if m:
                n = int(m.group(1))
                return min(young, n), min(old, max(n - young, 0))
        if op == "s_barrier":
            return 0, min(young + old, CAP)
        return st
    state = _fixpoint(code, (0, 0), step, lambda a, b: (max(a[0], b[0]), max(a[1], b[1])))
    return [state[k] for k, ins in enumerate(code) if ins[1] == "s_barrier" and state[k] is not None]


def _regs(operand):
    m = re.match(r"^([av])\[(\d+):(\d+)\]$", operand)
    if m:
        return [m.group(1) + str(i) for i in range(int(m.group(2)), int(m.group(3)) + 1)]
    return [operand] if re.match(r"^[av]\d+$", operand) else []


def operands_written_too_late(code, states):
    """the matrix products (address) one of whose operands may have been written by a vector instruction fewer than
    `states` wait states before"""
    def step(st, ins):
        _, op, args = ins
        n = int(args[0], 0) + 1 if op == "s_nop" else 1
        out = {r: left - n for r, left in st if left > n}
        if op.startswith("v_") and not op.startswith(("v_mfma", "v_cmp", "v_readfirstlane", "v_readlane")):
            written = args[:2] if op.startswith(("v_swap", "v_permlane")) else args[:1]
            out.update((r, states) for a in written for r in _regs(a))
        return frozenset(out.items())

    def join(a, b):
        out = dict(a)
        for r, left in b:
            out[r] = max(left, out.get(r, 0))
        return frozenset(out.items())
    state = _fixpoint(code, frozenset(), step, join)
    bad = []
    for k, (addr, op, args) in enumerate(code):
        if op.startswith("v_mfma") and state[k]:
            late = dict(state[k])
            if any(r in late for a in args[1:3] for r in _regs(a)):
                bad.append(addr)
    return bad
