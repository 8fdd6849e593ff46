"""What the build asks of the matrix-core decode kernels' generated code before it links the library.

The kernels issue the loads of their streaming loop in inline assembly and wait for them with hand-written counts; the
compiler does not know that the destination registers are being written until the wait.  check_decode_code refuses code
in which an instruction of the compiler's own touches such a register between the issue of a load and a wait that covers it.

Model.  Every path from the kernel's entry is followed: both ways of a conditional branch, loops until nothing new comes
up.  What a path carries is the list of pending hand-issued loads, in the order of their issue, and a few facts about
scalar registers (below).  Loads return in order, so after `s_waitcnt vmcnt(N)` at most the N youngest are pending (the
compiler's own loads are not listed, which can only make the list too long).  A statement that holds two waits
(await_loads_either: the count depends on whether the zero-points of the next blocks were asked for in this step) is taken
with the larger count if at least that many loads were issued since the last wait, else with the smaller.

The compiler leaves some decisions in a flag that a later branch tests (a scalar register pair that holds 0 or -1), so
paths that combine branches at random would reach code that no wave reaches.  A path therefore carries the flags: pairs set by
a move or a select of 0 / -1 or from other flags; a branch on one makes it known on either side.  It also carries whether
all lanes are known to be active (then a branch on an empty mask is not taken).  A fact is dropped when the register is
written in any other way, and where it is not read any more.
"""
import re

_LABEL = re.compile(r"^(\.LBB\d+_\d+):")
_VGPR = re.compile(r"\bv\[(\d+):(\d+)\]|\bv(\d+)\b")
_SGPR = re.compile(r"\bs\[(\d+):(\d+)\]|\bs(\d+)\b")
_PAIR = re.compile(r"^s\[(\d+):(\d+)\]$")
_UNKNOWN = 2                     # a flag that holds 0 or 1 (registers 0 or -1), not known which
_FULL, _SAVED_FULL = "exec", 3   # key of "all lanes active"; a pair that holds such a mask
_REST = 4                        # a pair that holds at least the lanes that are not active (those that have left a loop)


def kernel_bodies(asm: str, name: str):
    """(mangled name, text) of the kernels whose mangled name contains `name`."""
    return [(m.group(1), m.group(0)) for m in re.finditer(r"^(_Z\w*%s\w*):.*?^\.Lfunc_end\d+:" % name, asm, re.S | re.M)]


def _bits(pattern, text):
    mask = 0
    for a, b, c in pattern.findall(text):
        if c:
            mask |= 1 << int(c)
        else:
            mask |= ((1 << (int(b) - int(a) + 1)) - 1) << int(a)
    return mask


def _pair(text):
    m = _PAIR.match(text)
    return int(m.group(1)) if m and int(m.group(2)) == int(m.group(1)) + 1 else None


class _Op:
    """One instruction of the compiler's, or one inline-assembly statement (asm: its instructions)."""

    def __init__(self, text, asm=None):
        self.text, self.asm = text, asm
        self.loads, self.waits, self.target, self.cond, self.wait = [], [], None, None, None
        for t in asm if asm is not None else ():
            w = re.match(r"s_waitcnt\s+vmcnt\((\d+)\)$", t)
            if w:
                self.waits.append(int(w.group(1)))
            elif t.startswith(("buffer_load", "global_load")):
                self.loads.append(_bits(_VGPR, t.split(",")[0]))
        parts = text.split(None, 1)
        self.op = parts[0] if parts else ""
        self.args = [x.strip() for x in parts[1].split(",")] if len(parts) > 1 else []
        self.vgprs = 0 if asm is not None else _bits(_VGPR, text)
        # scalar registers written: the first operand, and the carry or condition that some vector instructions name second
        self.writes = 0
        for t in asm if asm is not None else (text,):
            p = t.split(None, 1)
            if len(p) < 2 or p[0].startswith(("s_cmp", "s_bitcmp", "s_waitcnt", "s_cbranch", "s_branch", "global_store", "buffer_store", "ds_write", "scratch_store")):
                continue
            a = [x.strip() for x in p[1].split(",")]
            self.writes |= _bits(_SGPR, a[0])
            if p[0].startswith("v_") and len(a) > 1 and re.search(r"_co_|div_scale|mad_[ui]64", p[0]):
                self.writes |= _bits(_SGPR, a[1])
        self.reads = _bits(_SGPR, text)
        if asm is None:
            w = re.match(r"s_waitcnt\b.*vmcnt\((\d+)\)", text)
            self.wait = int(w.group(1)) if w else None
            b = re.match(r"s_(c?)branch(?:_(\w+))?\s+(\.LBB\d+_\d+)", text)
            if b:
                self.target, self.cond = b.group(3), b.group(2)

        a = self.args
        if asm is None:
            self.writes_vcc = bool(a) and (a[0] == "vcc" or (len(a) > 1 and a[1] == "vcc" and self.op.startswith("v_")) or
                                           (self.op.startswith("v_cmp") and "_e32" in self.op))
        else:
            self.writes_vcc = any("vcc" in t for t in asm)
        self.writes_exec = asm is None and bool(a) and (a[0] == "exec" or "saveexec" in self.op or self.op.startswith("v_cmpx"))
        # neither a load, a wait or a branch, nor a word about scalar registers
        self.plain = not (self.loads or self.waits or self.target or self.wait is not None or self.writes or self.writes_vcc or
                          self.writes_exec or self.op == "s_endpgm")


def _parse(body):
    ops, labels, asm = [], {}, None
    for line in body.split("\n"):
        m = _LABEL.match(line)
        if m:
            labels[m.group(1)] = len(ops)
            continue
        t = line.strip()
        if t.startswith(";;#ASMSTART"):
            asm = []
        elif t.startswith(";;#ASMEND"):
            ops.append(_Op("", asm))
            asm = None
        else:
            t = t.split(";")[0].strip()
            if t and t[0] != "." and not t.endswith(":"):
                asm.append(t) if asm is not None else ops.append(_Op(t))
    return ops, labels


def _look_ahead(ops, labels):
    """Per instruction: the scalar registers that some path from it reads before it writes them, and whether a path leads
    to a hand-issued load or hand-written wait."""
    live, ahead = [0] * (len(ops) + 1), [False] * (len(ops) + 1)
    changed = True
    while changed:
        changed = False
        for i in range(len(ops) - 1, -1, -1):
            o = ops[i]
            out, loads = (0, False) if o.op in ("s_endpgm", "s_branch") else (live[i + 1], ahead[i + 1])
            if o.target:
                out, loads = out | live[labels[o.target]], loads or ahead[labels[o.target]]
            new = (out & ~o.writes) | o.reads, loads or bool(o.loads or o.waits)
            if new != (live[i], ahead[i]):
                live[i], ahead[i], changed = new[0], new[1], True
    return live, ahead


def _flag_result(o, facts):
    """What a scalar instruction leaves in its first operand: 0, 1, _UNKNOWN (a flag), _SAVED_FULL, or None (no fact)."""
    a = o.args
    if o.op == "s_cselect_b64" and a[1:] in (["-1", "0"], ["0", "-1"]):
        return _UNKNOWN
    if o.op == "s_mov_b64":
        if a[1] in ("0", "-1"):
            return 1 if a[1] == "-1" else 0
        if a[1] == "exec":
            return _SAVED_FULL if facts.get(_FULL) else None
        return facts.get(_pair(a[1]))
    if o.op in ("s_and_saveexec_b64", "s_or_saveexec_b64"):
        return _SAVED_FULL if facts.get(_FULL) else None
    if o.op in ("s_and_b64", "s_or_b64", "s_andn2_b64", "s_xor_b64"):
        x, y = (facts.get(_pair(z)) if _pair(z) is not None else None for z in a[1:3])
        if x not in (0, 1, _UNKNOWN) or y not in (0, 1, _UNKNOWN):
            own = facts.get(_pair(a[0])) if a[0] in a[1:3] else None         # a loop's mask of finished lanes, with more of them
            return _REST if o.op == "s_or_b64" and a[0] in a[1:3] and (own == _REST or facts.get(_FULL)) else None
        if o.op == "s_andn2_b64":
            y = 1 - y if y != _UNKNOWN else y
        if o.op == "s_or_b64":
            return 1 if 1 in (x, y) else 0 if x == y == 0 else _UNKNOWN
        if o.op == "s_xor_b64":
            return _UNKNOWN if _UNKNOWN in (x, y) else x ^ y
        return 0 if 0 in (x, y) else 1 if x == y == 1 else _UNKNOWN
    return None


def _check_kernel(name, body):
    ops, labels = _parse(body)
    heads, (live, ahead) = set(labels.values()), _look_ahead(ops, labels)
    ids, masks = {}, []                              # loads numbered through the kernel: (instruction, place in the statement)
    for i, o in enumerate(ops):
        for k, m in enumerate(o.loads):
            ids[i, k] = len(masks)
            masks.append(m)
    reached, visited = set(), set()
    work = [(0, (), 0, ((_FULL, 1),), None)]         # instruction, pending loads, loads since the last wait, facts, condition in vcc
    while work:
        pc, pending, issued, facts, vcc = work.pop()
        facts = dict(facts)
        busy = 0
        for x in pending:
            busy |= masks[x]
        while pc < len(ops):
            o = ops[pc]
            if pc in heads or o.target:
                if not pending and not ahead[pc]:
                    break                            # nothing left to check on the way
                facts = {k: v for k, v in facts.items() if k == _FULL or live[pc] >> k & 1 or (vcc and vcc[0] == k)}
                state = (pc, pending, issued, tuple(sorted(facts.items(), key=str)), vcc)
                if state in visited:
                    break
                visited.add(state)
            if o.plain and not o.vgprs & busy:
                pc += 1
                continue
            count = None
            if o.asm is not None:
                reached.add(pc)
                for k in range(len(o.loads)):
                    pending += (ids[pc, k],)
                    busy |= o.loads[k]
                    issued = min(issued + 1, 63)
                if o.waits:
                    count = max(o.waits) if issued >= max(o.waits) else min(o.waits)
            else:
                count = o.wait
                if o.vgprs & busy:
                    regs = [r for r in range(512) if (o.vgprs & busy) >> r & 1]
                    raise RuntimeError("%s: `%s` touches v%s while a hand-issued load may still be writing it" % (name, o.text, regs))
            if count is not None:
                pending, issued, busy = pending[max(0, len(pending) - count):] if count else (), 0, 0
                for x in pending:
                    busy |= masks[x]
            if o.op == "s_endpgm":
                break
            if o.op == "s_branch":
                pc = labels[o.target]
                continue
            if o.cond:
                taken, through, may_take, may_pass = facts, facts, True, True
                if o.cond in ("execz", "execnz") and facts.get(_FULL):
                    may_take, may_pass = o.cond == "execnz", o.cond == "execz"
                elif o.cond in ("vccz", "vccnz") and vcc:
                    key, zero_value = vcc            # vcc is zero exactly when the flag `key` (or the constant, key None) has this value
                    if key is None:
                        may_take = (o.cond == "vccz") == bool(zero_value)
                        may_pass = not may_take
                    elif facts.get(key) == _UNKNOWN:
                        value = zero_value if o.cond == "vccz" else 1 - zero_value      # the flag's where the branch is taken
                        taken, through = {**facts, key: value}, {**facts, key: 1 - value}
                if may_take:
                    work.append((labels[o.target], pending, issued, tuple(taken.items()), vcc))
                if not may_pass:
                    break
                facts = dict(through)
                pc += 1
                continue
            # facts about scalar registers
            result = _flag_result(o, facts) if o.asm is None else None
            exec_full = facts.get(_FULL, 0)
            if o.writes_exec:
                restores = o.op == "s_or_b64" and o.args[1] == "exec" and facts.get(_pair(o.args[2])) in (_SAVED_FULL, _REST)
                moves = o.op == "s_mov_b64" and facts.get(_pair(o.args[1])) == _SAVED_FULL
                kept = _pair(o.args[2]) if o.op == "s_andn2_b64" and o.args[1] == "exec" else None     # lanes leave a loop
                if kept is not None and not exec_full and facts.get(kept) != _REST:
                    kept = None
                facts = {k: v for k, v in facts.items() if v != _REST or k == _FULL or k == kept}
                if kept is not None:
                    facts[kept] = _REST
                exec_full = 1 if restores or moves or (exec_full and o.op == "s_or_saveexec_b64") else 0
            if o.writes_vcc:
                vcc = None
                if o.op in ("s_and_b64", "s_andn2_b64") and o.args[0] == "vcc" and o.args[1] == "exec" and facts.get(_FULL):
                    key, zero_value = _pair(o.args[2]), 0 if o.op == "s_and_b64" else 1
                    value = facts.get(key) if key is not None else None
                    if value in (0, 1):
                        vcc = (None, int(value == zero_value))
                    elif value == _UNKNOWN:
                        vcc = (key, zero_value)
            if o.writes:
                for key in [k for k in facts if k != _FULL and (o.writes >> k) & 3]:
                    del facts[key]
                    if vcc and vcc[0] == key:
                        vcc = None
            if result is not None and _pair(o.args[0]) is not None:
                facts[_pair(o.args[0])] = result
            facts[_FULL] = exec_full
            pc += 1
    missed = [i for i, o in enumerate(ops) if (o.loads or o.waits) and i not in reached]
    if missed:
        raise RuntimeError("%s: no path leads to the statement %s" % (name, ops[missed[0]].asm))
    return len(masks)


def check_decode_code(asm: str) -> int:
    """Raises RuntimeError if the code breaks the rule above; returns the number of hand-issued loads it holds."""
    return sum(_check_kernel(name, body) for name, body in kernel_bodies(asm, "decode_mfma"))
