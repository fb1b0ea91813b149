"""Check of generated gfx950 assembly for the hazards that the compiler cannot see.

The product kernels issue their MFMAs and direct global->LDS loads in inline assembly. The compiler inserts no wait states
around them, so the ones they need stand in the source (mfma_results_ready, valu_results_ready, the s_nop of dma_load16 and
mfma16_acc_and_load), and nothing keeps the compiler from placing an instruction of its own (a copy, a spill, a reload of a
scalar register) inside that distance. Here the distances are read off the listing, along every path through a kernel,
back edges of loops included:

  MFMA -> other access to an accumulation register      12 wait states (eight are asked for behind one of four passes)
  access to an accumulation register -> MFMA             3 (two are asked for)
  vector write of an ordinary register -> MFMA reads it  2
  vector write of a scalar register -> base of a direct load  5
  write of M0 -> direct load                             1

An instruction stands for one wait state, s_nop N for N + 1.
"""
from __future__ import annotations

import re

AFTER_MFMA, BEFORE_MFMA, OPERAND, SCALAR_BASE, M0 = 12, 3, 2, 5, 1
_FAR = 16                      # longer distances are all the same

_REG = re.compile(r"\b([vsa])(?:(\d+)\b|\[(\d+):(\d+)\])|\b(vcc|vcc_lo|vcc_hi|m0)\b")
_TWO_RESULTS = ("v_add_co", "v_addc_co", "v_sub_co", "v_subb_co", "v_subrev_co", "v_subbrev_co", "v_mad_u64_u32", "v_mad_i64_i32",
                "v_div_scale", "v_swap")


def _registers(text: str) -> list[str]:
    out = []
    for kind, one, first, last, special in _REG.findall(text):
        if special:
            out += ["vcc_lo", "vcc_hi"] if special == "vcc" else [special]
        elif one:
            out.append(kind + one)
        else:
            out += [f"{kind}{i}" for i in range(int(first), int(last) + 1)]
    return out


class _Inst:
    """What of an instruction matters here. writes: ordinary and scalar registers written by a vector instruction, and M0."""
    __slots__ = ("line", "text", "states", "mfma", "acc", "direct", "reads", "writes")

    def __init__(self, line: int, text: str):
        name, _, rest = text.partition(" ")
        ops = [o.strip() for o in rest.split(",")]
        self.line, self.text = line, text
        self.states = int(ops[0], 0) + 1 if name == "s_nop" else 1
        self.mfma = name.startswith("v_mfma")
        self.direct = "_load_lds_" in name
        self.acc = not self.mfma and any(r[0] == "a" for r in _registers(rest))
        self.reads = self.writes = ()
        if self.mfma:
            self.reads = tuple(r for r in _registers(",".join(ops[1:])) if r[0] == "v")
        elif self.direct:
            self.reads = tuple(r for r in _registers(",".join(ops[1:])) if r[0] == "s" or r.startswith("vcc"))
        elif name.startswith("v_"):
            results = ops[:2] if name.startswith(_TWO_RESULTS) else ops[:1]
            self.writes = tuple(r for r in _registers(",".join(results)) if r[0] in "vs")
            if name.startswith("v_cmp") and name.endswith("_e32"):
                self.writes = ("vcc_lo", "vcc_hi")
        if name.startswith("s_") and ops[0] == "m0":
            self.writes = ("m0",)


class _Block:
    def __init__(self):
        self.insts: list[_Inst] = []
        self.next: list[str | int] = []   # labels, or the number of the block that follows
        self.entry: dict[str, int] | None = None


def _functions(lines):
    """Blocks of each function: [(name, blocks, label -> block number)]."""
    out, name, blocks, labels = [], None, [], {}
    for n, line in enumerate(lines, 1):
        code = line.split(";", 1)[0].strip()
        if not code:
            continue
        if code.endswith(":"):
            label = code[:-1]
            if label.startswith(".Lfunc_end"):
                if name is not None:
                    out.append((name, blocks, labels))
                name = None
            elif label.startswith(".L"):
                if name is not None:
                    blocks.append(_Block())
                    labels[label] = len(blocks) - 1
            else:
                name, blocks, labels = label, [_Block()], {}
            continue
        if name is None or code.startswith("."):
            continue
        inst = _Inst(n, re.sub(r"\s+", " ", code))
        blocks[-1].insts.append(inst)
        op = code.split()[0]
        if op.startswith(("s_cbranch", "s_branch", "s_endpgm", "s_setpc")):
            if op.startswith(("s_cbranch", "s_branch")):
                blocks[-1].next.append(code.split()[1])
            if op.startswith("s_cbranch"):
                blocks[-1].next.append(len(blocks))
            blocks.append(_Block())
            blocks[-2].next.append(None)   # the end of the block is explicit
    return out


def _walk(block: _Block, entry: dict[str, int], report=None) -> dict[str, int]:
    """Distances (wait states passed since) at the end of a block, from those at its start."""
    now = 0
    at = {k: -d for k, d in entry.items()}   # time of each last event

    def passed(key):
        return now - at[key] if key in at else _FAR

    for i in block.insts:
        if i.mfma:
            if report is not None:
                if passed("acc") < BEFORE_MFMA:
                    report(i, "an accumulation register is touched just ahead of an MFMA")
                for r in i.reads:
                    if passed(r) < OPERAND:
                        report(i, f"{r} is written by a vector instruction just ahead of the MFMA that reads it")
        elif i.acc:
            if report is not None and passed("mfma") < AFTER_MFMA:
                report(i, "an accumulation register is touched behind an MFMA")
        if i.direct and report is not None:
            if passed("m0") < M0:
                report(i, "M0 is written just ahead of a direct load")
            for r in i.reads:
                if passed(r) < SCALAR_BASE:
                    report(i, f"{r} is written by a vector instruction just ahead of the direct load that it is the base of")
        now += i.states
        # an event is timed behind its own instruction, so that the next one stands zero wait states from it
        if i.mfma:
            at["mfma"] = now
        if i.acc:
            at["acc"] = now
        for r in i.writes:
            at[r] = now
    return {k: now - t for k, t in at.items() if now - t < _FAR}


def hazards(lines) -> list[str]:
    """What stands too close together in a listing, as 'line: reason: instruction'."""
    found = {}
    for name, blocks, labels in _functions(lines):
        if not any(i.mfma or i.direct for b in blocks for i in b.insts):
            continue
        for number, b in enumerate(blocks):
            if None in b.next:
                b.next = [x for x in b.next if x is not None]
            else:
                b.next.append(number + 1)   # falls through
            b.next = [labels.get(x, -1) if isinstance(x, str) else x for x in b.next]
        blocks[0].entry = {}
        work = [0]
        while work:
            b = blocks[work.pop()]
            out = _walk(b, b.entry)
            for x in b.next:
                if not 0 <= x < len(blocks):
                    continue
                old = blocks[x].entry
                new = dict(out) if old is None else {**out, **{k: min(d, out.get(k, d)) for k, d in old.items()}}
                if new != old:
                    blocks[x].entry = new
                    work.append(x)
        for b in blocks:
            if b.entry is not None:
                _walk(b, b.entry, lambda i, why: found.setdefault((i.line, why), f"{i.line}: {why}: {i.text}"))
    return [found[k] for k in sorted(found)]
