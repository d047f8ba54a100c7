"""The kernels that read LDS behind the compiler's back (lds_read_*_untracked and the like) count
their own waits.  Checked in the assembly of the library's own sources, without a GPU: along every
path of every kernel, no instruction uses a register between the LDS read that fills it and a
wait that lets that read land.  A plain copy of such a register is followed and only counts once
the copy is used; a wait for lgkmcnt(n) leaves the n newest LDS operations in flight, which
return in order.
"""
import os
import re
import subprocess

import pytest

from paper_2512_06989_amd import build

HIPCC = build.HIPCC
REG_RANGE = re.compile(r"\b([va])\[(\d+):(\d+)\]")
REG = re.compile(r"\b([va])(\d+)\b")
MOST = 64   # operations followed at once (the counter holds 15)


def _regs(text):
    out = {k + n for k, n in REG.findall(text)}
    for k, a, b in REG_RANGE.findall(text):
        out.update(k + str(i) for i in range(int(a), int(b) + 1))
    return frozenset(out)


class Instr:
    def __init__(self, text):
        self.text, self.op = text, text.split()[0]
        first, _, rest = text.partition(",")
        self.all, self.dest, self.src = _regs(text), _regs(first), _regs(rest)
        self.is_lds = self.op.startswith("ds_")
        self.fills = self.is_lds and ("read" in self.op or "permute" in self.op or "rtn" in self.op)
        self.stores = "store" in self.op or self.op.startswith(("ds_write", "v_cmp"))
        m = re.search(r"lgkmcnt\((\d+)\)", text)
        self.wait = int(m.group(1)) if self.op == "s_waitcnt" and m else None
        m = re.match(r"(s_branch|s_cbranch\w+)\s+(\S+)", text)
        self.target = m.group(2) if m else None


def kernels(asm):
    """name -> (instructions, label -> index) of every function in the assembly text"""
    out, cur = {}, None
    for line in asm.splitlines():
        if line.startswith(".Lfunc_end"):
            cur = None
        m = re.match(r"^(_Z\w+):", line)
        if m:
            cur = out[m.group(1)] = ([], {})
            continue
        if cur is None:
            continue
        line = line.split(";")[0].strip()
        m = re.match(r"^(\.L\w+):", line)
        if m:
            cur[1][m.group(1)] = len(cur[0])
        elif line and not line.startswith("."):
            cur[0].append(Instr(line))
    return out


def early_uses(ins, labels):
    """Instructions that name a register whose LDS read may still be in flight."""
    # state at a label: the registers of the LDS operations in flight, oldest first, -> what may
    # hold an early copy (united over the paths that arrive with the same operations in flight)
    bad, seen, work = set(), {}, [(0, (), frozenset())]
    heads = set(labels.values())
    while work:
        pc, flight, copies = work.pop()
        while pc < len(ins):
            if pc in heads:
                known = seen.get((pc, flight))
                if known is not None and copies <= known:
                    break
                copies = copies | known if known else copies
                seen[pc, flight] = copies
            i = ins[pc]
            if i.wait is not None:
                flight = flight[len(flight) - i.wait:] if 0 < i.wait < len(flight) else flight if i.wait else ()
            else:
                pending = frozenset().union(*flight) if flight else frozenset()
                if i.op.startswith(("v_mov_b", "v_accvgpr_read", "v_accvgpr_write")):
                    if i.dest & pending:
                        bad.add((pc, i.text))
                    copies = copies | i.dest if i.src & (pending | copies) else copies - i.dest
                else:
                    if i.all & pending or (i.all if i.stores else i.src) & copies:
                        bad.add((pc, i.text))
                    if not i.stores and not i.op.startswith("s_"):
                        copies = copies - i.dest
                if i.is_lds:
                    flight = (flight + (i.dest if i.fills else frozenset(),))[-MOST:]
                elif i.op.startswith(("s_load", "s_buffer_load")):
                    flight = (flight + (frozenset(),))[-MOST:]
            if i.target is not None:
                if i.op == "s_branch":
                    pc = labels[i.target]
                    continue
                work.append((labels[i.target], flight, copies))
            elif i.op in ("s_endpgm", "s_setpc_b64"):
                break
            pc += 1
    return sorted(bad)


def test_the_check_itself():
    def run(text):
        (k,) = kernels("_Zk:\n" + text + "\n.Lfunc_end0:\n").values()
        return [t for _, t in early_uses(*k)]
    read2 = "ds_read_b128 v[0:3], v9\nds_read_b128 v[4:7], v9 offset:64\n"
    use = "v_add_f32_e32 v8, v2, v2\n"
    assert run(read2 + "s_waitcnt lgkmcnt(1)\n" + use + "s_endpgm") == []
    assert run(read2 + "s_waitcnt lgkmcnt(2)\n" + use + "s_endpgm") == [use.strip()]
    assert run(read2 + "v_mov_b32_e32 v10, v2\ns_waitcnt lgkmcnt(0)\ns_endpgm") == []
    assert run(read2 + "v_mov_b32_e32 v10, v2\ns_waitcnt lgkmcnt(0)\nv_add_f32_e32 v8, v10, v10\ns_endpgm") != []
    assert run(read2 + "s_cbranch_scc1 .LBB0_1\ns_waitcnt lgkmcnt(0)\n.LBB0_1:\n" + use + "s_endpgm") == [use.strip()]


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
@pytest.mark.parametrize("src", ["bwd.hip", "fwd_bf16.hip", "gemm_bf16.hip"])
def test_no_register_is_used_before_its_lds_read_has_landed(src, tmp_path):
    asm = str(tmp_path / "kernels.asm")
    subprocess.run([HIPCC, *build.FLAGS, "--offload-device-only", "-S", "-o", asm, os.path.join(build.CSRC, src)],
                   check=True, capture_output=True)
    found, reads = {}, 0
    for name, (ins, labels) in kernels(open(asm).read()).items():
        reads += sum(i.fills for i in ins)
        bad = early_uses(ins, labels)
        if bad:
            found[name] = bad[:4]
    assert reads > 100
    assert not found, found
