"""LDS reads written as inline asm (`lds_issue_*`): the compiler takes their registers as written at once, and free where it sees no later use, while the
LDS still owes the data.  Every kernel file is compiled to assembly with the build's flags and every path of every kernel is walked:

* no instruction touches a register that a read on its way still owes (LDS answers come in order, so `lgkmcnt(N)` leaves at most the N youngest);
* no read written as asm is on its way into a register that nothing reads any more (the compiler may give it to another value at any time,
  whether or not this build did).

The walk itself is checked on a few lines of assembly that break each rule."""
import os
import re
import subprocess
import textwrap

import pytest

from paper_2407_12117_amd import build as lib_build

FILES = sorted(f for f in lib_build.SOURCES if f.endswith(".hip"))
REG = re.compile(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+)\b)")
WRITES_NOTHING = ("ds_write", "ds_add_u32", "ds_add_f32", "buffer_store", "global_store", "flat_store", "scratch_store", "buffer_atomic", "global_atomic", "v_cmp", "v_readfirstlane",
                  "v_readlane", "s_", "buffer_wbl2", "buffer_inv")


def registers(text):
    out = set()
    for kind, lo, hi, one in REG.findall(text):
        out.update((kind, i) for i in (range(int(lo), int(hi) + 1) if lo else (int(one),)))
    return out


def scalars(text):
    out = set()
    for lo, hi, one in re.findall(r"\bs(?:\[(\d+):(\d+)\]|(\d+)\b)", text):
        out.update(range(int(lo), int(hi) + 1) if lo else (int(one),))
    return out


class Instruction:
    def __init__(self, line, text, in_asm):
        self.line, self.text = line, text
        self.op, _, args = text.partition(" ")
        first, _, rest = args.partition(", ")
        self.is_lds = self.op.startswith("ds_")
        self.is_read = self.op.startswith(("ds_read", "ds_load", "ds_bpermute", "ds_permute", "ds_swizzle"))
        self.asm_read = self.is_read and in_asm
        self.regs = registers(args)
        to_lds = self.op.startswith("buffer_load") and args.endswith(" lds")
        self.writes = set() if to_lds or self.op.startswith(WRITES_NOTHING) else registers(first)
        self.reads = registers(rest) if self.writes else set(self.regs)
        if self.op.startswith(("v_permlane", "v_swap")):
            self.writes = self.reads = self.regs
        elif self.op.startswith(("v_fmac", "v_mac", "v_dot2c", "v_pk_fmac")) or "d16_hi" in self.op or "dst_sel" in args or "_mov_b32_dpp" in self.op:
            self.reads = self.reads | self.writes
        self.wait = None
        if self.op == "s_waitcnt":
            count = re.search(r"lgkmcnt\((\d+)\)", args)
            self.wait = int(count.group(1)) if count else 0 if args.strip() == "0" else None


def kernels(assembly):
    """(name, blocks): a block is (instructions, indices of the blocks that may follow)"""
    name, lines, in_asm = None, [], False
    for number, raw in enumerate(assembly.splitlines(), 1):
        if "#ASMSTART" in raw or "#ASMEND" in raw:
            in_asm = "#ASMSTART" in raw
            continue
        text, _, comment = (" ".join(part.split()) for part in raw.partition(";"))
        if re.match(r"(\.Lfunc_end\w*|\.section)", text) and name:
            yield name, flow(lines)
            name, lines = None, []
        elif re.match(r"[\w.$]+:", text):
            label = text.split(":")[0]
            if name is None and not label.startswith("."):
                name = label
            elif name:
                lines.append(label)
        elif name and text and not text.startswith("."):
            lines.append(Instruction(number, text, in_asm))
            if in_asm:                                 # registers that an asm takes without an instruction of its own using them
                lines[-1].regs |= registers(comment)
                lines[-1].reads |= registers(comment)


def flow(lines):
    blocks, labels = [[]], {}
    for item in lines:
        if isinstance(item, str):
            if blocks[-1]:
                blocks.append([])
            labels[item] = len(blocks) - 1
            continue
        assert item.op not in ("s_setpc_b64", "s_swappc_b64", "s_cbranch_i_fork"), item.text
        blocks[-1].append(item)
        if item.op.startswith(("s_branch", "s_cbranch", "s_endpgm")):
            blocks.append([])
    out = []
    for i, block in enumerate(blocks):
        last = block[-1] if block else None
        follow = []
        if last and last.op.startswith(("s_branch", "s_cbranch")):
            follow.append(labels[last.text.split()[-1]])
        if not (last and last.op in ("s_branch", "s_endpgm")) and i + 1 < len(blocks):
            follow.append(i + 1)
        out.append((block, follow))
    return out


def ways(block, known):
    """The (block, flag) pairs that may follow a block entered with the flag `known`: a scalar pair of all ones or zeros and which it is."""
    instructions, follow = block
    uniform, vcc = {known[0]} if known else set(), None          # pairs that hold all ones or zeros; vcc as a copy of one, or of its inverse
    for ins in instructions:
        written = set() if ins.op.startswith(("s_cmp", "s_cbranch", "s_branch")) else scalars(ins.text.partition(" ")[2].split(", ")[0])
        if known and written & scalars(known[0]):
            known = None
        uniform = {pair for pair in uniform if not written & scalars(pair)}
        if vcc and (written & scalars(vcc[0]) or ins.text.split(",")[0].endswith(" vcc")):
            vcc = None
        flag = re.fullmatch(r"s_cselect_b64 (s\[\d+:\d+\]), -1, 0", ins.text)
        if flag:
            uniform.add(flag.group(1))
        copy = re.fullmatch(r"s_(and|andn2)_b64 vcc, exec, (s\[\d+:\d+\])", ins.text)
        if copy and copy.group(2) in uniform:
            vcc = copy.group(2), copy.group(1) == "and"
    last = instructions[-1].op if instructions else ""
    if last not in ("s_cbranch_vccnz", "s_cbranch_vccz") or vcc is None or len(follow) != 2:
        return [(f, known) for f in follow]
    taken = (last == "s_cbranch_vccnz") == vcc[1]                # the flag's value where the branch is taken
    return [(f, (vcc[0], value)) for f, value in zip(follow, (taken, not taken)) if known is None or known[0] != vcc[0] or known[1] == value]


def faults(blocks):
    """Both rules over one kernel's blocks, as a list of texts."""
    live_in = [set() for _ in blocks]                 # registers that some path reads before it writes them
    changed = True
    while changed:
        changed = False
        for i in reversed(range(len(blocks))):
            block, follow = blocks[i]
            live = set().union(*(live_in[f] for f in follow))
            for ins in reversed(block):
                live = (live - ins.writes) | ins.reads
            if live != live_in[i]:
                live_in[i], changed = live, True
    found = set()

    def walk(i, owed, report):
        """owed: register -> (LDS operations certainly queued behind its read, the read)"""
        block, follow = blocks[i]
        after = []
        if report:
            live = set().union(*(live_in[f] for f in follow))
            for ins in reversed(block):
                after.append(live)
                live = (live - ins.writes) | ins.reads
            after.reverse()
            lost(owed, live_in[i])
        for n, ins in enumerate(block):
            if ins.wait is not None:
                owed = {r: x for r, x in owed.items() if x[0] < ins.wait}
            if report:
                found.update(f"line {ins.line}: `{ins.text}` touches {r[0]}{r[1]}, which `{owed[r][1].text}` of line {owed[r][1].line} still owes"
                             for r in ins.regs & owed.keys())
            if ins.is_lds:
                owed = {r: (count + 1, read) for r, (count, read) in owed.items()}
                if ins.is_read:
                    owed.update((r, (0, ins)) for r in ins.writes)
            if report:
                lost(owed, after[n])
        return owed

    def lost(owed, live):
        found.update(f"line {read.line}: `{read.text}` is on its way into {r[0]}{r[1]}, which nothing reads any more"
                     for r, (_, read) in owed.items() if read.asm_read and r not in live)

    # states by (block, the flag last branched on): a loop left from its middle tests the same flag again behind the join of the two ways
    entry, todo = {(0, None): {}}, [(0, None)]
    while todo:
        at = todo.pop()
        owed = walk(at[0], entry[at], False)
        for to in ways(blocks[at[0]], at[1]):
            merged = dict(entry.get(to, {}))
            for r, x in owed.items():
                if r not in merged or (x[0], x[1].line) < (merged[r][0], merged[r][1].line):
                    merged[r] = x
            if to not in entry or merged != entry[to]:
                entry[to] = merged
                todo.append(to)
    for (i, _), owed in entry.items():
        walk(i, owed, True)
    return sorted(found)


@pytest.mark.parametrize("source", FILES)
def test_no_register_is_touched_or_given_away_before_its_lds_read_is_there(source):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    res = subprocess.run([hipcc, *lib_build.FLAGS, *lib_build.SOURCES[source], "--cuda-device-only", "-S", "-o", "-", os.path.join(lib_build.CSRC, source)],
                         capture_output=True, text=True, timeout=600)
    assert res.returncode == 0, res.stderr[-4000:]
    found = [f"{name}: {f}" for name, blocks in kernels(res.stdout) for f in faults(blocks)]
    assert not found, "\n".join(found[:40])


READ = ";;#ASMSTART\nds_read_b128 v[4:7], v0\n;;#ASMEND\n"


@pytest.mark.parametrize("body, expect", [
    (READ + "s_waitcnt lgkmcnt(0)\nv_add_f32_e32 v1, v4, v5\nv_add_f32_e32 v1, v6, v7", None),
    (READ + "v_mov_b32_e32 v5, 0\ns_waitcnt lgkmcnt(0)\nv_add_f32_e32 v1, v4, v6\nv_add_f32_e32 v1, v5, v7", "still owes"),
    (READ + "ds_write_b32 v0, v1\ns_waitcnt lgkmcnt(1)\nv_mfma_f32_4x4x1_16b_f32 a[0:3], v[4:5], v[6:7], 0", None),
    (READ + "ds_write_b32 v0, v1\ns_waitcnt lgkmcnt(2)\nv_mfma_f32_4x4x1_16b_f32 a[0:3], v[4:5], v[6:7], 0", "still owes"),
    # read again in the loop, but not on the way out of it
    (".LBB0_1:\n" + READ + "s_cbranch_scc0 .LBB0_2\ns_waitcnt lgkmcnt(0)\nv_mfma_f32_4x4x1_16b_f32 a[0:3], v[4:5], v[6:7], 0\ns_branch .LBB0_1\n.LBB0_2:\ns_nop 0",
     "nothing reads any more"),
    (READ + ";;#ASMSTART\ns_waitcnt lgkmcnt(0) ; v[4:7]\n;;#ASMEND", None),
    (".LBB0_1:\n" + READ + "s_waitcnt lgkmcnt(0)\ns_cbranch_scc0 .LBB0_2\nv_mfma_f32_4x4x1_16b_f32 a[0:3], v[4:5], v[6:7], 0\ns_branch .LBB0_1\n.LBB0_2:\ns_nop 0", None),
])
def test_the_walk_finds_what_it_is_for(body, expect):
    assembly = "kernel:\n" + textwrap.indent(body, "\t").replace("\t.LBB0_1:", ".LBB0_1:").replace("\t.LBB0_2:", ".LBB0_2:") + "\n\ts_endpgm\n.Lfunc_end0:\n"
    found = [f for _, blocks in kernels(assembly) for f in faults(blocks)]
    assert any(expect in f for f in found) if expect else not found, found
