"""Wait states around the inline assembly of the attention kernels, read off the assembly the compiler makes of
them.  The compiler inserts the wait states the hardware asks for between instructions it knows; it looks
into no asm statement.  These rules are checked over every path through every attention kernel:

  exponentials   a v_exp_f32 in a statement is followed in the same statement by an instruction that does not read
                 its result (one wait state before a vector instruction may)
  mfma operands  an MFMA in a statement has two wait states before it in the same statement, so that whatever wrote
                 an operand is that old, and what the statement itself writes before it is no operand of it
  mfma results   nothing but another MFMA touches those of an MFMA in a statement for 20 wait states (what a
                 16-pass MFMA asks for; these have 8); no statement touches those of any other MFMA for as long
  query loads    nothing touches the registers of a load in a statement before the next wait for vmcnt
  tile loads     M0 is written one wait state before the load that uses it; a scalar base address that a vector
                 instruction wrote is five wait states old
"""
import os
import re
import shutil
import subprocess

import pytest

from paper_2603_06199_amd import build as hip_build

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
MFMA_RESULT = 20


class Ins:
    def __init__(self, text, asm):
        self.text, self.asm = text, asm
        self.op, _, rest = text.partition(" ")
        self.args = [a.strip() for a in re.split(r",(?![^\[]*\])", rest)] if rest else []
        dst = 0 if self.op.startswith(("global_store", "ds_write", "global_load_lds", "s_")) else 1
        self.writes = _regs(self.args[:dst])
        self.reads = _regs(self.args[dst:])
        if "permlane32_swap" in self.op or self.op.startswith("v_swap"):
            self.writes = self.reads = _regs(self.args)
        self.valu = self.op.startswith("v_") and "mfma" not in self.op
        self.mfma = "mfma" in self.op
        self.states = int(self.args[0], 0) + 1 if self.op == "s_nop" else 1


def _regs(args):
    out = set()
    for a in args:
        for f, lo, hi, one in re.findall(r"\b([vas])(?:\[(\d+):(\d+)\]|(\d+)\b)", a):
            lo, hi = (int(lo), int(hi)) if lo else (int(one), int(one))
            out.update((f, i) for i in range(lo, hi + 1))
    return out


class Kernel:
    def __init__(self, name, lines):
        self.name, self.ins, labels, self.regions = name, [], {}, []
        region = None
        for line in lines:
            t = line.split(";")[0].strip() if "ASM" not in line else line.strip()
            if "#ASMSTART" in t:
                region = []
            elif "#ASMEND" in t:
                self.regions.append(region)
                region = None
            elif re.match(r"^[\w.$]+:", t):
                labels[t.split(":")[0]] = len(self.ins)
            elif t and not t.startswith("."):
                self.ins.append(Ins(re.sub(r"\s+", " ", t), region is not None))
                if region is not None:
                    region.append(len(self.ins) - 1)
        self.next = []
        for i, n in enumerate(self.ins):
            to = [] if n.op in ("s_branch", "s_endpgm") else [i + 1]
            if n.op.startswith(("s_branch", "s_cbranch")):
                to.append(labels[n.args[0]])
            self.next.append([j for j in to if j < len(self.ins)])

    def after(self, i, depth):
        """Instructions that start fewer than `depth` wait states after instruction i, on any path."""
        seen, todo = {}, [(j, 0) for j in self.next[i]]
        while todo:
            j, at = todo.pop()
            if at >= depth or seen.get(j, depth) <= at:
                continue
            seen[j] = at
            todo += [(k, at + self.ins[j].states) for k in self.next[j]]
        return [self.ins[j] for j in sorted(seen)]


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    if not (os.path.exists(HIPCC) or shutil.which(HIPCC)):
        pytest.skip("needs hipcc")
    out = tmp_path_factory.mktemp("isa") / "flashprefill.s"
    flags = [f for f in hip_build.HIPCC_FLAGS if f not in ("-fPIC", "-shared", "-Wall")]
    subprocess.run([HIPCC] + flags + ["--cuda-device-only", "-S", "-o", str(out)] +
                   [os.path.join(hip_build.CSRC, s) for s in hip_build.SOURCES], check=True, capture_output=True)
    kernels = {}
    for m in re.finditer(r"^(_ZN2fp\w+):.*?\n(.*?)^\s*\.section", out.read_text(), re.S | re.M):
        kernels[m.group(1)] = m.group(2).split("\n")
    return kernels


@pytest.fixture(scope="module")
def attention(assembly):
    kernels = [Kernel(n, lines) for n, lines in assembly.items() if "attn_kernel" in n]
    assert len(kernels) == 10 and all(any(i.mfma for i in k.ins) for k in kernels)
    return kernels


def _fail_if(bad):
    assert not bad, "\n".join(bad[:20])


def test_exponentials(attention):
    n, bad = 0, []
    for k in attention:
        for region in k.regions:
            for at, i in enumerate(region):
                e = k.ins[i]
                if e.op.startswith("v_exp_f32"):
                    n += 1
                    if at + 1 == len(region) or e.writes & k.ins[region[at + 1]].reads:
                        bad.append(f"{k.name}: {e.text}: no wait state behind it in its statement")
    _fail_if(bad)
    assert n >= 10 * 16 * 4


def test_mfma_operands(attention):
    bad = []
    for k in attention:
        for region in k.regions:
            before = 0
            for i in region:
                if k.ins[i].mfma and before < 2:
                    bad.append(f"{k.name}: {k.ins[i].text}: {before} wait states before it in its statement")
                before += k.ins[i].states
        for i, p in enumerate(k.ins):
            if p.valu:
                bad += [f"{k.name}: {p.text} -> {u.text}" for u in k.after(i, 2) if u.mfma and u.asm and u.reads & p.writes]
    _fail_if(bad)


def test_mfma_results(attention):
    n, bad = 0, []
    for k in attention:
        for i, p in enumerate(k.ins):
            if p.mfma:
                n += p.asm
                bad += [f"{k.name}: {p.text} -> {u.text}" for u in k.after(i, MFMA_RESULT)
                        if not u.mfma and (p.asm or u.asm) and (u.reads | u.writes) & p.writes]
    _fail_if(bad)
    assert n >= 2 * 6 * 32        # the S^T products at head dimension 256


def test_query_loads(attention):
    n, bad = 0, []
    for k in attention:
        for i, p in enumerate(k.ins):
            if p.asm and p.op == "global_load_dwordx4":
                n += 1
                todo, seen = list(k.next[i]), set()
                while todo:
                    j = todo.pop()
                    u = k.ins[j]
                    if j in seen or (u.op == "s_waitcnt" and "vmcnt" in u.text):
                        continue
                    seen.add(j)
                    if (u.reads | u.writes) & p.writes:
                        bad.append(f"{k.name}: {p.text} -> {u.text}")
                    todo += k.next[j]
    _fail_if(bad)
    assert n == 2 * (4 + 8 + 8 + 8 + 16)


def test_tile_loads(attention):
    n, bad = 0, []
    for k in attention:
        for region in k.regions:
            ops = [k.ins[i] for i in region]
            if any(o.op.startswith("global_load_lds") for o in ops):
                n += 1
                if not (len(ops) == 3 and ops[0].text.startswith("s_mov_b32 m0") and ops[2].op.startswith("global_load_lds")):
                    bad.append(f"{k.name}: {[o.text for o in ops]}")
        for i, p in enumerate(k.ins):
            sgprs = {r for r in p.writes if r[0] == "s"} if p.valu else set()
            if sgprs:
                bad += [f"{k.name}: {p.text} -> {u.text}" for u in k.after(i, 5)
                        if u.asm and u.op.startswith("global_load") and u.reads & sgprs]
    _fail_if(bad)
    assert n > 100


def test_pooled_key_loads(assembly):
    """The pooling kernel has no more row loads in flight than a full key block has rows for its row groups."""
    for d, block, loads in ((64, 128, 4), (128, 64, 4), (128, 128, 8), (128, 256, 8), (256, 128, 8)):
        lines = [v for n, v in assembly.items() if f"pool_k_kernelILi{d}ELi{block}E" in n]
        assert len(lines) == 1
        assert sum("global_load_dwordx4" in line for line in lines[0]) == loads, (d, block)
