"""Wait states around the attention kernel's O MFMAs.

Those MFMAs are inline assembly, which the compiler's hazard pass does not look into, so what it
guarantees for every other MFMA is checked here on the assembly of the kernels (gfx950 needs no GPU to
compile for): two wait states between a vector instruction that writes one of the MFMA's operands and the
MFMA, and, after the MFMA, at least the 18 wait states of the longest MFMA before anything but another
MFMA touches its result.  The copies from memory to LDS are inline assembly too: one wait state behind a
scalar write of M0, five behind a vector instruction that writes one of their scalar operands."""
import os
import re
import subprocess

import pytest

from paper_2603_06664_amd import build

OPERAND_WAITS = 2
RESULT_WAITS = 18
M0_WAITS = 1
SCALAR_WAITS = 5

_REG = re.compile(r"\b([av])(?:\[(\d+):(\d+)\]|(\d+))(?![\w\]])")


def _regs(text):
    out = set()
    for kind, lo, hi, one in _REG.findall(text):
        first, last = (int(one), int(one)) if one else (int(lo), int(hi))
        out.update((kind, i) for i in range(first, last + 1))
    return out


_SREG = re.compile(r"\bs(?:\[(\d+):(\d+)\]|(\d+))(?![\w\]])")


def _scalar_regs(text):
    out = set()
    for lo, hi, one in _SREG.findall(text):
        out.update(range(int(lo or one), int(hi or one) + 1))
    return out


class Ins:
    def __init__(self, text, in_asm):
        self.text, self.in_asm = text, in_asm
        self.op, _, rest = text.partition(" ")
        ops, depth, cur = [], 0, ""
        for ch in rest:
            depth += ch == "["
            depth -= ch == "]"
            if ch == "," and depth == 0:
                ops.append(cur)
                cur = ""
            else:
                cur += ch
        ops.append(cur)
        self.mfma = self.op.startswith("v_mfma")
        self.copy = self.op.startswith("global_load_lds") or (self.op.startswith("buffer_load") and rest.endswith("lds"))
        self.first = ops[0].strip()
        self.scalar = _scalar_regs(rest) if self.copy else set()
        self.vector_writes_scalar = _scalar_regs(self.first) if self.op.startswith("v_") else set()
        self.regs = _regs(rest)
        n_dst = 0 if not self.op.startswith("v_") or self.op.startswith("v_cmp") else 2 if "swap" in self.op else 1
        self.writes = _regs(",".join(ops[:n_dst]))
        # a copy that its inline-assembly branch may skip counts for nothing
        self.waits = int(rest, 0) + 1 if self.op == "s_nop" else 0 if in_asm and self.copy else 1
        self.target = rest.strip() if self.op.startswith(("s_cbranch", "s_branch")) else None


def _kernels(asm):
    """name -> instructions and labels (strings) of every kernel in the file."""
    out, name, in_asm = {}, None, False
    for line in asm.splitlines():
        m = re.match(r"^(_Z\w+):", line)
        if m:
            name = m.group(1)
            out[name] = []
            continue
        if name is None:
            continue
        if line.startswith(".Lfunc_end"):
            name = None
            continue
        s = line.strip()
        if s.startswith(";;#ASMSTART") or s.startswith(";;#ASMEND"):
            in_asm = s.startswith(";;#ASMSTART")
            continue
        s = s.split(";")[0].strip()
        if re.match(r"^\.LBB\w+:$", s):
            out[name].append(s[:-1])
        elif s and not s.startswith(".") and not s.endswith(":"):
            out[name].append(Ins(re.sub(r"\s+", " ", s), in_asm))
    return {k: v for k, v in out.items() if any(isinstance(i, Ins) and i.mfma for i in v)}


def _edges(code):
    at = {x: i for i, x in enumerate(code) if isinstance(x, str)}
    succ = [[] for _ in code]
    for i, x in enumerate(code):
        if isinstance(x, Ins) and x.target in at:
            succ[i].append(at[x.target])
        falls = not (isinstance(x, Ins) and (x.op in ("s_endpgm", "s_branch")))
        if falls and i + 1 < len(code):
            succ[i].append(i + 1)
    pred = [[] for _ in code]
    for i, s in enumerate(succ):
        for j in s:
            pred[j].append(i)
    return pred, succ


def _walk(code, edges, start, limit, bad):
    """The first instruction with bad(ins) fewer than `limit` wait states from `start` along `edges`."""
    todo, seen = [(j, 0) for j in edges[start]], {}
    while todo:
        i, waits = todo.pop()
        if waits >= limit or seen.get(i, limit) <= waits:
            continue
        seen[i] = waits
        x = code[i]
        if isinstance(x, Ins):
            if bad(x):
                return x.text
            waits += x.waits
        todo += [(j, waits) for j in edges[i]]
    return None


def faults(asm):
    out = []
    kernels = _kernels(asm)
    for name, code in kernels.items():
        pred, succ = _edges(code)
        for i, x in enumerate(code):
            if isinstance(x, Ins) and x.copy and x.in_asm:
                w = _walk(code, pred, i, M0_WAITS, lambda y: y.first == "m0") or \
                    _walk(code, pred, i, SCALAR_WAITS, lambda y: bool(y.vector_writes_scalar & x.scalar))
                if w:
                    out.append("%s: '%s' too close before '%s'" % (name, w, x.text))
            if not (isinstance(x, Ins) and x.mfma and x.in_asm):
                continue
            w = _walk(code, pred, i, OPERAND_WAITS, lambda y: not y.mfma and bool(y.writes & x.regs))
            if w:
                out.append("%s: '%s' too close before '%s'" % (name, w, x.text))
            result = _regs(x.text.split(",")[0])
            w = _walk(code, succ, i, RESULT_WAITS, lambda y: not y.mfma and bool(y.regs & result))
            if w:
                out.append("%s: '%s' too close behind '%s'" % (name, w, x.text))
    return out, kernels


@pytest.fixture(scope="module")
def attention_asm(tmp_path_factory):
    s = str(tmp_path_factory.mktemp("asm") / "attention.s")
    src = os.path.join(build.CSRC, "attention.hip")
    subprocess.run(["hipcc", *build.FLAGS, *build.SOURCE_FLAGS["attention.hip"], "-S", "--cuda-device-only", src, "-o", s],
                   check=True, stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)
    with open(s) as f:
        return f.read()


def test_planted_faults_are_seen():
    text = "_Zk:\n%s\n;;#ASMSTART\nv_mfma_f32_32x32x16_bf16 a[0:15], v[0:3], v[4:7], a[0:15]\n;;#ASMEND\n%s\ns_endpgm\n.Lfunc_end0:\n"
    ok = "s_nop 1"
    far = "s_nop 15\ns_nop 1"
    assert not faults(text % (ok, far + "\nv_accvgpr_read_b32 v9, a3"))[0]
    for before in ("v_accvgpr_mov_b32 a3, a77\ns_waitcnt lgkmcnt(0)", "v_cvt_pk_bf16_f32 v5, v8, v9",
                   "v_mov_b32_e32 v0, v8\n.LBB0_1:\ns_nop 0"):
        assert len(faults(text % (before, far))[0]) == 1
    assert len(faults(text % (ok, "s_nop 15\ns_nop 0\nv_accvgpr_read_b32 v9, a3"))[0]) == 1
    # the operand is written at the end of a loop body whose head holds the MFMA
    assert len(faults(text % (".LBB0_1:", far + "\nv_mov_b32_e32 v4, v8\ns_cbranch_scc1 .LBB0_1"))[0]) == 1


def test_planted_copy_faults_are_seen():
    text = "_Zk:\nv_mfma_f32_32x32x16_bf16 a[0:15], v[0:3], v[4:7], a[0:15]\n%s\n;;#ASMSTART\n%s\n;;#ASMEND\ns_endpgm\n.Lfunc_end0:\n"
    copy = "s_add_u32 s7, s7, s8\nbuffer_load_dwordx4 v3, s[12:15], s7 offen lds"
    assert not faults(text % ("v_readfirstlane_b32 s14, v0\ns_nop 3\ns_mov_b32 m0, s3", copy))[0]
    assert len(faults(text % ("s_mov_b32 m0, s3", "buffer_load_dwordx4 v3, s[12:15], s7 offen lds"))[0]) == 1
    assert len(faults(text % ("v_readlane_b32 s14, v0, 3\ns_nop 2", copy))[0]) == 1
    assert len(faults(text % ("v_readfirstlane_b32 s7, v0\ns_mov_b32 m0, s3", copy))[0]) == 1


def test_o_mfmas_have_their_wait_states(attention_asm):
    found, kernels = faults(attention_asm)
    assert len(kernels) == 8   # 2 work-group shapes x limited or not x folded or not
    for code in kernels.values():
        assert sum(isinstance(x, Ins) and x.mfma and x.in_asm for x in code) >= 32
        assert sum(isinstance(x, Ins) and x.copy and x.in_asm for x in code) >= 16
    assert not found, "\n".join(found[:20])


def test_projection_copies_have_their_wait_states(tmp_path):
    s = str(tmp_path / "project.s")
    subprocess.run(["hipcc", *build.FLAGS, *build.SOURCE_FLAGS.get("project.hip", []), "-S", "--cuda-device-only",
                    os.path.join(build.CSRC, "project.hip"), "-o", s], check=True, stdout=subprocess.DEVNULL,
                   stderr=subprocess.DEVNULL)
    with open(s) as f:
        found, kernels = faults(f.read())
    assert len(kernels) == 4   # 2 tile widths x norm per head or over the row
    for code in kernels.values():
        assert sum(isinstance(x, Ins) and x.copy and x.in_asm for x in code) >= 48
    assert not found, "\n".join(found[:20])
