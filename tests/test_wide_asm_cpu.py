"""Wait states around the assembly of the wide contraction kernels.

gemm_wide.hip writes its MFMAs, its copies into LDS and m0 in inline assembly,
before which the compiler inserts no wait states of its own.  What the
hardware asks of the instructions around them then depends on register
allocation (spilled scalars are read back by VALU instructions), so it is
checked in the assembly of the very build, over every kernel and across every
branch:

* a scalar register that a VALU instruction writes is read by a copy at the
  earliest five wait states later;
* every copy has m0 written for it, at least one wait state ahead, by the
  copy's own s_add_u32;
* a register that a VALU instruction writes is read by an MFMA at the earliest
  two wait states later;
* what an MFMA writes (16x16x32: 8 passes) is touched by other instructions
  than MFMAs at the earliest eleven wait states later.
"""
import os
import re
import subprocess

import pytest

from paper_2007_00072_amd import build

LOOK = 12  # wait states that the longest of the rules reaches back


def regs(op):
    """Registers an operand names, as (file, number)."""
    out = set()
    for f, lo, hi, one in re.findall(r"\b([sva])(?:\[(\d+):(\d+)\]|(\d+)\b)", op):
        out |= {(f, i) for i in range(int(lo or one), int(hi or one) + 1)}
    if "vcc" in op:
        out |= {("s", "vcc")}
    if re.search(r"\bm0\b", op):
        out.add(("s", "m0"))
    return out


class Ins:
    def __init__(self, line):
        self.line = line
        name, _, rest = line.partition(" ")
        self.name, self.ops = name, [o.strip() for o in rest.split(",")] if rest else []
        self.mfma = name.startswith("v_mfma")
        self.valu = name.startswith("v_") and not self.mfma
        self.copy = name.startswith("buffer_load") and re.search(r"\blds\b", rest) is not None
        self.wait = 1 + (int(self.ops[0], 0) if name == "s_nop" else 0)
        self.regs = regs(rest)
        first = regs(self.ops[0]) if self.ops else set()
        self.writes = first if self.valu or self.mfma else set()
        if self.valu and re.search(r"_co_|v_mad_[ui]64|v_div_scale", name) and len(self.ops) > 1:
            self.writes = first | regs(self.ops[1])
        self.reads = set().union(*[regs(o) for o in self.ops[1:]]) if self.ops[1:] else set()
        self.sets_m0 = name.startswith("s_") and self.ops and self.ops[0] == "m0"


def functions(text):
    """{kernel: [Ins or label]} of the kernels in a device assembly file."""
    kernels = set(re.findall(r"\.amdhsa_kernel (\S+)", text))
    out, cur = {}, None
    for line in text.splitlines():
        line = line.split(";")[0].rstrip() if not line.lstrip().startswith(";") else ""
        m = re.match(r"^([\w.$]+):", line)
        if m:
            if m[1] in kernels:
                cur = out.setdefault(m[1], [])
            elif cur is not None:
                cur.append(m[1])
            continue
        if re.match(r"^\s+\.(section|size|end_amdhsa_kernel)", line):
            cur = None
        body = line.strip()
        if cur is not None and body and not body.startswith("."):
            cur.append(Ins(body))
    return out


def runs(items):
    """The straight runs of instructions that can execute one after another:
    the text order (up to each jump that is always taken) and, for every
    branch, the end of the code before it followed by the code at its target."""
    at = {x: i for i, x in enumerate(items) if isinstance(x, str)}

    def forward(i, n):
        got = []
        while i < len(items) and len(got) < n:
            if not isinstance(items[i], str):
                got.append(items[i])
                if items[i].name in ("s_branch", "s_endpgm", "s_setpc_b64"):
                    break
            i += 1
        return got

    def back(i, n):
        got = []
        while i >= 0 and len(got) < n:
            if not isinstance(items[i], str):
                if got and items[i].name in ("s_branch", "s_endpgm", "s_setpc_b64"):
                    break
                got.append(items[i])
            i -= 1
        return got[::-1]

    cur = []
    for x in items:
        if isinstance(x, str):
            continue
        cur.append(x)
        if x.name in ("s_branch", "s_endpgm", "s_setpc_b64"):
            yield cur, True
            cur = []
    if cur:
        yield cur, True
    for i, x in enumerate(items):
        if not isinstance(x, str) and (x.name == "s_branch" or x.name.startswith("s_cbranch")):
            target = x.ops[0]
            if target in at:
                yield back(i, LOOK) + forward(at[target], LOOK), False


def faults(items):
    bad = []
    for run, whole in runs(items):
        clock, last_m0 = 0, None
        s_written, v_written, m_written = {}, {}, {}
        for x in run:
            if x.copy:
                late = [r for r in x.regs if r in s_written and clock - s_written[r] < 5]
                if late:
                    bad.append(f"copy {late} too early: {x.line}")
                if last_m0 is None:
                    if whole:
                        bad.append(f"copy without m0 of its own: {x.line}")
                elif clock - last_m0 < 1:
                    bad.append(f"copy right after m0: {x.line}")
                last_m0 = None
            if x.mfma:
                late = [r for r in x.reads if r in v_written and clock - v_written[r] < 2]
                if late:
                    bad.append(f"MFMA {late} too early: {x.line}")
            elif not x.name.startswith("s_"):
                late = [r for r in x.regs if r in m_written and clock - m_written[r] < 11]
                if late:
                    bad.append(f"MFMA result {late} touched: {x.line}")
            clock += x.wait
            if x.sets_m0:
                if x.name != "s_add_u32" or last_m0 is not None:
                    bad.append(f"m0 written between a copy's own write and the copy: {x.line}")
                last_m0 = clock
            if x.valu:
                for r in x.writes:
                    (s_written if r[0] == "s" else v_written)[r] = clock
            if x.mfma:
                for r in x.writes:
                    m_written[r] = clock
    return bad


@pytest.fixture(scope="module")
def kernels():
    src, out = os.path.join(build.CSRC, "gemm_wide.hip"), os.path.join(build.BUILD, "gemm_wide.s")
    os.makedirs(build.BUILD, exist_ok=True)
    if not os.path.exists(out) or os.path.getmtime(out) <= build._deps_mtime("gemm_wide.hip"):
        cmd = [build.hipcc(), *build.HIPCC_FLAGS, "--offload-device-only", "-S", src, "-o", out + ".tmp"]
        r = subprocess.run(cmd, capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-2000:]
        os.replace(out + ".tmp", out)
    return functions(open(out).read())


def test_every_kernel_keeps_its_wait_states(kernels):
    wide = {k: v for k, v in kernels.items() if "gemm_wide" in k or "gemm_mid" in k}
    assert len(wide) >= 60
    for name, items in wide.items():
        ins = [x for x in items if not isinstance(x, str)]
        assert sum(x.copy for x in ins) >= 16 and sum(x.mfma for x in ins) >= 64, name
        assert not faults(items), (name, faults(items)[:5])


def test_the_check_sees_each_fault():
    # the rules on lines like the kernels', sound and with one thing wrong each
    sound = ["v_readlane_b32 s5, v1, 0", "v_mov_b32 v9, 0", "s_nop 3", "s_add_u32 m0, s1, 4096",
             "v_mfma_f32_16x16x32_f16 a[0:3], v[8:11], v[12:15], a[0:3]", "buffer_load_dwordx4 v2, s[4:7], s8 offen lds",
             "s_nop 10", "v_accvgpr_read_b32 v3, a0"]

    def check(lines):
        return faults([Ins(x) for x in lines])

    assert not check(sound)
    assert not check(["v_mov_b32 v3, 0"] + sound)
    for gone in (2, 3, 6):
        assert check(sound[:gone] + sound[gone + 1:]), sound[gone]
    assert check(sound[:4] + [sound[5]])                                       # m0 and its copy next to each other
    assert check(sound[:4] + ["s_mov_b32 m0, s2"] + sound[4:])                 # m0 overwritten in between
    assert check(sound[:4] + ["v_mov_b32 v12, 0"] + sound[4:])                 # an MFMA operand written just before
    assert check(["s_nop 0", ".L1"][:1] + sound[:3] + sound[4:])               # a copy with the m0 of none
    # across a branch: the loop's end writes what its head copies with
    loop = [Ins("s_add_u32 m0, s1, 0"), "L", Ins("s_nop 0"), Ins("buffer_load_dwordx4 v2, s[4:7], s8 offen lds"),
            Ins("s_nop 7"), Ins("s_add_u32 m0, s1, 0"), Ins("v_readlane_b32 s5, v1, 0"), Ins("s_cbranch_scc1 L")]
    assert any("too early" in b for b in faults(loop))
